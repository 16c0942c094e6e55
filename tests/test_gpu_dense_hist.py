"""The exact cluster-size histogram where its paths part: sizes below 256
sites are counted per tile and per group of 16 tiles, larger ones go straight
to the histogram; lattices of more than 64 groups fold in k_roots<1>."""
import math

import numpy as np
import pytest

import oracle
import paper_2302_14720_amd as sw

pytestmark = pytest.mark.gpu

BETA_C = math.log(1.0 + math.sqrt(2.0)) / 2.0


def _hist(labels):
    sizes = np.bincount(labels)
    return np.bincount(sizes[sizes > 0], minlength=labels.size + 1).astype(np.uint64)


@pytest.mark.parametrize("L,beta,cold", [
    (32, 0.0, False),        # one 32-wide tile, clusters of one site only
    (64, BETA_C, False),     # one 64-wide tile
    (1056, BETA_C, False),   # 33 x 33 tiles of 32: 69 groups, the last one ragged
    (2048, 0.35, False),     # 64 groups, folded in the same launch
    (2112, BETA_C, True),    # 69 groups of 64-wide tiles, clusters of every size
])
def test_ising(L, beta, cold):
    print(f"\n[case] dense histogram L={L} beta={beta}", flush=True)
    seed, T = 77 + L, oracle.threshold(beta)
    sp = oracle.init(L, seed, cold=cold)
    with sw.Sim(L, beta, 1.0, seed, flags=sw.SW_FLAG_DENSE_HIST, init=sw.SW_INIT_COLD if cold else sw.SW_INIT_HOT) as s:
        for t in range(3):
            rec, _, _, dense = oracle.sweep(L, 1.0, T, seed, t, sp, dense=True)
            s.sweep(1)
            assert np.array_equal(s.cluster_hist(), dense), f"sweep {t}"
        assert s.observables().tobytes() == rec.tobytes()
        assert np.array_equal(s.spins(), sp)


@pytest.mark.parametrize("q,L", [(3, 192), (8, 96), (4, 2112), (5, 1056)])
def test_potts(q, L):
    print(f"\n[case] dense histogram q={q} L={L}", flush=True)
    seed, beta = 31 + q, math.log(1.0 + math.sqrt(q))
    T = oracle.potts_threshold(beta)
    sp = oracle.potts_init(L, seed, q)
    with sw.Sim(L, beta, 1.0, seed, q=q, flags=sw.SW_FLAG_DENSE_HIST) as s:
        for t in range(3):
            _, lab = oracle.potts_sweep(L, 1.0, T, q, seed, t, sp)
            s.sweep(1)
            assert np.array_equal(s.cluster_hist(), _hist(lab)), f"sweep {t}"
        assert np.array_equal(s.spins(), sp)

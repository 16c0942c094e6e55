"""Tile kernels with 4 and with 16 sites per thread on both sides of the line
between them (400 tiles of 64, 256 for Potts, 2304 tiles of 32), Ising and Potts, with and
without labels; one and several bonds, runs that cross many lanes."""
import math

import numpy as np
import pytest

import oracle
import paper_2302_14720_amd as sw

pytestmark = pytest.mark.gpu

BETA_C = math.log(1.0 + math.sqrt(2.0)) / 2.0


@pytest.mark.parametrize("L,tile,q,beta,cold", [
    (64, 64, 0, 0.0, False),
    (64, 64, 0, 3.0, True),       # runs over all lanes of a row
    (96, 32, 0, 0.5, True),
    (64, 64, 3, 0.9, False),
    (32, 32, 7, 1.6, True),
    (1280, 64, 0, BETA_C, False),  # 400 tiles: 4 sites per thread
    (1344, 64, 0, BETA_C, False),  # 441: 16
    (1536, 32, 0, 0.4, False),     # 2304: 4
    (1568, 32, 0, 0.4, True),      # 2401: 16
    (1024, 64, 4, 1.05, False),
    (1088, 64, 2, 0.88, True),
    (1536, 32, 6, 1.2, False),
    (1568, 32, 8, 1.4, False),
])
@pytest.mark.parametrize("flags", [0, sw.SW_FLAG_LABELS])
def test_both_sides(L, tile, q, beta, cold, flags):
    print(f"\n[case] sites per thread L={L} tile={tile} q={q} beta={beta} flags={flags}", flush=True)
    seed, n = 40 + L + q, 3
    with sw.Sim(L, beta, 1.0, seed, tile=tile, q=q, flags=flags, init=sw.SW_INIT_COLD if cold else sw.SW_INIT_HOT) as s:
        s.sweep(n)
        if q:
            T = oracle.potts_threshold(beta)
            sp = oracle.potts_init(L, seed, q, cold=cold)
            ref = oracle.potts_run(L, 1.0, T, q, seed, 0, n - 1, sp)
            rec, lab = oracle.potts_sweep(L, 1.0, T, q, seed, n - 1, sp)
        else:
            T = oracle.threshold(beta)
            sp = oracle.init(L, seed, cold=cold)
            ref = oracle.run(L, 1.0, T, seed, 0, n - 1, sp)
            rec, lab = oracle.sweep(L, 1.0, T, seed, n - 1, sp)[:2]
        assert s.series(0, n).tobytes() == ref.tobytes() + rec.tobytes()
        assert np.array_equal(s.spins(), sp)
        if flags:
            assert np.array_equal(s.labels(), lab)

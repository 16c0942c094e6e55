"""The cubic bricks where they can go wrong: one brick that is its own
neighbour, even and odd numbers of bricks per side (a group of 2x2x2 bricks
cut off by the lattice's end), no bonds (the most nodes a brick can have, all
components single sites), everything bonded (one component of a whole brick),
labels asked for in between, sweeps one by one and together."""
import numpy as np
import pytest

import oracle
import paper_2302_14720_amd as sw

pytestmark = pytest.mark.gpu


def _hist(labels):
    sizes = np.bincount(labels)
    return np.bincount(sizes[sizes > 0], minlength=labels.size + 1).astype(np.uint64)


@pytest.mark.parametrize("L,q,beta,cold", [
    (16, 0, 0.2216544, False),
    (16, 8, 30.0, True),      # one component of 4096 sites
    (32, 0, 0.0, False),      # 1352 nodes in every brick
    (32, 3, 0.5505, False),
    (64, 0, 0.24, True),
    (80, 0, 0.2216544, False),  # five bricks a side
    (80, 5, 0.65, False),
    (112, 2, 0.443, True),
])
def test_bricks_match_oracle(L, q, beta, cold):
    print(f"\n[case] bricks L={L} q={q} beta={beta} cold={cold}", flush=True)
    seed = 600 + L + q
    T = oracle.potts_threshold(beta) if q else oracle.threshold(beta)
    sp = oracle.cubic_init(L, seed, q, cold=cold)
    with sw.Sim(L, beta, 1.0, seed, q=q, dims=3, flags=sw.SW_FLAG_DENSE_HIST,
                init=sw.SW_INIT_COLD if cold else sw.SW_INIT_HOT) as s, \
            sw.Sim(L, beta, 1.0, seed, q=q, dims=3, init=sw.SW_INIT_COLD if cold else sw.SW_INIT_HOT) as plain:
        recs = []
        for t in range(4):
            rec, lab = oracle.cubic_sweep(L, 1.0, T, q, seed, t, sp)[:2]
            recs.append(rec)
            s.sweep(1)
            assert np.array_equal(s.labels(), lab), f"labels, sweep {t}"
            assert np.array_equal(s.cluster_hist(), _hist(lab)), f"histogram, sweep {t}"
            assert np.array_equal(s.spins(), sp), f"spins, sweep {t}"
            assert s.observables().tobytes() == rec.tobytes(), f"record, sweep {t}"
        plain.sweep(4)
        assert np.array_equal(plain.spins(), sp) and np.array_equal(plain.labels(), lab)
        assert b"".join(r.tobytes() for r in plain.series(0, 4)) == b"".join(r.tobytes() for r in recs)

"""The cubic lattice on both sides of the line up to which node unions go straight
to global memory (five bricks a side in the ordered phase, else six), one sweep after another and together:
spins, records, labels and histogram against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2302_14720_amd as sw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [16, 48, 80, 96, 112])
@pytest.mark.parametrize("q,beta,cold", [(0, 0.0, False), (0, 0.2216544, False), (0, 0.4, True), (3, 0.5505, False)])
def test_both_sides(L, q, beta, cold):
    print(f"\n[case] few bricks L={L} q={q} beta={beta} cold={cold}", flush=True)
    seed = 3000 + L + q
    T = oracle.potts_threshold(beta) if q else oracle.threshold(beta)
    init = sw.SW_INIT_COLD if cold else sw.SW_INIT_HOT
    sp = oracle.cubic_init(L, seed, q, cold=cold)
    with sw.Sim(L, beta, 1.0, seed, q=q, dims=3, flags=sw.SW_FLAG_DENSE_HIST, init=init) as s, \
            sw.Sim(L, beta, 1.0, seed, q=q, dims=3, init=init) as plain:
        recs = []
        for t in range(3):
            rec, lab = oracle.cubic_sweep(L, 1.0, T, q, seed, t, sp)[:2]
            recs.append(rec.tobytes())
            s.sweep(1)
            assert s.observables().tobytes() == recs[-1], f"record, sweep {t}"
        sizes = np.bincount(lab)
        assert np.array_equal(s.cluster_hist(), np.bincount(sizes[sizes > 0], minlength=L ** 3 + 1).astype(np.uint64))
        assert np.array_equal(s.labels(), lab) and np.array_equal(s.spins(), sp)
        plain.sweep(3)
        assert plain.series(0, 3).tobytes() == b"".join(recs)
        assert np.array_equal(plain.spins(), sp) and np.array_equal(plain.labels(), lab)

"""Both link orders of the global union, on either side of the critical
coupling and of the 16 groups a side from which it matters, with labels."""
import math

import numpy as np
import pytest

import oracle
import paper_2302_14720_amd as sw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,tile,q,beta", [
    (2048, 32, 0, 0.5),   # 16 groups a side, ordered
    (2048, 32, 0, 0.43),  # not ordered
    (1920, 32, 0, 0.5),   # 15 groups a side
    (3904, 64, 0, 0.46),  # 16 groups a side, the last cut off
    (2080, 32, 8, 1.4),
    (2048, 32, 3, 0.99),
])
def test_orders(L, tile, q, beta):
    print(f"\n[case] link order L={L} tile={tile} q={q} beta={beta}", flush=True)
    seed = 30 + L + q
    with sw.Sim(L, beta, 1.0, seed, tile=tile, q=q, flags=sw.SW_FLAG_LABELS, init=sw.SW_INIT_COLD) as s:
        if q:
            T = oracle.potts_threshold(beta)
            sp = oracle.potts_init(L, seed, q, cold=True)
            recs = [oracle.potts_sweep(L, 1.0, T, q, seed, t, sp)[:2] for t in range(2)]
        else:
            T = oracle.threshold(beta)
            sp = oracle.init(L, seed, cold=True)
            recs = [oracle.sweep(L, 1.0, T, seed, t, sp)[:2] for t in range(2)]
        s.sweep(2)
        assert s.series(0, 2).tobytes() == b"".join(r.tobytes() for r, _ in recs)
        assert np.array_equal(s.spins(), sp)
        assert np.array_equal(s.labels(), recs[-1][1])

"""Results copied to the host around the sizes where the copy changes: one
small slot, one large slot, several slots in turn, several threads; the same
sim reads back different sizes, and the ring's records in two pieces."""
import numpy as np
import pytest

import oracle
import paper_2302_14720_amd as sw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [32, 256, 288, 1024, 1056, 2880, 2912, 4096])
def test_spins_and_labels(L):
    """N = 1 KB .. 16 MB: below and above 64 KB, 1 MB, 8 MB, odd remainders of 1 MB."""
    print(f"\n[case] readback L={L}", flush=True)
    seed, T = 50 + L, oracle.threshold(0.4)
    sp = oracle.init(L, seed)
    with sw.Sim(L, 0.4, 1.0, seed, flags=sw.SW_FLAG_LABELS) as s:
        assert np.array_equal(s.spins(), sp)
        rec, lab, _ = oracle.sweep(L, 1.0, T, seed, 0, sp)
        s.sweep(1)
        assert s.observables().tobytes() == rec.tobytes()
        assert np.array_equal(s.labels(), lab)
        assert np.array_equal(s.spins(), sp)
        assert s.observables().tobytes() == rec.tobytes()


def test_series_across_the_ring_end():
    L, seed, n = 64, 5, 700
    print("\n[case] readback ring", flush=True)
    sp = oracle.init(L, seed)
    ref = oracle.run(L, 1.0, oracle.threshold(0.44), seed, 0, n, sp)
    with sw.Sim(L, 0.44, 1.0, seed, ring=400) as s:
        s.sweep(n)
        assert s.series(n - 400, 400).tobytes() == ref[n - 400:].tobytes()  # 128 KB in two pieces
        assert s.series(n - 1, 1).tobytes() == ref[n - 1:].tobytes()
        assert np.array_equal(s.spins(), sp)

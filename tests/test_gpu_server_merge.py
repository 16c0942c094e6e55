"""A server whose active jobs go past the number of merge workgroups up to which
k_merge is taken, or are joined by one that it cannot take, and back: jobs change
merge in the middle of their chains, and every one of them still runs the
oracle's."""
import math

import numpy as np
import pytest

import oracle
import paper_2302_14720_amd as sw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("late", [[(1024, 0, 3)] * 33, [(1088, 0, 3)]], ids=["528 groups more", "one of 25"])
def test_jobs_change_merge_and_back(late):
    # (L, q, sweeps): 16 groups each, 4 of 32-wide tiles, 1 that never changes
    early = [(1024, 0, 9), (1024, 3, 8), (320, 0, 12), (160, 5, 11), (128, 0, 10)]
    beta = lambda q: math.log(1.0 + math.sqrt(q)) if q else 0.44
    print("\n[case] server merge change", flush=True)
    srv = sw.Server(256 << 20, 64)
    ids = [srv.submit(L, beta(q), seed=100 + i, sweeps=n, q=q) for i, (L, q, n) in enumerate(early)]
    assert srv.step(2) == []
    ids += [srv.submit(L, beta(q), seed=200 + i, sweeps=n, q=q) for i, (L, q, n) in enumerate(late)]
    assert srv.step(1) == []
    left = len(ids)
    while left:
        left -= len(srv.step(4))
    seeds = [100 + i for i in range(len(early))] + [200 + i for i in range(len(late))]
    for i in list(range(len(early))) + [len(early), len(ids) - 1]:
        (L, q, n), seed = (early + late)[i], seeds[i]
        if q:
            sp = oracle.potts_init(L, seed, q)
            ref = oracle.potts_run(L, 1.0, oracle.potts_threshold(beta(q)), q, seed, 0, n, sp)
        else:
            sp = oracle.init(L, seed)
            ref = oracle.run(L, 1.0, oracle.threshold(beta(q)), seed, 0, n, sp)
        assert np.asarray(srv.series(ids[i], 0, n)).tobytes() == ref.tobytes(), (L, q)
        assert np.array_equal(srv.spins(ids[i]), sp), (L, q)

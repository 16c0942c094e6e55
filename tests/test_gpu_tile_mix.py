"""Tile launches that take replicas of several kinds at once (GPU).

A batch or a server whose lattices have both tile widths, or Ising and Potts
jobs, runs all tiles in one kernel while they are few: 64-wide tiles with 16
sites per thread beside 32-wide ones with 4.  Every replica must be, word for
word, the oracle's; above the limit each kind has its own launch
again, and both lead to the same configurations.
"""
import math

import numpy as np
import oracle
import pytest

import paper_2302_14720_amd as sw

pytestmark = pytest.mark.gpu


def _expected(L, beta, seed, n, q):
    if q:
        sp = oracle.potts_init(L, seed, q)
        return oracle.potts_run(L, 1.0, oracle.potts_threshold(beta), q, seed, 0, n, sp).tobytes(), sp
    sp = oracle.init(L, seed, cold=False)
    return oracle.run(L, 1.0, oracle.threshold(beta), seed, 0, n, sp).tobytes(), sp


@pytest.mark.parametrize("q", [None, 3, 8])
@pytest.mark.parametrize("sides", [
    [64, 32],  # one tile of each width
    [96, 128, 160, 576, 1024],  # one-launch merges and a global one
    [1024] * 13 + [1056],  # 4417 tiles: a launch per width
])
def test_batch_of_both_widths(sides, q):
    beta, n = math.log(1.0 + math.sqrt(q)) if q else 0.44, 4
    seeds = [11 + i for i in range(len(sides))]
    b = sw.Batch(sides, beta, 1.0, seeds, q=q)
    b.sweep(n)
    for r in sorted({0, len(sides) // 2, len(sides) - 1}):
        rec, spins = _expected(sides[r], beta, seeds[r], n, q)
        assert np.asarray(b.series(r, 0, n)).tobytes() == rec, (sides[r], q)
        assert np.array_equal(b.spins(r), spins), (sides[r], q)


def test_server_of_four_kinds():
    jobs = [(64, 0.44, 3, 0), (96, 0.44, 4, 0), (128, 1.0, 5, 3), (160, 1.3, 6, 8), (576, 0.5, 7, 0)]
    n = 5
    srv = sw.Server(64 << 20, len(jobs))
    ids = [srv.submit(L, beta, seed=seed, sweeps=n, q=q) for L, beta, seed, q in jobs]
    left = len(ids)
    while left:
        left -= len(srv.step(64))
    for i, (L, beta, seed, q) in zip(ids, jobs):
        rec, spins = _expected(L, beta, seed, n, q)
        assert np.asarray(srv.series(i, 0, n)).tobytes() == rec, (L, q)
        assert np.array_equal(srv.spins(i), spins), (L, q)


def test_batch_of_many_large_replicas():
    """528 merge workgroups: the large replicas take the global merge, the small ones still one launch."""
    sides, n, beta = [1024] * 33 + [256, 64], 2, 0.44
    seeds = [31 + i for i in range(len(sides))]
    b = sw.Batch(sides, beta, 1.0, seeds)
    b.sweep(n)
    for r in (0, 32, 33, 34):
        rec, spins = _expected(sides[r], beta, seeds[r], n, 0)
        assert np.asarray(b.series(r, 0, n)).tobytes() == rec, sides[r]
        assert np.array_equal(b.spins(r), spins), sides[r]

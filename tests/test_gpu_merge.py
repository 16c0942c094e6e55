"""The one-launch merge at the edges of its range: one group of tiles with its
wrap inside, groups cut off by the lattice's end, the largest lattices it
takes and the first it leaves to the global merge, both tile widths, and more
open clusters than level 2 holds in LDS.  Bit for bit against the oracle."""
import math

import numpy as np
import pytest

import oracle
import paper_2302_14720_amd as sw

pytestmark = pytest.mark.gpu

BETA_C = math.log(1.0 + math.sqrt(2.0)) / 2.0


@pytest.mark.parametrize("L,tile,beta,cold", [
    (32, 32, 0.4, False),       # one tile that is its own neighbour
    (128, 32, BETA_C, False),   # 16 tiles, one group
    (160, 32, BETA_C, False),   # 5 tiles a side: groups of 4 and 1
    (256, 64, 0.4, True),       # 16 tiles, one group
    (320, 64, BETA_C, True),    # 5 tiles a side
    (448, 64, 0.5, True),       # 7 tiles a side
    (768, 64, 0.0, False),      # no bonds: nothing open
    (1024, 64, 40.0, True),     # one cluster
    (512, 32, 0.4, False),      # 16 groups of 32-wide tiles: the most
    (544, 32, BETA_C, False),   # 25 groups: the global merge
    (1024, 64, 0.4, False),     # 16 groups of 64-wide tiles: the most
    (1088, 64, BETA_C, False),  # 25 groups: the global merge
    (1536, 64, 0.4, True),
])
def test_ising(L, tile, beta, cold):
    print(f"\n[case] merge L={L} tile={tile} beta={beta} cold={cold}", flush=True)
    seed, n = 70 + L, 6
    sp = oracle.init(L, seed, cold=cold)
    ref = oracle.run(L, 1.0, oracle.threshold(beta), seed, 0, n, sp)
    with sw.Sim(L, beta, 1.0, seed, tile=tile, init=sw.SW_INIT_COLD if cold else sw.SW_INIT_HOT) as s:
        s.sweep(1)
        s.sweep(n - 1)
        assert s.series(0, n).tobytes() == ref.tobytes()
        assert np.array_equal(s.spins(), sp)


@pytest.mark.parametrize("L,q", [(64, 4), (96, 8), (320, 3), (480, 5), (1056, 8)])
def test_potts(L, q):
    print(f"\n[case] merge L={L} q={q}", flush=True)
    seed, n, beta = 90 + L, 6, math.log(1.0 + math.sqrt(q))
    T = oracle.potts_threshold(beta)
    sp = oracle.potts_init(L, seed, q)
    ref = oracle.potts_run(L, 1.0, T, q, seed, 0, n, sp)
    with sw.Sim(L, beta, 1.0, seed, q=q) as s:
        s.sweep(n - 2)
        s.sweep(2)
        assert s.series(0, n).tobytes() == ref.tobytes()
        assert np.array_equal(s.spins(), sp)


@pytest.mark.parametrize("L,tile", [(512, 64), (1024, 64), (1024, 32)])
def test_every_perimeter_site_open(L, tile):
    """A checkerboard whose phase changes from one group of 4x4 tiles to the
    next, at zero temperature: no bond inside a group and one at every site of
    its perimeter -- the most open clusters there can be (16320 at L = 1024
    with 64-wide tiles, more than fit in LDS)."""
    print(f"\n[case] merge perimeter L={L} tile={tile}", flush=True)
    side = 4 * tile
    y, x = np.mgrid[0:L, 0:L]
    sp = (1 - 2 * ((x + y + x // side + y // side) & 1)).astype(np.int8).reshape(-1)
    seed, beta = 3, 40.0
    with sw.Sim(L, beta, 1.0, seed, tile=tile) as s:
        s.set_spins(sp, 7)
        want = sp.copy()
        ref = oracle.run(L, 1.0, oracle.threshold(beta), seed, 7, 2, want)
        s.sweep(2)
        assert s.series(7, 2).tobytes() == ref.tobytes()
        assert np.array_equal(s.spins(), want)


def test_batch_of_all_kinds():
    """Replicas of both tile widths, Ising and Potts, through one merge launch
    beside ones of the global merge."""
    print("\n[case] merge batch", flush=True)
    L = [64, 96, 320, 1056, 1536, 1600, 128, 256]
    q = [0, 3, 8, 0, 0, 0, 4, 0]
    merge = [sw.SW_MERGE_AUTO] * 7 + [sw.SW_MERGE_GLOBAL]
    beta = [0.44 if v == 0 else math.log(1.0 + math.sqrt(v)) for v in q]
    seed = list(range(500, 508))
    with sw.Batch(L, beta, 1.0, seed, q=q, merge=merge) as b:
        b.sweep(3)
        b.sweep(2)
        for r in range(8):
            if q[r]:
                sp = oracle.potts_init(L[r], seed[r], q[r])
                ref = oracle.potts_run(L[r], 1.0, oracle.potts_threshold(beta[r]), q[r], seed[r], 0, 5, sp)
            else:
                sp = oracle.init(L[r], seed[r])
                ref = oracle.run(L[r], 1.0, oracle.threshold(beta[r]), seed[r], 0, 5, sp)
            assert b.series(r, 0, 5).tobytes() == ref.tobytes(), f"replica {r}"
            assert np.array_equal(b.spins(r), sp), f"replica {r}"

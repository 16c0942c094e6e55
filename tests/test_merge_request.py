"""A batch replica whose caller asks for the global merge gets it at every
size, and counts as that: on the CPU by the work maps that its workspace holds,
on the GPU by its bits."""
import numpy as np
import pytest

import oracle
import paper_2302_14720_amd as sw


@pytest.mark.parametrize("L", [128, 320, 512, 1024])
def test_global_merge_is_planned(L):
    """The maps of the global merge (edges, groups of 16 tiles, groups of 4 x 4)
    are longer than k_merge's one entry per group of 4 x 4 tiles."""
    n, nt, ngx = 8, (L // 64) ** 2, -(-(L // 64) // 4)
    sides = np.full(n, L, dtype=np.int32)
    auto, asked = (sw.sw_batch_workspace_bytes(sides, ring=1, merge=m) for m in (sw.SW_MERGE_AUTO, sw.SW_MERGE_GLOBAL))
    words = n * (2 * ngx * (L // 64) + -(-nt // 16))  # what the maps are longer by
    assert asked - auto >= 4 * words - 256


@pytest.mark.parametrize("other,merge", [(1088, sw.SW_MERGE_AUTO), (64, sw.SW_MERGE_GLOBAL)])
def test_beside_a_global_replica_all_large_ones_are(other, merge):
    """Replicas of more than 16 tiles take k_merge only where nothing needs the
    global merge's launches."""
    sides = np.array([1024] * 8 + [other], dtype=np.int32)
    auto = sw.sw_batch_workspace_bytes(sides, ring=1, merge=[sw.SW_MERGE_AUTO] * 8 + [merge])
    asked = sw.sw_batch_workspace_bytes(sides, ring=1, merge=[sw.SW_MERGE_GLOBAL] * 8 + [merge])
    assert auto == asked
    alone = sw.sw_batch_workspace_bytes(sides[:8], ring=1, merge=sw.SW_MERGE_AUTO)
    assert alone < sw.sw_batch_workspace_bytes(sides[:8], ring=1, merge=sw.SW_MERGE_GLOBAL)


@pytest.mark.gpu
def test_global_and_automatic_give_the_same_bits():
    L = [320, 1024, 320, 1024, 96]
    merge = [sw.SW_MERGE_GLOBAL, sw.SW_MERGE_GLOBAL, sw.SW_MERGE_AUTO, sw.SW_MERGE_AUTO, sw.SW_MERGE_GLOBAL]
    seed, n, beta = [7, 8, 7, 8, 9], 4, 0.44
    print("\n[case] merge asked for", flush=True)
    with sw.Batch(L, beta, 1.0, seed, merge=merge) as b:
        b.sweep(3)
        b.sweep(1)
        for r in range(len(L)):
            sp = oracle.init(L[r], seed[r])
            ref = oracle.run(L[r], 1.0, oracle.threshold(beta), seed[r], 0, n, sp)
            assert b.series(r, 0, n).tobytes() == ref.tobytes(), f"replica {r}"
            assert np.array_equal(b.spins(r), sp), f"replica {r}"
        assert [b.replica_merge(r) for r in (0, 1, 4)] == [sw.SW_MERGE_GLOBAL] * 3

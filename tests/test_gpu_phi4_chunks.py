"""The phi^4 update where its chunks of 1024 sites matter: one site past a
chunk's end, whole chunks only, no bonds at all, every aligned link bonded
(one cluster over all chunks), and more chunks than k_phi_record has
workgroups.  Bit for bit against the oracle, as everywhere."""
import numpy as np
import pytest

import oracle
import paper_2302_14720_amd as sw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,kappa,n,cold", [
    (6, 0.0, 4, False),    # 1296 sites: a full and a ragged chunk, single sites
    (8, 0.304, 12, False), # four whole chunks
    (9, 4.0, 6, True),     # 6561 sites, cold: one cluster over all chunks
    (11, 0.25, 6, False),  # 14641 sites
    (28, 4.0, 2, True),    # 601 chunks, 512 record workgroups
])
def test_chunks(L, kappa, n, cold):
    print(f"\n[case] phi4 chunks L={L} kappa={kappa}", flush=True)
    seed = 9100 + L
    phi = oracle.phi4_init(4, L, seed, cold=cold)
    with sw.Phi4(L, kappa, seed, init=sw.SW_INIT_COLD if cold else sw.SW_INIT_HOT) as p:
        for t in range(n):
            rec, lab, _ = oracle.phi4_sweep(4, L, kappa, seed, t, phi)
            p.sweep(1)
            assert p.series(t, 1)[0].tobytes() == rec.tobytes(), f"sweep {t}"
            assert np.array_equal(p.labels(), lab), f"sweep {t}"
        assert np.array_equal(p.field().view(np.uint64), phi.view(np.uint64))
        prof = p.profile(2)
        assert set(prof) == set(sw.PHI4_KERNELS) and p.next_sweep == n + 2

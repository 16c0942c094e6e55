"""Results read into memory of every kind through the C ABI: pageable, pinned,
and a tensor on the device."""
import numpy as np
import pytest

import oracle
import paper_2302_14720_amd as sw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [32, 288, 1056, 2912])  # 1 KB, 83 KB, 1.1 MB, 8.5 MB
def test_spins_into_any_memory(L):
    import torch

    print(f"\n[case] copy into L={L}", flush=True)
    want = oracle.init(L, 9)
    with sw.Sim(L, 0.4, 1.0, 9) as s:
        for out in (torch.zeros(L * L, dtype=torch.int8), torch.zeros(L * L, dtype=torch.int8, pin_memory=True),
                    torch.zeros(L * L, dtype=torch.int8, device="cuda")):
            torch.cuda.synchronize()
            assert sw.lib().sw_get_spins(s.handle, out.data_ptr(), L * L) == sw.SW_OK
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), want), out.device

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


@pytest.mark.parametrize("threads", [8, 11])  # as many as have pinned memory of their own, and more
def test_threads_read_at_once(threads):
    import threading

    L, n = 2912, 3
    print(f"\n[case] copy from {threads} threads", flush=True)
    sims = [sw.Sim(L, 0.4, 1.0, 20 + i) for i in range(threads)]
    for s in sims:
        s.sweep(n)
    want = [(s.spins(), s.series(0, n)) for s in sims]
    sp = oracle.init(L, 20)
    ref = oracle.run(L, 1.0, oracle.threshold(0.4), 20, 0, n, sp)
    assert np.array_equal(want[0][0], sp) and want[0][1].tobytes() == ref.tobytes()
    bad, start = [], threading.Barrier(threads)

    def read(i):
        start.wait()
        for _ in range(4):
            if not np.array_equal(sims[i].spins(), want[i][0]) or sims[i].series(0, n).tobytes() != want[i][1].tobytes():
                bad.append(i)

    th = [threading.Thread(target=read, args=(i,)) for i in range(threads)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for s in sims:
        s.close()
    assert not bad


def test_spins_on_the_per_thread_stream():
    """A handle that names another stream in every thread (16 MB, read by four)."""
    import torch

    L, n = 4096, 20
    print("\n[case] copy per-thread stream", flush=True)
    sp = oracle.init(L, 3)
    ref = oracle.run(L, 1.0, oracle.threshold(0.44), 3, 0, n, sp)
    cfg = sw.sw_config_init(L, 0.44, 1.0, 3, ring=n)
    ws = torch.empty(sw.sw_workspace_bytes_ex(cfg), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    h = sw.sw_create_ex(cfg, ws.data_ptr(), ws.numel(), 2)
    sw.sw_sweep(h, n)
    assert np.array_equal(sw.sw_get_spins(h, L * L), sp)
    assert sw.sw_series(h, 0, n).tobytes() == ref.tobytes()
    sw.sw_destroy(h)

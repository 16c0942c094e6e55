"""sw_sweep_noalloc takes its spins from device memory, where the host cannot
check them: a byte that is no spin counts as +1, whatever tile looks at it."""
import os
import subprocess

import numpy as np
import pytest

import oracle
import paper_2302_14720_amd as sw

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_EVERY_BYTE = r"""
#include "sw_internal.h"
int main() {
    for (uint32_t b = 0; b < 256u; ++b)
        for (uint32_t o = 0; o < 256u; ++o)
            for (int at = 0; at < 32; at += 8) {
                const uint32_t w = (o * 0x01010101u & ~(0xFFu << at)) | (b << at);
                const uint32_t fb = b == 0xFFu ? 0xFFu : 0x01u, fo = o == 0xFFu ? 0xFFu : 0x01u;
                if (swmi::spin_bytes(w) != ((fo * 0x01010101u & ~(0xFFu << at)) | (fb << at))) return 1;
            }
    return 0;
}
"""


def test_every_byte_becomes_a_spin(tmp_path):
    src, exe = tmp_path / "bytes.cpp", tmp_path / "bytes"
    src.write_text(_EVERY_BYTE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2302_14720_amd", "csrc"),
                    "-o", str(exe), str(src)], check=True)
    assert subprocess.run([str(exe)]).returncode == 0


@pytest.mark.gpu
@pytest.mark.parametrize("L", [64, 96, 512, 1024, 1088, 1696])  # one-launch merges and the global one
@pytest.mark.parametrize("coding", ["0/1", "any"])
def test_bytes_that_are_no_spins(L, coding):
    import torch

    print(f"\n[case] noalloc bytes L={L} {coding}", flush=True)
    rng = np.random.default_rng(L)
    raw = rng.integers(0, 2 if coding == "0/1" else 256, L * L, dtype=np.uint8)
    want = np.where(raw == 0xFF, -1, 1).astype(np.int8)
    ref = oracle.run(L, 1.0, oracle.threshold(0.44), 5, 3, 1, want)
    dev = torch.from_numpy(raw).to("cuda")
    rec = torch.zeros(sw.OBS_DTYPE.itemsize, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    sw.sw_sweep_noalloc(L, 0.44, 1.0, 5, 3, dev.data_ptr(), rec.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert np.array_equal(dev.cpu().numpy().view(np.int8), want)
    assert rec.cpu().numpy().tobytes() == ref.tobytes()

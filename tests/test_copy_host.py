"""The read-back of csrc/sw_copy.hip on the CPU, against a stand-in for the HIP
runtime (tests/copy_host.cpp): every copy has to come after the caller's work
in stream order, whatever stream the caller uses, and goes straight to memory
that the device reaches by itself; reading again makes no pinned memory, from
however many threads and devices."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = tmp_path_factory.mktemp("copy_host") / "copy_host"
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2302_14720_amd", "csrc"),
                    "-o", str(exe), os.path.join(ROOT, "tests", "copy_host.cpp")], check=True)
    return str(exe)


@pytest.mark.parametrize("scenario", ["stream", "null_stream", "per_thread_stream", "into_mapped",
                                      "eight_threads", "more_threads", "six_devices"])
def test_read_back(program, scenario):
    res = subprocess.run([program, scenario], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout + res.stderr

"""What a kernel needs once per device (csrc/zo_device_once.h), compiled for the host against a stand-in for the runtime: each
device gets its own call, a failed call is made again, devices past the bit mask are served every time."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "zo_device_once.h"
#include <cstdio>
static int current = 0;
extern "C" hipError_t hipGetDevice(int *dev) { *dev = current; return current < 0 ? hipErrorInvalidDevice : hipSuccess; }
int main()
{
    std::atomic<uint64_t> done{0}, other{0};
    hipError_t answer = hipSuccess;
    int calls = 0;
    auto at = [&](std::atomic<uint64_t> &mask, int dev) { current = dev; return zo::once_per_device(mask, [&] { ++calls; return answer; }); };
    auto expect = [&](const char *what, bool ok, int n) { if (!ok || calls != n) { printf("%s: %d calls\n", what, calls); return false; } calls = 0; return true; };
    bool ok = true;
    ok &= expect("first device", at(done, 0) == hipSuccess && at(done, 0) == hipSuccess, 1);
    ok &= expect("second device", at(done, 5) == hipSuccess && at(done, 5) == hipSuccess && at(done, 0) == hipSuccess, 1);
    ok &= expect("last bit", at(done, 63) == hipSuccess && at(done, 63) == hipSuccess, 1);
    ok &= expect("past the mask", at(done, 64) == hipSuccess && at(done, 64) == hipSuccess, 2);
    ok &= expect("another kernel", at(other, 0) == hipSuccess, 1);
    answer = hipErrorOutOfMemory;
    ok &= expect("failure is passed on", at(done, 7) == hipErrorOutOfMemory, 1);
    answer = hipSuccess;
    ok &= expect("and tried again", at(done, 7) == hipSuccess && at(done, 7) == hipSuccess, 1);
    ok &= expect("no device", at(done, -1) == hipErrorInvalidDevice, 0);
    return ok ? 0 : 1;
}
"""


def test_once_per_device(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    rocm = next((p for p in (os.environ.get("ROCM_PATH"), "/opt/rocm") if p and os.path.exists(os.path.join(p, "include", "hip"))), None)
    if not cxx or not rocm:
        pytest.skip("no host compiler or no HIP headers")
    src, exe = tmp_path / "once.cpp", tmp_path / "once"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "paper_2507_03211_amd", "csrc"),
                    "-I", os.path.join(rocm, "include"), str(src), "-o", str(exe)], check=True, timeout=120)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stdout

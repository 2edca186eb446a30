"""The cached compute-unit count: each device's own, whichever device was asked
about first, and from several threads at once.  Compiled on the host against
stand-ins for the HIP queries (each thread is on a device of its own); run
under the thread sanitizer where the compiler has it.
"""
import os
import shutil
import subprocess

import pytest

from paper_2607_20652_amd import build

PROGRAM = r"""
#include "dpb_internal.hpp"
#include <cstdio>
#include <thread>
#include <vector>

static thread_local int current = 0;

extern "C" {
hipError_t hipGetDevice(int* d) { *d = current; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int d) { *v = 100 + d; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int d)
{
    p->multiProcessorCount = 100 + d;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
}

int main()
{
    int bad = 0;
    std::vector<int> got(16, 0);
    std::vector<std::thread> threads;
    for (int t = 0; t < 16; ++t)
        threads.emplace_back([&got, t] {
            current = t % 4;
            for (int i = 0; i < 100; ++i) got[t] = dpb::device_cus();
        });
    for (auto& th : threads) th.join();
    for (int t = 0; t < 16; ++t) bad += got[t] != 100 + t % 4;
    std::printf("%d wrong\n", bad);
    return bad ? 1 : 0;
}
"""


def test_compute_units_of_each_device(tmp_path):
    cxx = shutil.which("g++")
    if not cxx or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("no host compiler or HIP headers")
    src, exe = tmp_path / "query.cpp", tmp_path / "query"
    src.write_text(PROGRAM)
    cmd = [cxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{build.CSRC}", "-w",
           str(src), "-o", str(exe), "-pthread"]
    tsan = subprocess.run(cmd + ["-fsanitize=thread"], capture_output=True, text=True)
    if tsan.returncode != 0:
        subprocess.run(cmd, check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and "WARNING: ThreadSanitizer" not in run.stderr, run.stdout + run.stderr[-2000:]

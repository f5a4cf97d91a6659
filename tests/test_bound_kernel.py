"""The launcher of the sweep loops (BoundKernel in lbm_host.hpp) against a
stand-in for the HIP runtime with two devices, on the CPU.  The stand-in's
handles belong to the device that is current when they are looked up, a launch
by handle on a stream of another device fails, and a launch by address takes the
stream's device."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1111_1129_amd", "csrc")
ROCM = "/opt/rocm/include"

SOURCE = r"""
#include "lbm_host.hpp"
#include <cstdio>

static int current = 0, launched_on = -1, sum = 0;
static bool no_kernel = false, no_launch = false;
static hipError_t last = hipSuccess;
static int device_of(hipStream_t s) { return s ? int(reinterpret_cast<uintptr_t>(s) - 0x10) : current; }
static hipError_t fail(hipError_t e) { return last = e; }
static hipError_t ran(int device, void** args) {
    launched_on = device;
    sum = *static_cast<int*>(args[0]) + int(*static_cast<long*>(args[1]));
    return hipSuccess;
}

extern "C" {
hipError_t hipGetDevice(int* d) { *d = current; return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d) { *d = device_of(s); return hipSuccess; }
hipError_t hipGetFuncBySymbol(hipFunction_t* f, const void*) {
    if (no_kernel) return fail(hipErrorInvalidDeviceFunction);
    *f = reinterpret_cast<hipFunction_t>(uintptr_t(0x100 + current));
    return hipSuccess;
}
hipError_t hipModuleLaunchKernel(hipFunction_t f, unsigned, unsigned, unsigned, unsigned, unsigned,
                                 unsigned, unsigned, hipStream_t s, void** args, void**) {
    if (no_launch || int(reinterpret_cast<uintptr_t>(f) - 0x100) != device_of(s))
        return fail(hipErrorInvalidResourceHandle);
    return ran(device_of(s), args);
}
hipError_t hipLaunchKernel(const void*, dim3, dim3, void** args, size_t, hipStream_t s) {
    if (no_kernel || no_launch) return fail(hipErrorInvalidDeviceFunction);
    return ran(device_of(s), args);
}
hipError_t hipGetLastError() { const hipError_t e = last; last = hipSuccess; return e; }
}

static void kernel(int, long) {}
static hipStream_t stream(int device) { return reinterpret_cast<hipStream_t>(uintptr_t(0x10 + device)); }

int main() {
    for (int cur = 0; cur < 2; ++cur)
        for (int own = -1; own < 2; ++own) {
            current = cur;
            launched_on = -1;
            const lbm::BoundKernel k(kernel, dim3(1), dim3(1), own < 0 ? nullptr : stream(own));
            const int st = k(40, 2l);
            std::printf("device %d stream %d: status %d on %d sum %d current %d\n", cur, own, st,
                        launched_on, sum, current);
        }
    current = 0;
    for (int f = 0; f < 2; ++f) {
        (f ? no_launch : no_kernel) = true;
        for (int own = 0; own < 2; ++own) {
            const lbm::BoundKernel k(kernel, dim3(1), dim3(1), stream(own));
            const int st = k(1, 2l);
            std::printf("failure %d stream %d: status %d left %d\n", f, own, st, int(hipGetLastError()));
        }
        no_kernel = no_launch = false;
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def output(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists(os.path.join(ROCM, "hip", "hip_runtime.h")):
        pytest.skip("g++ or the HIP headers are missing")
    d = tmp_path_factory.mktemp("bound")
    src, exe = d / "bound.cpp", d / "bound"
    src.write_text(SOURCE)
    subprocess.run([gxx, "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}",
                    f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}", str(src), "-o", str(exe)],
                   check=True, timeout=300)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True,
                          timeout=60).stdout.splitlines()


@pytest.mark.parametrize("current", [0, 1])
@pytest.mark.parametrize("own", [-1, 0, 1])  # -1: the null stream, the current device's
def test_launches_on_the_device_of_its_stream(output, current, own):
    want = current if own < 0 else own
    assert (f"device {current} stream {own}: status 0 on {want} sum 42 current {current}"
            in output), "\n".join(output)


@pytest.mark.parametrize("failure", [0, 1])  # no such kernel; the launch is refused
@pytest.mark.parametrize("own", [0, 1])
def test_a_failed_call_leaves_no_error_behind(output, failure, own):
    assert f"failure {failure} stream {own}: status -5 left 0" in output, "\n".join(output)

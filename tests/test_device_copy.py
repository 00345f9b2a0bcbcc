"""Cached device lists (windows, work lists) when device memory runs out: the apply
tuning skips a schedule whose list does not fit, so the failing copy must leave
nothing behind.  The header is compiled for the host against a HIP runtime of the
test's own, whose allocations or copies fail on request; it counts what is held."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include <cstdio>
#include <cstdlib>
#include <new>
static long host_held = 0, device_held = 0;
void *operator new(size_t n) { ++host_held; return std::malloc(n); }
void operator delete(void *p) noexcept { if (p) { --host_held; std::free(p); } }
void operator delete(void *p, size_t) noexcept { operator delete(p); }
#define __HIP_PLATFORM_AMD__
#include "%s/paper_1004_3354_amd/csrc/ed_internal.h"
static bool no_memory = false, no_copy = false;
extern "C" {
hipError_t hipMalloc(void **p, size_t n) {
    if (no_memory) return hipErrorOutOfMemory;
    ++device_held;
    *p = std::malloc(n);
    return hipSuccess;
}
hipError_t hipFree(void *p) { --device_held; std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    if (no_copy) return hipErrorInvalidValue;
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipHostFree(void *) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return ""; }
}
namespace ed {
void fail(ed_status st, const char *, ...) { throw Failure{st}; }
void throw_hip(hipError_t, const char *, const char *, int) { throw Failure{ED_EDEVICE}; }
void clear_error() {}
}
int main(int argc, char **argv) {
    no_memory = std::atoi(argv[1]) == 1;
    no_copy = std::atoi(argv[1]) == 2;
    const std::vector<int> list(100, 7);
    int status = ED_OK;
    const long before = host_held;
    try {
        const auto m = ed::device_copy(list);
        if (m->as<int>()[99] != 7 || m->bytes != 400) status = -1;
    } catch (const ed::Failure &f) {
        status = f.st;
    }
    std::printf("%%d %%ld %%ld\n", status, host_held - before, device_held);
}
"""


@pytest.mark.parametrize("fault,status", [(0, 0), (1, 2), (2, 3)], ids=["fits", "no-memory", "copy-fails"])
def test_device_copy_leaves_nothing_behind(tmp_path, fault, status):
    src, exe = tmp_path / "copy.cpp", tmp_path / "copy"
    src.write_text(SRC % ROOT)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I/opt/rocm/include", "-w", str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe), str(fault)], check=True, capture_output=True, text=True).stdout.split()
    assert [int(v) for v in out] == [status, 0, 0]

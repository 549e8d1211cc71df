"""Builds a C++ driver with the library's host code of radio_kernels.hip (its host
pass alone: the planner and the launches, no kernel code), for tests on the CPU.

The driver stands in for the parts of the HIP runtime that this code calls; STUBS has
those that every driver needs.
"""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2302_14812_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

STUBS = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include "radio_internal.h"
static dim3 g_grid, g_block;
extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* p; return &p; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*,
                           void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t)
{
    g_grid = grid; g_block = block;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shmem, hipStream_t* s)
{
    *grid = g_grid; *block = g_block; *shmem = 0; *s = nullptr;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t)
{
    *n = 4;
    return hipSuccess;
}
}
"""


def available():
    return os.path.exists(HIPCC)


def run(tmp, source, defines=()):
    """The standard output of `source` (after STUBS) linked with radio_kernels.hip."""
    drv = tmp / "driver.cpp"
    drv.write_text(STUBS + source)
    common = [HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "--cuda-host-only", "-x", "hip",
              *defines, "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c"]
    objs = []
    for src in (str(drv), os.path.join(CSRC, "radio_kernels.hip")):
        obj = str(tmp / (os.path.basename(src) + ".o"))
        subprocess.run(common + [src, "-o", obj], check=True, capture_output=True)
        objs.append(obj)
    exe = str(tmp / "driver")
    # nothing is launched, so the kernels' code is not linked in
    subprocess.run(["g++"] + objs + ["-Wl,--unresolved-symbols=ignore-all", "-no-pie", "-o", exe],
                   check=True, capture_output=True)
    return subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout

"""The allocation-free batch call asks the HIP runtime for no memory, device or
pinned: the library runs in a process of its own on a stand-in for the runtime
(host memory for device memory, kernels that do nothing) that counts its
allocation calls."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1909_09213_amd", "libcubics.so")

RUNTIME = r"""
#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>
static int calls;
static void *take(size_t n) { ++calls; return calloc(1, n); }
extern "C" {
int allocation_calls() { return calls; }
hipError_t hipMalloc(void **p, size_t n) { *p = take(n); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = take(n); return hipSuccess; }
hipError_t hipFree(void *p) { ++calls; free(p); return hipSuccess; }
hipError_t hipHostFree(void *p) { ++calls; free(p); return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) {
    static void *scratch = calloc(1, (size_t)256 << 20);
    *p = scratch;
    return hipSuccess;
}
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) {
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    p->sharedMemPerBlock = p->maxSharedMemoryPerMultiProcessor = 160 * 1024;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 100000; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 2; return hipSuccess; }
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}
}
"""

USER = r"""
import ctypes, sys
sys.path.insert(0, sys.argv[1])
rt = ctypes.CDLL(sys.argv[2], mode=ctypes.RTLD_GLOBAL)
import numpy as np
import cspgen
from paper_1909_09213_amd import cubics as cb
lib = ctypes.CDLL(cb.LIB_PATH)
lib.cubics_last_error.restype = ctypes.c_char_p
vp = ctypes.c_void_p
ctx, prob = vp(), vp()
assert lib.cubics_create(0, None, ctypes.byref(ctx)) == 0
inst = cspgen.queens(6)
a = cb.Context._arrays(inst)
ptr = lambda x: vp(x.ctypes.data) if x.size else None
assert lib.cubics_load(ctx, inst.n, ptr(a["lo"]), ptr(a["dsize"]), None, inst.m, ptr(a["type"]), ptr(a["arity"]),
                       ptr(a["var_off"]), ptr(a["vars"]), ptr(a["par_off"]), ptr(a["params"]), ptr(a["tab_off"]),
                       ptr(a["tabs"]), ctypes.byref(prob)) == 0
def batch(call, n):
    probs, lims, res = (vp * n)(*[prob.value] * n), (cb.Limits * n)(), (cb._Result * n)()
    for x in lims:
        x.donate = 1
    before = rt.allocation_calls()
    assert call(probs, n, cb.MODE_COUNT, lims, res) == 0, lib.cubics_last_error()
    return rt.allocation_calls() - before
print([batch(lib.cubics_solve_batch_static, n) for n in (1, 3, 700, 2)], batch(lib.cubics_solve_batch, 700) > 0)
"""


@pytest.mark.skipif(not os.path.exists(LIB), reason="libcubics.so not built")
def test_static_batch_makes_no_allocation_call(tmp_path):
    src, rt = tmp_path / "runtime.cpp", tmp_path / "libruntime.so"
    src.write_text(RUNTIME)
    subprocess.check_call(["g++", "-shared", "-fPIC", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           str(src), "-o", str(rt)])
    out = subprocess.run([sys.executable, "-c", USER, ROOT, str(rt)], capture_output=True, text=True)
    assert out.returncode == 0, out.stderr[-2000:]
    assert out.stdout.split("\n")[-2] == "[0, 0, 0, 0] True"

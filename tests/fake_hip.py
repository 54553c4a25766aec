"""HIP memory calls on host memory, for host-side tests of the C ABI without a GPU:
a small shared library that stands in for the runtime's functions the library's
host code calls (its symbols are found before the runtime's).  Allocations are
host memory; fake_words sets what hipPointerGetAttributes says of every pointer,
and a kernel launch and a copy are counted.  run() executes Python code in a
process of its own where ``lib`` is the C library and ``fake`` the stand-in."""
import os
import subprocess
import sys
import textwrap

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
static int g_type, g_device, g_known = 1, g_launches, g_copies;
extern "C" {
void fake_words(int known, int type, int device) { g_known = known; g_type = type; g_device = device; }
int fake_launches() { return g_launches; }
int fake_copies() { return g_copies; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = calloc(1, n ? n : 1); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    g_copies++;
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void*) {
    memset(a, 0, sizeof *a);
    a->type = (hipMemoryType)g_type;
    a->device = g_device;
    return g_known ? hipSuccess : hipErrorInvalidValue;
}
// the status kernel's arguments: overflow word, instance count, host pair
hipError_t hipLaunchKernel(const void*, dim3, dim3, void** args, size_t, hipStream_t) {
    g_launches++;
    int64_t* host = *(int64_t**)args[2];
    host[0] = **(int32_t**)args[0];
    host[1] = **(int64_t**)args[1];
    return hipSuccess;
}
}
"""


def run(tmp_path, code: str) -> str:
    so = os.path.join(tmp_path, "libfakehip.so")
    if not os.path.exists(so):
        src = os.path.join(tmp_path, "fake_hip.cpp")
        with open(src, "w") as f:
            f.write(SOURCE)
        subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", src, "-o", so],
                       check=True)
    prelude = f"""
        import ctypes as C, sys
        sys.path[:0] = [{ROOT!r}, {os.path.join(ROOT, 'tests')!r}]
        fake = C.CDLL({so!r}, mode=C.RTLD_GLOBAL)      # before the library: its calls land here
        from paper_2602_23040_amd import _abi as abi
        lib = abi.lib()
    """
    r = subprocess.run([sys.executable, "-c", textwrap.dedent(prelude) + textwrap.dedent(code)], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout

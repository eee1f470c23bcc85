"""A device allocation that fails, with a host-memory stand-in for the HIP runtime (no GPU).

The stand-in's kernels do nothing and its device memory is host memory, so that only the host
side of the library runs: which buffers it asks for and which calls it accepts."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2603_09277_amd", "libgsr.so")

FAKE = r"""
#include <stdlib.h>
#include <string.h>
size_t fail_above = (size_t)-1;
int n_malloc = 0, n_launch = 0;
int hipMalloc(void** p, size_t n) { if (n > fail_above) return 2; ++n_malloc; *p = calloc(1, n); return 0; }
int hipFree(void* p) { free(p); return 0; }
int hipHostMalloc(void** p, size_t n, unsigned f) { *p = calloc(1, n); return 0; }
int hipHostFree(void* p) { free(p); return 0; }
int hipMemset(void* p, int v, size_t n) { memset(p, v, n); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { memcpy(d, s, n); return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipSetDevice(int d) { return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipStreamSynchronize(void* s) { return 0; }
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int e) { return "stand-in"; }
int hipGetSymbolAddress(void** p, const void* s) { static char m[64]; *p = m; return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { *e = 0; return 0; }
int hipEventDestroy(void* e) { return 0; }
int hipEventRecord(void* e, void* s) { return 0; }
int hipEventSynchronize(void* e) { return 0; }
typedef struct { unsigned x, y, z; } dim3_;
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t m, void* s) { return 0; }
int __hipPopCallConfiguration(dim3_* g, dim3_* b, size_t* m, void** s) { return 0; }
int hipLaunchKernel(const void* f, dim3_ g, dim3_ b, void** a, size_t m, void* s) { ++n_launch; return 0; }
"""

CHILD = r"""
import ctypes as C, sys
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
gsr = C.CDLL(sys.argv[2])
flags = 7 | int(sys.argv[3])
class Cam(C.Structure):
    _fields_ = [("w", C.c_int32), ("h", C.c_int32), ("f", C.c_float * 4), ("R", C.c_float * 9), ("t", C.c_float * 3), ("near", C.c_float)]
class Opts(C.Structure):
    _fields_ = [("v", C.c_int32 * 5), ("flags", C.c_uint32)]
class Gauss(C.Structure):
    _fields_ = [("n", C.c_int64), ("p", C.c_void_p * 5)]
class Out(C.Structure):
    _fields_ = [("p", C.c_void_p * 5), ("frame", C.c_int64)]
class Grads(C.Structure):
    _fields_ = [("p", C.c_void_p * 5)]
cam = Cam(128, 128, (128, 128, 64, 64), (1, 0, 0, 0, 1, 0, 0, 0, 1), (0, 0, 0), 0.2)
opts = Opts((16, 16, 64, 0, 0), flags)
mem = C.create_string_buffer(1 << 20)
ptr = [C.addressof(mem) + 64] * 5
ctx = C.c_void_p()
assert gsr.gsr_create(C.byref(ctx), 1, 0) == 0
limit = C.c_size_t.in_dll(fake, "fail_above")
mallocs, launches = C.c_int.in_dll(fake, "n_malloc"), C.c_int.in_dll(fake, "n_launch")
def forward(n, above=(1 << 64) - 1):
    limit.value, mallocs.value, launches.value = above, 0, 0
    out = Out((C.c_void_p * 5)(*ptr), 0)
    s = gsr.gsr_forward(ctx, None, C.byref(Gauss(n, (C.c_void_p * 5)(*ptr))), C.byref(cam), 1, C.byref(opts), C.byref(out))
    return s, out, mallocs.value
def backward(n, out):
    launches.value = 0
    s = gsr.gsr_backward(ctx, None, C.byref(Gauss(n, (C.c_void_p * 5)(*ptr))), C.byref(cam), 1, C.byref(opts), C.byref(out),
                         C.c_void_p(ptr[0]), None, None, C.byref(Grads((C.c_void_p * 5)(*ptr))))
    return s, launches.value
for n in (100, 100):                    # (a second frame asks for nothing)
    s, old, asked = forward(n)
    assert s == 0
assert asked == 0 and backward(100, old)[0] == 0
# records that do not fit, or only pair rows (a plain frame of 8,000 Gaussians over 64 tiles is
# sized for all of their pairs)
for above in (300_000, 4_000_000) if flags == 7 else (300_000,):
    s, _, _ = forward(8000, above)
    assert s == 6, s
    s, k = backward(100, old)           # an older frame, whose buffers are gone in part
    assert s != 0 and k == 0, (s, k)
    s, out, asked = forward(100)        # what was given back is asked for again
    assert s == 0 and asked > 0, (s, asked)
    assert backward(100, out)[0] == 0
    s, old, asked = forward(100)
    assert s == 0 and asked == 0 and backward(100, old)[0] == 0
limit.value = 300_000                   # a pair count's records that do not fit
counts = (C.c_int64 * 1)()
assert gsr.gsr_pair_counts(ctx, None, C.byref(Gauss(50_000, (C.c_void_p * 5)(*ptr))), C.byref(cam), 1, C.byref(opts), counts) == 6
s, k = backward(100, old)
assert s != 0 and k == 0, (s, k)
print("ok")
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    d = tmp_path_factory.mktemp("hip")
    (d / "fake.c").write_text(FAKE)
    (d / "child.py").write_text(CHILD)
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", "-o", str(d / "fake.so"), str(d / "fake.c")], check=True)
    return d


@pytest.mark.parametrize("mode", [0, 32])                  # plain, GSR_NO_SYNC
def test_context_is_usable_after_a_failed_allocation(fake, mode):
    r = subprocess.run([sys.executable, str(fake / "child.py"), str(fake / "fake.so"), LIB, str(mode)], capture_output=True,
                       text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr

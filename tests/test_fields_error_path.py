"""lb_get_fields copies into the caller's arrays: when a later chunk fails, it
returns the error only after the copies already queued have ended.  On the CPU,
against a stand-in for the HIP runtime in which the second chunk's launch
fails; it logs copies (C) and waits (S)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STUB = r"""
#include <stddef.h>
#include <stdint.h>
#include <string.h>
typedef struct { uint32_t x, y, z; } dim;
char log_[4096];
int at_, launches_, fail_at_ = -1;
static int pending_;
static void put(char c) { if (at_ < 4095) log_[at_++] = c; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { memcpy(d, s, n); put('C'); return 0; }
int hipMemsetAsync(void* d, int v, size_t n, void* st) { memset(d, v, n); return 0; }
int hipLaunchKernel(const void* f, dim g, dim b, void** a, size_t m, void* st) {
    return pending_ = launches_++ == fail_at_ ? 9 : 0;
}
int hipGetLastError(void) { int e = pending_; pending_ = 0; return e; }
const char* hipGetErrorString(int e) { return e ? "stand-in failure" : "no error"; }
int hipStreamSynchronize(void* st) { put('S'); return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { *s = (void*)16; return 0; }
int hipStreamDestroy(void* s) { return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { *e = (void*)16; return 0; }
int hipEventDestroy(void* e) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { *v = 256; return 0; }
int __hipPushCallConfiguration(dim g, dim b, size_t m, void* st) { return 0; }
int __hipPopCallConfiguration(dim* g, dim* b, size_t* m, void** st) {
    g->x = g->y = g->z = b->x = b->y = b->z = 1; *m = 0; *st = 0; return 0;
}
"""

RUN = r"""
import ctypes as C, sys
import numpy as np
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
from paper_2403_05443_amd import lbell
lib = C.CDLL(lbell.LIB_PATH)
for name, (res, args) in lbell.SIGNATURES.items():
    getattr(lib, name).restype, getattr(lib, name).argtypes = res, args
i = lambda k: C.c_int.in_dll(stub, k)
log = lambda: bytes((C.c_char * 4096).in_dll(stub, "log_"))[:i("at_").value].decode()
cfg = lbell.Config()
lib.lb_config_default(C.byref(cfg))
n = 80  # 512000 sites: two chunks
boxes = (lbell.Box * 1)(lbell.make_box(n, n, n))
need = lib.lb_arena_bytes(C.byref(cfg), 1, boxes)
arena = np.zeros(need + 256, dtype=np.uint8)
ctx = C.c_void_p()
assert lib.lb_init(C.byref(cfg), 1, boxes, C.c_void_p((arena.ctypes.data + 255) // 256 * 256), need, None,
                   C.byref(ctx)) == 0
assert i("launches_").value > 0  # the library runs on the stand-in
D = C.POINTER(C.c_double)
rho, u = np.zeros(n ** 3), np.zeros(3 * n ** 3)
i("at_").value = 0
assert lib.lb_get_fields(ctx, 0, rho.ctypes.data_as(D), u.ctypes.data_as(D)) == 0
print("whole", log())
i("at_").value, i("fail_at_").value = 0, i("launches_").value + 1
st = lib.lb_get_fields(ctx, 0, rho.ctypes.data_as(D), u.ctypes.data_as(D))
print("failed", st, log(), lib.lb_last_error(ctx).decode())
"""


def test_copies_end_before_an_error_returns(tmp_path):
    (tmp_path / "stub.c").write_text(STUB)
    so = str(tmp_path / "stub.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", str(tmp_path / "stub.c"), "-o", so], check=True)
    r = subprocess.run([sys.executable, "-c", RUN, so, ROOT], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    whole, failed = r.stdout.split("\n")[:2]
    assert whole == "whole CCCCS"
    f = failed.split(None, 3)
    assert f[1] == "-3" and "stand-in failure" in f[3]
    assert f[2] == "CCS"

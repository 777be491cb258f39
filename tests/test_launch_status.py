"""Failed launches are reported, whichever launch of a call it is.  No GPU: a stand-in for the runtime's launch call (compiled
here, loaded in front of the real one in a process of its own) counts the launches and refuses one of them; nothing runs, so
the pointers are numbers."""
import os
import subprocess
import sys

import pytest

from paper_2410_06511_amd import f8

STAND_IN = r"""
static int launches, refused = -1, error;
static unsigned grids[64];
void f8_test_reset(int k) { launches = 0, refused = k, error = 0; }
int f8_test_launches(void) { return launches; }
unsigned f8_test_grid(int k) { return grids[k]; }
int hipLaunchKernel(const void* f, unsigned long long gxy, unsigned gz, unsigned long long bxy, unsigned bz, void** a, unsigned long s, void* st)
{
    (void)f, (void)gxy, (void)gz, (void)bxy, (void)bz, (void)a, (void)s, (void)st;
    if (launches++ != refused) return 0;
    return error = 719;
}
int __hipPushCallConfiguration(unsigned long long gxy, unsigned gz, unsigned long long bxy, unsigned bz, unsigned long s, void* st)
{
    (void)gz, (void)bxy, (void)bz, (void)s, (void)st;
    if (launches < 64) grids[launches] = (unsigned)gxy;
    return 0;
}
int __hipPopCallConfiguration(void* g, void* b, unsigned long* s, void** st) { (void)g, (void)b, *s = 0, *st = 0; return 0; }
int hipGetLastError(void) { int e = error; error = 0; return e; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int what, int d) { (void)what, (void)d; *v = 256; return 0; }
"""

CALLS = r"""
import ctypes as C, sys
stand_in = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
l = C.CDLL(sys.argv[2])

class Q(C.Structure):
    _fields_ = [(n, C.c_void_p) for n in ("q", "q_t", "amax", "scale", "inv_scale", "amax_t", "scale_t", "inv_scale_t")]
class Saved(C.Structure):
    _fields_ = [(n, Q) for n in ("x", "w", "dy")]
class Desc(C.Structure):
    _fields_ = [("M", C.c_int64), ("K", C.c_int64), ("N", C.c_int64), ("granularity", C.c_int), ("grad_format", C.c_int)]
class State(C.Structure):
    _fields_ = [("mode", C.c_int), ("history_len", C.c_int)] + [(n, C.c_void_p) for n in ("hx", "hw", "hdy", "sx", "sw", "sdy")]

top = 1 << 32
def at(nbytes=1 << 24):     # addresses apart from each other
    global top
    top += 2 * nbytes
    return C.c_void_p(top)
def saved(rowwise=False):
    return Saved(*[Q(*[at().value for _ in range(8)]) if rowwise else Q(at().value, None, at().value, at().value, at().value) for _ in range(3)])

M, K, N = 256, 512, 1024
d, rows, sv, svr = Desc(M, K, N, 0, 0), Desc(M, K, N, 1, 0), saved(), saved(True)
delayed = State(1, 16, *[at().value for _ in range(6)])
X, W, Y, dY, dX, dW, amax, other = (at() for _ in range(8))
ws, size, i64, ref = at(1 << 28), C.c_size_t(1 << 28), C.c_int64, C.byref
over_w = saved()
over_w.x.q = W.value        # X's codes over the weight: one after the other
calls = {
    "linear_fwd": lambda: l.f8_linear_fwd(ref(d), X, W, Y, ref(sv), ws, size, None),
    "linear_fwd rowwise": lambda: l.f8_linear_fwd(ref(rows), X, W, Y, ref(svr), ws, size, None),
    "linear_fwd_scaled": lambda: l.f8_linear_fwd_scaled(ref(d), ref(delayed), X, W, Y, ref(sv), ws, size, None),
    "linear_fwd_chained": lambda: l.f8_linear_fwd_chained(ref(d), X, None, W, Y, other, ref(sv), ws, size, None),
    "linear_fwd_chained, known amax": lambda: l.f8_linear_fwd_chained(ref(d), X, amax, W, Y, other, ref(sv), ws, size, None),
    "linear_fwd_chained, known amax, apart": lambda: l.f8_linear_fwd_chained(ref(d), X, amax, W, Y, other, ref(over_w), ws, size, None),
    "linear_bwd": lambda: l.f8_linear_bwd(ref(d), dY, ref(sv), dX, dW, ws, size, None),
    "linear_bwd_chained, known amax": lambda: l.f8_linear_bwd_chained(ref(d), dY, amax, ref(sv), dX, other, dW, ws, size, None),
    "silu_mul_quantise_delayed": lambda: l.f8_silu_mul_quantise_delayed(X, i64(M), i64(K), 0, other, i64(16), amax, ref(sv.x), ws, size, None),
    "rope_qkv": lambda: l.f8_rope_qkv(X, i64(512), i64(M), i64(64), i64(2), i64(1), i64(128), C.c_double(1e4), Y, i64(256), dX, i64(128), dW, None),
    "sdpa_bwd_rows": lambda: l.f8_sdpa_bwd_rows(X, i64(256), W, i64(128), Y, i64(128), dY, i64(256), other, i64(256), amax, i64(1), i64(M), i64(2), i64(1),
                                               i64(128), dX, i64(256), dW, i64(128), at(), i64(128), at(), None, ws, size, None),
}
call = calls[sys.argv[3]]
stand_in.f8_test_reset(-1)
status, n = call(), stand_in.f8_test_launches()
seen = []
for k in range(n):
    stand_in.f8_test_reset(k)
    seen.append(call())
print(status, n, *seen)
"""

# entry point -> launches at the sizes above
LAUNCHES = {
    "linear_fwd": 3, "linear_fwd rowwise": 7, "linear_fwd_scaled": 3, "linear_fwd_chained": 4, "linear_fwd_chained, known amax": 4,
    "linear_fwd_chained, known amax, apart": 5, "linear_bwd": 3, "linear_bwd_chained, known amax": 3, "silu_mul_quantise_delayed": 2,
    "rope_qkv": 1, "sdpa_bwd_rows": 3,
}


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    d = tmp_path_factory.mktemp("stand_in")
    src, so = d / "stand_in.c", d / "stand_in.so"
    src.write_text(STAND_IN)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)
    return str(so)


@pytest.mark.parametrize("call", LAUNCHES)
def test_a_failed_launch_is_reported(stand_in, call):
    r = subprocess.run([sys.executable, "-c", CALLS, stand_in, os.path.abspath(f8.LIB_PATH), call], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    status, n, *seen = map(int, r.stdout.split())
    assert (status, n) == (0, LAUNCHES[call])
    assert seen == [6] * n  # F8_ERR_LAUNCH

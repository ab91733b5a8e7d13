"""The kernel forms that a call takes (csrc/dd_routes.hpp, compiled
by the host compiler), so that tests can say which one they mean to reach."""
import ctypes
import functools
import os
import subprocess
import tempfile

from paper_2405_13226_amd import build as B

CUS = 256  # an MI355X
SRC = """
#include "dd_routes.hpp"
extern "C" {
int fwd(int D, long long n, int L, int c, int d, int cus) { return dd::fwd_key_groups(D, n, L, c, d, cus); }
int dq(int D, long long n, int L, int c, int d, int cus) { return dd::dq_key_groups(D, n, L, c, d, cus); }
int kv(long long n, int L, int c, int d, int cus) { return dd::dkdv_query_groups(n, L, c, d, cus); }
int both(int D, long long n, int L, int c, int r, int cus) { return dd::bwd_together(D, n, L, c, r, cus); }
int gemm(int M, long long N, long long K, int split, int cus) {
    const dd::GemmPlan p = dd::gemm_plan(M, N, K, split, cus);
    return 1000 * p.tile + p.splits;
}
}
"""


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "routes.cpp"), os.path.join(d, "routes.so")
        with open(src, "w") as f:
            f.write(SRC)
        subprocess.run(["g++", *B.CXX_FLAGS, "-shared", "-o", so, src], check=True)
        h = ctypes.CDLL(so)
    n = ctypes.c_longlong
    h.fwd.argtypes = h.dq.argtypes = [ctypes.c_int, n] + [ctypes.c_int] * 4
    h.both.argtypes = [ctypes.c_int, n] + [ctypes.c_int] * 4
    h.kv.argtypes = [n] + [ctypes.c_int] * 4
    h.gemm.argtypes = [ctypes.c_int, n, n] + [ctypes.c_int] * 2
    return h


def blocks(B, L, H):
    return B * H * ((L + 127) // 128)


def forward(B, L, H, D, causal=True, docs=False):
    """Wave groups of the forward: 1, 2 or 4."""
    return _lib().fwd(D, blocks(B, L, H), L, causal, docs, CUS)


def backward(B, L, H, D, causal=True, docs=False, rope=False):
    """"joint", "short", or the wave groups of (dQ, dK/dV)."""
    n = blocks(B, L, H)
    if _lib().both(D, n, L, causal, rope, CUS):
        return "joint"
    if D == 64 and L <= 256 and not rope:
        return "short"
    return (_lib().dq(D, n, L, causal, docs, CUS),
            _lib().kv(n, L, causal, docs, CUS) if D == 64 else 1)


def gemm(M, N, K, split=True):
    """(tile, K splits) of a product; N is the columns of all groups."""
    v = _lib().gemm(M, N, K, split, CUS)
    return ("large", "tall", "small")[v // 1000], v % 1000

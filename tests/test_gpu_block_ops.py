"""GPU parity of the block kernels around the attention (the bf16 GEMM, the
LayerNorm and the SwiGLU of one OpenLM block) through the C ABI, against
plain float64 numpy definitions of the same operations on the same bf16
inputs.

Tolerances: every output is rounded to bf16 once (RMS relative rounding
error 2^-9 / sqrt(3) ~ 1.1e-3 over a binade, measured 1.66e-3 relative L2 on
N(0,1) products); fp32 accumulation adds far less at these depths.  Bound:
relative L2 <= 3e-3 per output.  The LayerNorm parameter gradients (sums
over all rows) and the outputs with a residual (two roundings) use 5e-3.
"""
import numpy as np
import pytest
import torch

from paper_2405_13226_amd import block_ops as ops

import routes
from parity import log, rel_l2

pytestmark = pytest.mark.gpu
RTOL, RTOL2 = 3e-3, 5e-3


def bf16(shape, seed, scale=1.0):
    g = torch.Generator(device="cpu").manual_seed(seed)
    return (torch.randn(shape, generator=g) * scale).to(torch.bfloat16)


def f64(t):
    return t.float().cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("M,N,K,ta,tb", [
    (256, 256, 64, 0, 0), (512, 768, 320, 0, 1), (768, 512, 192, 1, 0),
    (1024, 512, 8192, 1, 0),      # long K: split over several workgroups
    # 40 tile rows (5 per XCD: a band of 4 rows and one of 1) and 11 tile
    # columns (column groups of 8 and 3) in the grouped tile order
    (10240, 2816, 128, 0, 0), (10240, 2816, 128, 0, 1),
    (65536, 2048, 2048, 0, 0),    # the block's output projection at 65,536 tokens
    (2048, 2048, 65536, 1, 0),    # its weight gradient
    (1024, 2048, 16384, 1, 0),    # tall tiles, K split
    (1024, 2048, 16384, 0, 0), (1024, 2048, 16384, 0, 1),
])
def test_gemm(cuda, M, N, K, ta, tb):
    log(f"gemm M={M} N={N} K={K} ta={ta} tb={tb}")
    a = bf16((K, M) if ta else (M, K), M + K)
    b = bf16((N, K) if tb else (K, N), N + K + 1)
    c = ops.gemm(a.to(cuda), b.to(cuda), bool(ta), bool(tb))
    torch.cuda.synchronize()
    if M * N * K > 2 ** 33:  # sampled rows at full size
        rows = np.random.default_rng(0).choice(M, 64, replace=False)
        an = f64(a.t() if ta else a)[rows]
        ref = an @ f64(b.t() if tb else b)
        got = f64(c)[rows]
    else:
        ref = f64(a.t() if ta else a) @ f64(b.t() if tb else b)
        got = f64(c)
    err = rel_l2(got, ref)
    log(f"  rel-L2 {err:.3g}")
    assert err <= RTOL


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("K", [64, 128, 192, 256, 320])
# small tiles; tall tiles (more of them than CUs' halves); one large tile per CU
@pytest.mark.parametrize("M,N", [(256, 512), (2048, 2816), (2048, 8192)])
def test_gemm_short_reductions(cuda, M, N, K, ta, tb):
    # 1 to 5 K steps: the pipelined loops' first, last and odd steps
    a = bf16((K, M) if ta else (M, K), K + 1)
    b = bf16((N, K) if tb else (K, N), K + 2)
    c = ops.gemm(a.to(cuda), b.to(cuda), bool(ta), bool(tb))
    ref = f64(a.t() if ta else a) @ f64(b.t() if tb else b)
    assert rel_l2(f64(c), ref) <= RTOL


@pytest.mark.parametrize("M,N,K,ta,tb,tile", [
    (256, 256, 64, 0, 0, "small"), (256, 256, 64, 0, 1, "small"), (256, 256, 64, 1, 0, "small"),
    (2048, 2816, 64, 0, 0, "tall"), (2048, 2816, 64, 1, 0, "tall"),
    (2048, 8192, 64, 0, 0, "large"), (2048, 8192, 64, 1, 0, "large")])
def test_gemm_wide_row_strides(cuda, M, N, K, ta, tb, tile):
    # Row strides from which eight rows no longer fit 32-bit byte offsets, on
    # the operand with 64 rows (34 GB, of which 64 rows are used); A B^T has
    # none with so few, its A is 2^25 elements a row (17 GB), short of them.
    assert routes.gemm(M, N, K) == (tile, 1)
    ld = (1 << (25 if tb else 28)) + 8
    a = bf16((K, M) if ta else (M, K), 1)
    b = bf16((N, K) if tb else (K, N), 2)
    narrow = (a if ta or tb else b)
    rows, cols = narrow.shape
    flat = torch.empty((rows - 1) * ld + cols, dtype=torch.bfloat16, device=cuda)
    wide = flat.as_strided((rows, cols), (ld, 1))
    wide.copy_(narrow.to(cuda))
    A, Bm = (wide, b.to(cuda)) if ta or tb else (a.to(cuda), wide)
    c = ops.gemm(A, Bm, bool(ta), bool(tb))
    ref = f64(a.t() if ta else a) @ f64(b.t() if tb else b)
    assert rel_l2(f64(c), ref) <= RTOL


def test_gemm_strided_slices_and_residual(cuda):
    # Column slices of wider matrices as operands and output (row strides
    # passed through), and the residual added in place.
    M, K, N, W = 512, 256, 256, 768
    a = bf16((M, K), 1).to(cuda)
    wide = bf16((K, W), 2).to(cuda)
    out = torch.zeros((M, W), dtype=torch.bfloat16, device=cuda)
    res = bf16((M, N), 3).to(cuda)
    acc = res.clone()
    ops.gemm(a, wide[:, 256:512], out=out[:, 512:768])
    ops.gemm(a, wide[:, 0:256], residual=acc, out=acc)
    torch.cuda.synchronize()
    ref = f64(a) @ f64(wide)[:, 256:512]
    assert rel_l2(f64(out)[:, 512:768], ref) <= RTOL
    assert np.all(f64(out)[:, :512] == 0)  # nothing written outside the slice
    ref2 = f64(a) @ f64(wide)[:, 0:256] + f64(res)
    assert rel_l2(f64(acc), ref2) <= RTOL2


# Small, tall and large tiles (one and more per CU, rows ragged over the XCDs).
JOINT = [(256, 256, 64), (512, 768, 192), (2304, 2816, 128), (2048, 1536, 320), (4096, 4096, 192)]


@pytest.mark.parametrize("n", [2, 3])
# the last two split K, on small and (two groups) tall tiles
@pytest.mark.parametrize("M,N,K", JOINT + [(512, 512, 8192), (1024, 1024, 16384)])
def test_gemm_group(cuda, M, N, K, n):
    # both uses: columns of one weight matrix, and weight gradients written
    # into columns of one matrix
    a, w = bf16((M, K), 1).to(cuda), bf16((K, n * N), 2).to(cuda)
    cols = [slice(i * N, (i + 1) * N) for i in range(n)]
    for c, got in zip(cols, ops.gemm_group(a, [w[:, c] for c in cols])):
        assert rel_l2(f64(got), f64(a) @ f64(w[:, c])) <= RTOL
    x, ys = bf16((K, M), 3).to(cuda), [bf16((K, N), 4 + i).to(cuda) for i in range(n)]
    out = torch.zeros((M, n * N + 256), dtype=torch.bfloat16, device=cuda)
    ops.gemm_group(x, ys, trans_a=True, outs=[out[:, c] for c in cols])
    for c, y in zip(cols, ys):
        assert rel_l2(f64(out[:, c]), f64(x).T @ f64(y)) <= RTOL
    assert not out[:, n * N:].any()


@pytest.mark.parametrize("n", [1, 2, 3])
@pytest.mark.parametrize("M,N,K", JOINT)
def test_gemm_sum(cuda, M, N, K, n):
    xs = [bf16((M, K), 1 + i).to(cuda) for i in range(n)]
    w = bf16((N, n * K), 9).to(cuda)
    ws = [w[:, i * K:(i + 1) * K] for i in range(n)]
    got = ops.gemm_sum(xs, ws, trans_b=True)
    assert rel_l2(f64(got), sum(f64(x) @ f64(v).T for x, v in zip(xs, ws))) <= RTOL
    got = ops.gemm_sum(xs, [v.t().contiguous() for v in ws])
    assert rel_l2(f64(got), sum(f64(x) @ f64(v).T for x, v in zip(xs, ws))) <= RTOL


def test_joint_products_of_different_row_strides(cuda):
    # Weights whose strides differ run as one product each: the sum then rounds
    # after every addition, the rest is bit for bit the same.
    M, N, K = 256, 512, 256
    x, w1 = bf16((M, K), 1).to(cuda), bf16((K, N), 2, 0.1).to(cuda)
    w3 = bf16((K, N + 256), 3, 0.1).to(cuda)[:, :N]
    same = [w1, w3.contiguous()]
    for got, want in zip(ops.gemm_swiglu(x, w1, w3), ops.gemm_swiglu(x, *same)):
        assert torch.equal(got, want)
    us = [bf16((M, N), 4).to(cuda), bf16((M, N + 256), 5).to(cuda)[:, :N]]
    got = ops.gemm_sum(us, [w1, w3], trans_b=True)
    assert rel_l2(f64(got), sum(f64(u) @ f64(w).T for u, w in zip(us, same))) <= RTOL2


def test_the_tests_sizes_reach_every_tile():
    short = [(256, 512), (2048, 2816), (2048, 8192)]
    assert [routes.gemm(m, n, 64)[0] for m, n in short] == ["small", "tall", "large"]
    assert routes.gemm(1024, 512, 8192) == ("small", 8)
    assert routes.gemm(2048, 2048, 65536) == ("large", 4)
    assert routes.gemm(1024, 2048, 16384) == ("tall", 4)
    assert routes.gemm(512, 2 * 512, 8192)[1] > 1
    tiles = {routes.gemm(m, f * n, s * k, False)[0] for m, n, k in JOINT for f, s in ((2, 1), (1, 2))}
    assert tiles == {"small", "tall", "large"}


def test_gemm_sum_of_one_pair_takes_no_workspace(cuda):
    # a reduction long enough that a plain product of these sizes is split
    from paper_2405_13226_amd import lib
    M, N, K = 512, 512, 16384
    assert lib().dd_gemm_workspace_bytes(M, N, K) > 0
    x, w = bf16((M, K), 1).to(cuda), bf16((N, K), 2).to(cuda)
    got = ops.gemm_sum([x], [w], trans_b=True)
    assert rel_l2(f64(got), f64(x) @ f64(w).T) <= RTOL


@pytest.mark.parametrize("M,N,K", JOINT)
def test_gemm_swiglu_is_the_products_and_the_swiglu(cuda, M, N, K):
    # bit for bit the separate launches: same sums, same roundings
    x, w1, w3 = bf16((M, K), 1).to(cuda), bf16((K, N), 2, 0.1).to(cuda), bf16((K, N), 3, 0.1).to(cuda)
    u, v, y = ops.gemm_swiglu(x, w1, w3)
    assert torch.equal(u, ops.gemm(x, w1)) and torch.equal(v, ops.gemm(x, w3))
    assert torch.equal(y, ops.swiglu(u, v))
    dy, w2 = bf16((M, K), 4).to(cuda), bf16((N, K), 5, 0.1).to(cuda)
    du, dv = ops.gemm_swiglu_backward(dy, w2, u, v)
    ru, rv = ops.swiglu_backward(u, v, ops.gemm(dy, w2, trans_b=True))
    assert torch.equal(du, ru) and torch.equal(dv, rv)


def ln_ref(x, w, b, dy, dres, eps=1e-5):
    mu = x.mean(1, keepdims=True)
    var = ((x - mu) ** 2).mean(1, keepdims=True)
    rstd = 1 / np.sqrt(var + eps)
    xh = (x - mu) * rstd
    y = xh * w + b
    g = dy * w
    dx = rstd * (g - g.mean(1, keepdims=True) - xh * (g * xh).mean(1, keepdims=True)) + dres
    return y, dx, (dy * xh).sum(0), dy.sum(0), mu[:, 0], rstd[:, 0]


# (edges of the backward's rows per workgroup and of its one-launch column sums)
@pytest.mark.parametrize("rows,d", [(1, 512), (100, 512), (777, 1024), (2048, 1024), (2049, 1024),
                                    (4096, 2048), (8192, 512), (8193, 512), (16384, 2048),
                                    (16385, 2048), (32769, 2048)])
def test_layer_norm(cuda, rows, d):
    x = bf16((rows, d), rows, 2.0) + 0.5
    w, b = bf16((d,), 5) * 0.3 + 1, bf16((d,), 6) * 0.3
    dy, dres = bf16((rows, d), 7), bf16((rows, d), 8)
    X, W_, B_ = x.to(cuda), w.to(cuda), b.to(cuda)
    y, mean, rstd = ops.layer_norm(X, W_, B_)
    dx, dw, db = ops.layer_norm_backward(X, W_, mean, rstd, dy.to(cuda), dres.to(cuda))
    torch.cuda.synchronize()
    ry, rdx, rdw, rdb, rmu, rrs = ln_ref(f64(x), f64(w), f64(b), f64(dy), f64(dres))
    res = {"y": rel_l2(f64(y), ry), "dx": rel_l2(f64(dx), rdx), "dw": rel_l2(f64(dw), rdw),
           "db": rel_l2(f64(db), rdb),
           "mean": float(np.abs(mean.cpu().numpy() - rmu).max()),
           "rstd": float(np.abs(rstd.cpu().numpy() / rrs - 1).max())}
    log(f"  layernorm rows={rows} d={d}: " + "  ".join(f"{k}={v:.3g}" for k, v in res.items()))
    assert res["y"] <= RTOL and res["dx"] <= RTOL2
    assert res["dw"] <= RTOL2 and res["db"] <= RTOL2
    assert res["mean"] <= 1e-5 and res["rstd"] <= 1e-5


@pytest.mark.parametrize("R,C,pad", [(64, 64, 0), (192, 320, 0), (2048, 5632, 0),
                                     (5632, 2048, 64)])
def test_transpose(cuda, R, C, pad):
    # bit-exact against the transposed copy; pad > 0: strided views in and out
    x = bf16((R, C + pad), 7)
    xd = x.to(cuda)[:, pad // 2:pad // 2 + C]
    y = torch.empty((C, R + 2 * pad), dtype=torch.bfloat16, device=cuda)[:, :R]
    ops.transpose(xd, out=y)
    torch.cuda.synchronize()
    ref = x[:, pad // 2:pad // 2 + C].view(torch.int16).numpy().T
    assert np.array_equal(y.cpu().view(torch.int16).numpy(), ref)


def test_swiglu(cuda):
    n = 3 * 1024 * 8 + 64
    u, v, dy = bf16((n,), 1, 3.0), bf16((n,), 2), bf16((n,), 3)
    y = ops.swiglu(u.to(cuda), v.to(cuda))
    du, dv = ops.swiglu_backward(u.to(cuda), v.to(cuda), dy.to(cuda))
    torch.cuda.synchronize()
    U, V, DY = f64(u), f64(v), f64(dy)
    sig = 1 / (1 + np.exp(-U))
    assert rel_l2(f64(y), U * sig * V) <= RTOL
    assert rel_l2(f64(du), DY * V * sig * (1 + U * (1 - sig))) <= RTOL
    assert rel_l2(f64(dv), DY * U * sig) <= RTOL

"""Python binding of the block kernels around the attention (argument
marshalling only): the bf16 GEMM, LayerNorm and SwiGLU of include/dd_attn.h.

Every computation runs in the HIP kernels behind the C ABI; this module
checks tensor metadata, allocates outputs and scratch with torch on the
tensors' device and passes raw pointers, strides and the current stream.
Matrices are 2-D bf16 tensors with unit column stride (row-major, possibly
a column slice of a wider matrix: the row stride is passed through).
"""
from __future__ import annotations

import ctypes

import torch

from ._lib import check, lib
from .attention import _ptr as _p, _stream

LN_EPS = 1e-5


def _mat(t, name):
    if (isinstance(t, torch.Tensor) and t.dim() == 2 and t.is_cuda
            and t.dtype is torch.bfloat16 and t.stride(1) == 1):
        return
    if not isinstance(t, torch.Tensor) or t.dim() != 2:
        raise ValueError(f"{name} must be a 2-D tensor")
    if t.device.type != "cuda" or t.dtype != torch.bfloat16:
        raise ValueError(f"{name} must be a bf16 GPU tensor")
    if t.stride(1) != 1:
        raise ValueError(f"{name} must have unit column stride")


def gemm(a, b, trans_a: bool = False, trans_b: bool = False, residual=None, out=None):
    """op(a) @ op(b) (+ residual) in bf16 with fp32 accumulation.

    op(a) = a, or a.T when ``trans_a`` (a stored [K, M]); op(b) likewise.
    ``out`` (optional) receives the result and may be ``residual`` itself."""
    _mat(a, "a")
    _mat(b, "b")
    M, K = (a.shape[1], a.shape[0]) if trans_a else (a.shape[0], a.shape[1])
    Kb, N = (b.shape[1], b.shape[0]) if trans_b else (b.shape[0], b.shape[1])
    if K != Kb:
        raise ValueError(f"inner dimensions differ: {K} vs {Kb}")
    if out is None:
        out = torch.empty((M, N), dtype=torch.bfloat16, device=a.device)
    _mat(out, "out")
    if tuple(out.shape) != (M, N):
        raise ValueError(f"out has shape {tuple(out.shape)}, expected {(M, N)}")
    if residual is not None:
        _mat(residual, "residual")
        if tuple(residual.shape) != (M, N) or residual.stride(0) != out.stride(0):
            raise ValueError("residual must match out in shape and row stride")
    need = lib().dd_gemm_workspace_bytes(M, N, K)
    ws = torch.empty(max(need, 1), dtype=torch.uint8, device=a.device) if need else None
    st = lib().dd_gemm(_p(a), a.stride(0), int(bool(trans_a)), _p(b), b.stride(0),
                       int(bool(trans_b)), _p(residual), _p(out), out.stride(0), M, N, K,
                       _p(ws), need, _stream(a.device))
    check(st, "dd_gemm")
    return out


def _shared_stride(ts, name):
    """The row stride of matrices of one shape, or None where they differ."""
    for t in ts:
        _mat(t, name)
        if t.shape != ts[0].shape:
            raise ValueError(f"the {name} matrices must agree in shape")
    strides = {t.stride(0) for t in ts}
    return strides.pop() if len(strides) == 1 else None


def _same(ts, name):
    """Matrices of one shape and row stride; returns that stride."""
    ld = _shared_stride(ts, name)
    if ld is None:
        raise ValueError(f"the {name} matrices must agree in row stride")
    return ld


def _array(ts):
    return (ctypes.c_void_p * len(ts))(*(t.data_ptr() for t in ts))


def gemm_group(a, bs, trans_a: bool = False, trans_b: bool = False, outs=None):
    """[op(a) @ op(b) for b in bs] in one launch (at most three of one shape)."""
    _mat(a, "a")
    ldb = _same(bs, "b")
    M, K = (a.shape[1], a.shape[0]) if trans_a else (a.shape[0], a.shape[1])
    Kb, N = (bs[0].shape[1], bs[0].shape[0]) if trans_b else (bs[0].shape[0], bs[0].shape[1])
    if K != Kb:
        raise ValueError(f"inner dimensions differ: {K} vs {Kb}")
    n = len(bs)
    if outs is None:
        outs = [torch.empty((M, N), dtype=torch.bfloat16, device=a.device) for _ in bs]
    ldc = _same(outs, "out")
    if len(outs) != n or tuple(outs[0].shape) != (M, N):
        raise ValueError(f"need {n} outputs of shape {(M, N)}")
    need = lib().dd_gemm_group_workspace_bytes(M, N, K, n)
    ws = torch.empty(need, dtype=torch.uint8, device=a.device) if need else None
    st = lib().dd_gemm_group(_p(a), a.stride(0), int(bool(trans_a)), _array(bs), ldb,
                             int(bool(trans_b)), _array(outs), ldc, n, M, N, K, _p(ws), need,
                             _stream(a.device))
    check(st, "dd_gemm_group")
    return outs


def gemm_sum(as_, bs, trans_b: bool = False):
    """sum of a @ op(b) over the pairs of as_ and bs (at most three), summed in
    fp32 and rounded once.  The launch takes one row stride per side: where they
    differ, the products run one by one, each rounded as it is added."""
    lda, ldb = _shared_stride(as_, "a"), _shared_stride(bs, "b")
    M, K = as_[0].shape
    Kb, N = (bs[0].shape[1], bs[0].shape[0]) if trans_b else (bs[0].shape[0], bs[0].shape[1])
    if K != Kb or len(as_) != len(bs) or len(as_) > 3:
        raise ValueError("need at most three pairs that agree in their inner dimension")
    if lda is None or ldb is None:
        out = gemm(as_[0], bs[0], trans_b=trans_b)
        for a, b in zip(as_[1:], bs[1:]):
            gemm(a, b, trans_b=trans_b, residual=out, out=out)
        return out
    out = torch.empty((M, N), dtype=torch.bfloat16, device=as_[0].device)
    st = lib().dd_gemm_sum(_array(as_), lda, _array(bs), ldb, int(bool(trans_b)), _p(out), N,
                           len(as_), M, N, K, _stream(out.device))
    check(st, "dd_gemm_sum")
    return out


def gemm_swiglu(x, w1, w3):
    """(u, v, silu(u) * v) with u = x @ w1 and v = x @ w3, in one launch
    (one each where the row strides of w1 and w3 differ)."""
    _mat(x, "x")
    ldw = _shared_stride([w1, w3], "w")
    (M, K), (Kw, N) = x.shape, w1.shape
    if K != Kw:
        raise ValueError(f"inner dimensions differ: {K} vs {Kw}")
    if ldw is None:
        u, v = gemm(x, w1), gemm(x, w3)
        return u, v, swiglu(u, v)
    u, v, y = (torch.empty((M, N), dtype=torch.bfloat16, device=x.device) for _ in range(3))
    st = lib().dd_gemm_swiglu(_p(x), x.stride(0), _p(w1), _p(w3), ldw, _p(u), _p(v), _p(y), N,
                              M, N, K, _stream(x.device))
    check(st, "dd_gemm_swiglu")
    return u, v, y


def gemm_swiglu_backward(dy, w, u, v):
    """(du, dv) of silu(u) * v for the upstream gradient dy @ w.T, in one launch."""
    _mat(dy, "dy")
    _mat(w, "w")
    ldu = _same([u, v], "u")
    (M, K), (N, Kw) = dy.shape, w.shape
    if K != Kw or tuple(u.shape) != (M, N):
        raise ValueError("the shapes of dy, w and u do not agree")
    if ldu != N:
        raise ValueError("u and v must be contiguous")
    du, dv = torch.empty_like(u), torch.empty_like(v)
    st = lib().dd_gemm_swiglu_bwd(_p(dy), dy.stride(0), _p(w), w.stride(0), _p(u), _p(v), _p(du),
                                  _p(dv), N, M, N, K, _stream(dy.device))
    check(st, "dd_gemm_swiglu_bwd")
    return du, dv


def transpose(x, out=None):
    """x.T as a bf16 matrix with unit column stride (into ``out`` if given)."""
    _mat(x, "x")
    R, C = x.shape
    if out is None:
        out = torch.empty((C, R), dtype=torch.bfloat16, device=x.device)
    _mat(out, "out")
    if tuple(out.shape) != (C, R):
        raise ValueError(f"out has shape {tuple(out.shape)}, expected {(C, R)}")
    st = lib().dd_transpose(_p(x), x.stride(0), _p(out), out.stride(0), R, C,
                            _stream(x.device))
    check(st, "dd_transpose")
    return out


def layer_norm(x, w, b, eps: float = LN_EPS):
    """(y, mean, rstd) of LayerNorm over the rows of x [rows, d]."""
    _mat(x, "x")
    rows, d = x.shape
    if not x.is_contiguous():
        raise ValueError("x must be contiguous")
    y = torch.empty_like(x)
    mean = torch.empty(rows, dtype=torch.float32, device=x.device)
    rstd = torch.empty(rows, dtype=torch.float32, device=x.device)
    st = lib().dd_layernorm_fwd(_p(x), _p(w), _p(b), _p(y), _p(mean), _p(rstd), rows, d,
                                float(eps), _stream(x.device))
    check(st, "dd_layernorm_fwd")
    return y, mean, rstd


def layer_norm_backward(x, w, mean, rstd, dy, dres=None):
    """(dx, dw, db) of LayerNorm; ``dres`` (optional) is added to dx."""
    rows, d = x.shape
    dx = torch.empty_like(x)
    dw = torch.empty(d, dtype=torch.bfloat16, device=x.device)
    db = torch.empty(d, dtype=torch.bfloat16, device=x.device)
    need = lib().dd_layernorm_bwd_workspace_bytes(rows, d)
    ws = torch.empty(max(need, 16), dtype=torch.uint8, device=x.device)
    st = lib().dd_layernorm_bwd(_p(x), _p(w), _p(mean), _p(rstd), _p(dy.contiguous()),
                                _p(dres), _p(dx), _p(dw), _p(db), rows, d, _p(ws), ws.numel(),
                                _stream(x.device))
    check(st, "dd_layernorm_bwd")
    return dx, dw, db


def swiglu(u, v):
    """silu(u) * v elementwise."""
    y = torch.empty_like(u)
    st = lib().dd_swiglu_fwd(_p(u), _p(v), _p(y), u.numel(), _stream(u.device))
    check(st, "dd_swiglu_fwd")
    return y


def swiglu_backward(u, v, dy):
    """(du, dv) of y = silu(u) * v."""
    du, dv = torch.empty_like(u), torch.empty_like(v)
    st = lib().dd_swiglu_bwd(_p(u), _p(v), _p(dy.contiguous()), _p(du), _p(dv), u.numel(),
                             _stream(u.device))
    check(st, "dd_swiglu_bwd")
    return du, dv

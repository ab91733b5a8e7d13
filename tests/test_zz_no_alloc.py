"""dd_attn_bwd_noalloc (the backward that allocates nothing and takes no
workspace) against dd_attn_bwd with a caller workspace, through the C ABI.

The two run the same kernels, so the outputs must be bit-identical; the
calls come in a row, the later ones with smaller inputs than an earlier one
(the scratch keeps the previous call's contents, which must not matter),
and one at the largest shape the scratch covers (B*H*L = 2^21)."""
import ctypes

import numpy as np
import pytest
import torch

import routes
import synth
import paper_2405_13226_amd as dd
from paper_2405_13226_amd import _lib

from parity import log

pytestmark = pytest.mark.gpu

P = ctypes.c_void_p


def _p(t):
    return P(t.data_ptr())


def run_pair(B, L, H, D, cu, seed, dev):
    lib = _lib.lib()
    log(f"no-alloc backward: B={B} L={L} H={H} D={D} docs={None if cu is None else len(cu) - 1}")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    q, k, v, do = (torch.randn((B, L, H, D), generator=gen, device=dev).to(torch.bfloat16)
                   for _ in range(4))
    docs = dd.DocLens(cu, B * L, dev) if cu is not None else None
    o, lse = dd.forward(q, k, v, causal=True, cu_doclens=docs)
    cup = _p(docs.dev) if docs else None
    nd = docs.n_docs if docs else 0
    stream = P(torch.cuda.current_stream(dev).cuda_stream)
    ref = [torch.empty_like(q) for _ in range(3)]
    got = [torch.full_like(q, float("nan")) for _ in range(3)]
    ws_bytes = lib.dd_attn_bwd_workspace_bytes(B, L, H, D)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device=dev)
    _lib.check(lib.dd_attn_bwd(_p(q), _p(k), _p(v), _p(o), _p(do), _p(lse), *map(_p, ref),
                               B, L, H, D, 1, cup, nd, _p(ws), ws_bytes, stream), "dd_attn_bwd")
    _lib.check(lib.dd_attn_bwd_noalloc(_p(q), _p(k), _p(v), _p(o), _p(do), _p(lse),
                                       *map(_p, got), B, L, H, D, 1, cup, nd, stream),
               "dd_attn_bwd_noalloc")
    torch.cuda.synchronize(dev)
    for name, a, b in zip(("dq", "dk", "dv"), got, ref):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16)), name
    log("  bit-identical")


def test_noalloc_backward_matches_workspace_backward(cuda):
    lens = synth.lognormal_doc_lengths(4, total_tokens=4 * 1000, median=300, sigma=0.9)
    cu = dd.dd.chunk_doclens(lens, 4 * 1000)
    run_pair(4, 1000, 4, 128, cu, 1, cuda)      # first call
    run_pair(2, 300, 3, 64, None, 2, cuda)      # smaller, after it
    run_pair(3, 77, 2, 128, None, 3, cuda)      # smaller again, ragged
    run_pair(2, 200, 2, 64, None, 4, cuda)      # joint launch of a small grid
    assert routes.backward(60, 200, 2, 64) == "short"
    run_pair(60, 200, 2, 64, None, 7, cuda)     # one-kernel short-row path
    assert routes.backward(48, 700, 3, 64) == (1, 1)
    run_pair(48, 700, 3, 64, None, 8, cuda)     # dQ, then dK/dV


def test_noalloc_backward_largest_scratch_shape(cuda):
    run_pair(8, 8192, 32, 64, None, 5, cuda)    # B*H*L = 2^21: the whole scratch
    run_pair(1, 4096, 2, 128, None, 6, cuda)    # then a small call


def test_noalloc_rejects_shapes_beyond_scratch(cuda):
    lib = _lib.lib()
    t = torch.empty(16, dtype=torch.bfloat16, device=cuda)  # never read: rejected first
    st = lib.dd_attn_bwd_noalloc(*([_p(t)] * 9), 8, 8192, 33, 64, 1, None, 0, None)
    assert st == 9 and b"16 MiB" in lib.dd_status_str(st)

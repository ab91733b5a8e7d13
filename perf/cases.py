"""The work that a training or evaluation program has this package do.

Every case is one pass through the public entry points: the attention of one
step of a length bucket (forward and backward, functional or through
autograd, plain, document-masked or with rotary positions), the attention
forward alone, the products of one linear layer, and a whole OpenLM block.
Sizes are the ones of the benchmark and the tests (65,536-token steps of
length buckets, 16 heads, head dims 64 and 128, the OpenLM-1B block) and
their ragged and small neighbours.

    listed()                 the named cases
    draw(rng)                one more case of the same ranges
    prepare(case, seed)      what the program holds before the call
    run(state)               one pass; returns every output whole
    work(case)               bytes and flops that the pass cannot do without
    tolerance(case)          how far another correct implementation may be
    exact(case, seed)        the same outputs in 64 bits by plain torch
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2405_13226_amd as dda
from paper_2405_13226_amd import block_ops, dd
from paper_2405_13226_amd.layer import LN_EPS, OpenLMBlock

ROPE_BASE = 100000.0
DEVICE = "cuda"


def _attn(mode, B, L, H, D, docs=False, rope=False):
    return dict(kind="attn", mode=mode, B=B, L=L, H=H, D=D, docs=docs, rope=rope)


def listed():
    return [
        # the smallest step: launch latency, a few dozen workgroups
        dict(_attn("call", 4, 256, 4, 64), name="attn_tiny"),
        # the shortest bucket of a 65,536-token step: memory and latency
        dict(_attn("call", 256, 256, 16, 64), name="attn_d64_L256"),
        # a short bucket of the 1B model's heads
        dict(_attn("call", 128, 512, 16, 128), name="attn_d128_L512"),
        # the longest bucket at both head dims: matrix-core bound
        dict(_attn("call", 8, 8192, 16, 64), name="attn_d64_L8192"),
        dict(_attn("call", 8, 8192, 16, 128), name="attn_d128_L8192"),
        # the concat-and-chunk baseline: 8192-token rows of web documents
        dict(_attn("call", 8, 8192, 16, 64, docs=True), name="attn_masked_d64"),
        # a length that no tile divides, and a slice count that the 8 XCDs do
        # not divide, through autograd
        dict(_attn("grad", 11, 1531, 12, 64), name="attn_ragged"),
        # a middle bucket of the 1B model as its training step runs it
        dict(_attn("grad", 32, 2048, 16, 128, rope=True), name="attn_rope_d128_L2048"),
        # evaluation of one 4096-token context: forward only, one row
        dict(_attn("eval", 1, 4096, 16, 128, rope=True), name="attn_eval_d128_L4096"),
        # the three products of the query/key/value projection (forward, input
        # gradient, weight gradient) over a quarter step
        dict(kind="linear", T=16384, n_in=2048, n_out=6144, name="linear_qkv"),
        # a block of a small model on a small step
        dict(kind="block", B=4, L=512, d=1024, H=16, hidden=2816, docs=False,
             name="block_small"),
        # the OpenLM-1B block on a whole step
        dict(kind="block", B=32, L=2048, d=2048, H=16, hidden=5632, docs=False,
             name="block_1b"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attn", "attn", "attn", "linear", "block"])
    if kind == "attn":
        D, H = rng.choice([64, 128]), rng.choice([4, 8, 12, 16])
        L = _log_int(rng, 64, 8192)
        if rng.random() < 0.5:  # a bucket length; the others are ragged
            L = 1 << max(6, min(13, L.bit_length() - 1))
        tokens = _log_int(rng, 1024, 65536)
        mode = rng.choice(["call", "grad", "eval"])
        docs = rng.random() < 0.25
        return _attn(mode, max(1, tokens // L), L, H, D, docs=docs,
                     rope=mode == "eval" or (mode == "grad" and rng.random() < 0.5))
    if kind == "linear":
        d = rng.choice([512, 1024, 2048])
        hidden = 256 * (11 * d // 1024)
        n_in, n_out = rng.choice([(d, d), (d, 3 * d), (d, hidden), (hidden, d)])
        return dict(kind="linear", T=256 * _log_int(rng, 4, 256), n_in=n_in, n_out=n_out)
    d = rng.choice([512, 1024, 2048])
    # rows of 16 k tokens, 16 j of them: ragged lengths, B * L a multiple of 256
    L = 16 * _log_int(rng, 4, 128)
    B = 16 * max(1, _log_int(rng, 1024, 32768) // (16 * L))
    return dict(kind="block", B=B, L=L, d=d, H=d // rng.choice([64, 128]),
                hidden=256 * (11 * d // 1024), docs=rng.random() < 0.25)


# ---------------------------------------------------------------------------
# inputs


def _normal(gen, shape, scale=1.0):
    x = torch.randn(shape, generator=gen, device=DEVICE, dtype=torch.float32)
    return (x * scale).to(torch.bfloat16)


def _doc_offsets(case, seed):
    """Document offsets over the B * L tokens: log-normal web document
    lengths (median 600 tokens), or None."""
    if not case["docs"]:
        return None
    total = case["B"] * case["L"]
    rng = np.random.default_rng(seed)
    lens, left = [], total
    while left:
        n = min(left, int(np.clip(np.rint(np.exp(rng.normal(math.log(600.0), 1.2))), 1, 8192)))
        lens.append(n)
        left -= n
    return dd.chunk_doclens(lens, total)


def _inputs(case, seed):
    """The tensors of a pass, by name, from the seed alone."""
    gen = torch.Generator(device=DEVICE).manual_seed(int(seed))
    if case["kind"] == "attn":
        shape = (case["B"], case["L"], case["H"], case["D"])
        names = ["q", "k", "v"] + ([] if case["mode"] == "eval" else ["do"])
        return {n: _normal(gen, shape) for n in names}
    if case["kind"] == "linear":
        T, i, o = case["T"], case["n_in"], case["n_out"]
        return {"x": _normal(gen, (T, i)), "w": _normal(gen, (i, o), 0.02),
                "dy": _normal(gen, (T, o))}
    d, h = case["d"], case["hidden"]
    shape = (case["B"], case["L"], d)
    # the norms' weights and biases near where training starts them
    t = {"x": _normal(gen, shape), "dy": _normal(gen, shape),
         "ln1_w": 1 + _normal(gen, (d,), 0.1), "ln1_b": _normal(gen, (d,), 0.1),
         "w_qkv": _normal(gen, (d, 3 * d), 0.02), "w_o": _normal(gen, (d, d), 0.02),
         "ln2_w": 1 + _normal(gen, (d,), 0.1), "ln2_b": _normal(gen, (d,), 0.1),
         "w_1": _normal(gen, (d, h), 0.02), "w_3": _normal(gen, (d, h), 0.02),
         "w_2": _normal(gen, (h, d), 0.02)}
    return t


_WEIGHTS = ("ln1_w", "ln1_b", "w_qkv", "w_o", "ln2_w", "ln2_b", "w_1", "w_3", "w_2")
_BLOCKS = {}


def _block(case):
    """A block of these sizes.  Its initial weights are drawn on the host,
    which takes far longer than a step, so one per size is the template and
    prepare() gives each state its own copy."""
    key = (case["d"], case["H"], case["hidden"])
    if key not in _BLOCKS:
        _BLOCKS.clear()
        _BLOCKS[key] = OpenLMBlock(*key, rope_base=ROPE_BASE, device="cpu")
    return _BLOCKS[key]


def prepare(case, seed):
    t = _inputs(case, seed)
    state = dict(case=case, t=t, docs=None)
    if case["kind"] == "linear":
        return state
    cu = _doc_offsets(case, seed)
    if cu is not None:  # validated and copied once per step, used by every layer of it
        state["docs"] = dda.DocLens(cu, case["B"] * case["L"], t["x" if "x" in t else "q"].device)
    if case["kind"] == "block":
        import copy
        state["block"] = copy.deepcopy(_block(case)).to(DEVICE)
        with torch.no_grad():
            for n in _WEIGHTS:
                getattr(state["block"], n).copy_(t[n])
        t["x"].requires_grad_(True)
    elif case["mode"] == "grad":
        for n in "qkv":
            t[n].requires_grad_(True)
    return state


# ---------------------------------------------------------------------------
# one pass


def run(state):
    case, t, docs = state["case"], state["t"], state["docs"]
    if case["kind"] == "linear":
        y = block_ops.gemm(t["x"], t["w"])
        dx = block_ops.gemm(t["dy"], t["w"], trans_b=True)
        dw = block_ops.gemm(t["x"], t["dy"], trans_a=True)
        return {"y": y, "dx": dx, "dw": dw}
    if case["kind"] == "block":
        block = state["block"]
        y = block(t["x"], cu_doclens=docs)
        params = [getattr(block, n) for n in _WEIGHTS]
        grads = torch.autograd.grad(y, [t["x"]] + params, t["dy"])
        return dict(zip(("y", "dx") + tuple("d" + n for n in _WEIGHTS),
                        (y.detach(),) + grads))
    q, k, v = t["q"], t["k"], t["v"]
    if case["mode"] == "eval":
        o, lse, _, _ = dda.forward_rope(q, k, v, ROPE_BASE, True, docs)
        return {"o": o, "lse": lse}
    if case["mode"] == "grad":
        o = dda.attention(q, k, v, cu_doclens=docs, rope_base=ROPE_BASE if case["rope"] else None)
        dq, dk, dv = torch.autograd.grad(o, (q, k, v), t["do"])
        return {"o": o.detach(), "dq": dq, "dk": dk, "dv": dv}
    o, lse = dda.forward(q, k, v, True, docs)
    dq, dk, dv = dda.backward(q, k, v, o, lse, t["do"], True, docs)
    return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}


# ---------------------------------------------------------------------------
# what a pass cannot do without


def work(case):
    if case["kind"] == "linear":
        T, i, o = case["T"], case["n_in"], case["n_out"]
        # each of the three calls reads its two operands and writes its result
        return dict(bytes=6 * (T * i + i * o + T * o), flops=6 * T * i * o)
    B, L = case["B"], case["L"]
    # documents: their lengths come from the seed; these are seed 0's pairs
    cu = _doc_offsets(case, 0)
    if case["kind"] == "block":
        T, d, h = B * L, case["d"], case["hidden"]
        f, b = dd.attention_flops(B, L, case["H"], d // case["H"], True, cu)
        weights = 4 * d * d + 3 * d * h
        # x, dy in, y, dx out; the weights read by each direction, their
        # gradients written
        return dict(bytes=2 * (4 * T * d + 3 * weights), flops=6 * T * weights + f + b)
    H, D = case["H"], case["D"]
    f, b = dd.attention_flops(B, L, H, D, True, cu)
    fb, bb = dd.attention_bytes(B, L, H, D)
    if case["mode"] == "eval":
        return dict(bytes=fb, flops=f)
    return dict(bytes=fb + bb, flops=f + b)


def tolerance(case):
    if case["kind"] == "linear":
        # one rounding to bf16 of a 32-bit sum: measured 1.7e-3 from 64 bits;
        # a whole unit in the last place (2^-7) where two roundings part
        return {"rel": 7e-3, "max": 5e-2}
    if case["kind"] == "block":
        # every intermediate tensor is rounded to bf16: measured 3e-3 to 7e-3
        # from 64 bits
        return {"rel": 2e-2, "max": 5e-1}
    # probabilities and their gradients are rounded to bf16 before the second
    # products: measured 2.0e-3 to 3.6e-3 (rotated) from 64 bits
    return {"rel": 1e-2, "max": 2e-1}


# ---------------------------------------------------------------------------
# the same outputs in 64 bits


def _rope64(x, inverse=False):
    """Rotates consecutive pairs (2j, 2j+1) of [B, L, H, D] by pos * base^(-2j/D)."""
    L, D = x.shape[1], x.shape[3]
    j = torch.arange(D // 2, device=x.device, dtype=torch.float64)
    ang = torch.arange(L, device=x.device, dtype=torch.float64)[:, None] * ROPE_BASE ** (-2 * j / D)
    c, s = torch.cos(ang)[None, :, None], torch.sin(ang)[None, :, None]
    if inverse:
        s = -s
    a, b = x[..., 0::2], x[..., 1::2]
    return torch.stack([a * c - b * s, a * s + b * c], -1).reshape(x.shape)


def _attend64(q, k, v, do, cu):
    """(o, lse, dq, dk, dv) in float64 of [B, L, H, D] tensors, a few (b, h)
    slices at a time."""
    B, L, H, D = q.shape
    scale = 1.0 / math.sqrt(D)
    pos = torch.arange(L, device=q.device)
    causal = pos[None, :] > pos[:, None]
    doc = None
    if cu is not None:
        edges = torch.as_tensor(np.asarray(cu[1:], dtype=np.int64), device=q.device)
        doc = torch.bucketize(torch.arange(B * L, device=q.device), edges, right=True).view(B, L)
    o = torch.empty_like(q)
    lse = torch.empty(B, L, H, device=q.device, dtype=torch.float64)
    grads = [torch.empty_like(q) for _ in range(3)] if do is not None else None
    nb = max(1, (1 << 27) // (L * L * H))
    nh = H if nb > 1 else max(1, min(H, (1 << 27) // (L * L)))
    for b0 in range(0, B, nb):
        for h0 in range(0, H, nh):
            at = (slice(b0, b0 + nb), slice(None), slice(h0, h0 + nh))
            Q, K, V = (x[at].transpose(1, 2).contiguous() for x in (q, k, v))
            s = torch.matmul(Q, K.transpose(-1, -2).contiguous()) * scale
            mask = causal[None, None]
            if doc is not None:
                e = doc[b0:b0 + nb]
                mask = mask | (e[:, None, :] != e[:, :, None])[:, None]
            s.masked_fill_(mask, -math.inf)
            z = torch.logsumexp(s, -1)
            p = s.sub_(z[..., None]).exp_()
            out = torch.matmul(p, V)
            o[at] = out.transpose(1, 2)
            lse[at] = z.transpose(1, 2)
            if do is None:
                continue
            G = do[at].transpose(1, 2).contiguous()
            grads[2][at] = torch.matmul(p.transpose(-1, -2), G).transpose(1, 2)
            dp = torch.matmul(G, V.transpose(-1, -2).contiguous())
            ds = p.mul_(dp.sub_((G * out).sum(-1, keepdim=True))).mul_(scale)
            grads[0][at] = torch.matmul(ds, K).transpose(1, 2)
            grads[1][at] = torch.matmul(ds.transpose(-1, -2), Q).transpose(1, 2)
    return (o, lse) + (tuple(grads) if grads else ())


def _exact_block(case, t, cu):
    B, L, d, H = case["B"], case["L"], case["d"], case["H"]
    w = {n: t[n].requires_grad_(True) for n in _WEIGHTS}
    x = t["x"].reshape(B * L, d).requires_grad_(True)
    norm = torch.nn.functional.layer_norm
    a = norm(x, (d,), w["ln1_w"], w["ln1_b"], LN_EPS)
    q, k, v = (z.reshape(B, L, H, d // H) for z in torch.matmul(a, w["w_qkv"]).split(d, 1))
    q, k = _rope64(q), _rope64(k)
    qkv = [z.detach() for z in (q, k, v)]
    o = _attend64(*qkv, None, cu)[0].reshape(B * L, d).requires_grad_(True)
    h = x + torch.matmul(o, w["w_o"])
    m = norm(h, (d,), w["ln2_w"], w["ln2_b"], LN_EPS)
    y = h + torch.matmul(torch.nn.functional.silu(torch.matmul(m, w["w_1"]))
                         * torch.matmul(m, w["w_3"]), w["w_2"])
    tail = [w[n] for n in ("w_o", "ln2_w", "ln2_b", "w_1", "w_3", "w_2")]
    g = torch.autograd.grad(y, [o, x] + tail, t["dy"].reshape(B * L, d))
    out = {"y": y.detach().reshape(B, L, d)}
    del y, h, m
    dqkv = _attend64(*qkv, g[0].reshape(B, L, H, d // H), cu)[2:]
    f = torch.autograd.grad([q, k, v], [x] + [w[n] for n in ("ln1_w", "ln1_b", "w_qkv")], dqkv)
    out["dx"] = (g[1] + f[0]).reshape(B, L, d)
    by_name = dict(zip(("ln1_w", "ln1_b", "w_qkv", "w_o", "ln2_w", "ln2_b", "w_1", "w_3", "w_2"),
                       f[1:] + g[2:]))
    out.update({"d" + n: by_name[n] for n in _WEIGHTS})
    return out


def exact(case, seed):
    t = {n: x.double() for n, x in _inputs(case, seed).items()}
    if case["kind"] == "linear":
        x, w, dy = t["x"], t["w"], t["dy"]
        return {"y": x @ w, "dx": dy @ w.t(), "dw": x.t() @ dy}
    cu = _doc_offsets(case, seed)
    if case["kind"] == "block":
        return _exact_block(case, t, cu)
    q, k = (_rope64(t[n]) if case["rope"] else t[n] for n in "qk")
    got = _attend64(q, k, t["v"], t.get("do"), cu)
    if case["mode"] == "eval":
        return {"o": got[0], "lse": got[1]}
    o, lse, dq, dk, dv = got
    if case["rope"]:
        dq, dk = _rope64(dq, inverse=True), _rope64(dk, inverse=True)
    if case["mode"] == "grad":
        return {"o": o, "dq": dq, "dk": dk, "dv": dv}
    return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}

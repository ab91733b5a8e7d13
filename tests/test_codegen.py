"""Code-generation checks of the attention kernels (CPU: hipcc cross-compiles
for gfx950; nothing runs on a GPU).

* The kernels whose tile loads go through inline assembly (forward, dQ, the
  D = 64 dK/dV kernel, the one-block D = 128 dK/dV kernel, the joint backward
  of small grids and the GEMM), in every form, must not wait
  for outstanding vector memory operations (`s_waitcnt vmcnt`) right before a
  transposed LDS read:
  that wait is the one the builtin load made the compiler insert, for the
  next tile's prefetch in the middle of the current tile.
* Register budgets the launch shapes rely on: no spills in any attention or
  GEMM kernel, and the one-block D = 64 forward and dQ kernels within 128 VGPRs
  (four waves per SIMD), whatever the number of wave groups.
* The order of the GEMM's first refill and the shape of its one-step path.
"""
import functools
import os
import re
import shutil
import subprocess
import tempfile

import pytest

from paper_2405_13226_amd import build as B

HIPCC = B.HIPCC

pytestmark = pytest.mark.skipif(not (os.path.exists(HIPCC) or shutil.which("hipcc")),
                                reason="hipcc not available")


@functools.lru_cache(maxsize=None)
def device_asm(src):
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, src + ".s")
        cmd = [HIPCC, *B.HIP_FLAGS, *B.HIP_SOURCE_FLAGS.get(src, []), "--cuda-device-only", "-S",
               "-o", out, os.path.join(B.CSRC, src)]
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        with open(out) as f:
            return f.read()


def symbols(asm, mangled_prefix):
    """The kernels whose symbol starts with the prefix."""
    found = sorted(set(re.findall(r"^(" + re.escape(mangled_prefix) + r"\w*):", asm, re.M)))
    assert found, mangled_prefix
    return found


def kernel_body(asm, symbol):
    """Instruction lines of a kernel."""
    m = re.search(r"^(" + re.escape(symbol) + r"):", asm, re.M)
    assert m, symbol
    start = m.end()
    end = asm.index(".end_amdhsa_kernel", start)
    lines = []
    for ln in asm[start:end].splitlines():
        t = ln.strip()
        if not t or t.startswith(";") or t.startswith(".") or t.endswith(":"):
            continue
        lines.append(t)
    return lines


def kernel_resources(asm):
    """{symbol: (vgpr_count, vgpr_spill_count)} from the metadata."""
    out = {}
    for m in re.finditer(r"\.name:\s+(_Z\S+)\s*\n(?:.*\n)*?\s+\.vgpr_count:\s+(\d+)\s*\n"
                         r"\s+\.vgpr_spill_count:\s+(\d+)", asm):
        out[m.group(1)] = (int(m.group(2)), int(m.group(3)))
    return out


def waits_before_transposed_reads(lines):
    n = 0
    for prev, cur in zip(lines, lines[1:]):
        if cur.startswith("ds_read_b64_tr_b16") and prev.startswith("s_waitcnt") and "vmcnt" in prev:
            n += 1
    return n


# (source, symbol prefix, instantiations)
@pytest.mark.parametrize("src, prefix, count", [
    ("dd_bwd.hip", "_ZN2dd12dkdv1_kernelILi64ELb0E", 2),   # one and two wave groups
    ("dd_bwd.hip", "_ZN2dd12dkdv1_kernelILi64ELb1E", 1),
    ("dd_bwd.hip", "_ZN2dd9dq_kernelILi64ELb0E", 3),       # one, two and four
    ("dd_bwd.hip", "_ZN2dd9dq_kernelILi64ELb1E", 1),
    ("dd_bwd.hip", "_ZN2dd9dq_kernelILi128ELb0E", 2),
    ("dd_bwd.hip", "_ZN2dd15bwd_pair_kernelI", 2),
    ("dd_dkdv.hip", "_ZN2dd11dkdv_kernelILi128ELb0E", 1),
    ("dd_fwd.hip", "_ZN2dd10fwd_kernelILi64ELb0ELb0E", 3),
    ("dd_fwd.hip", "_ZN2dd10fwd_kernelILi64ELb0ELb1E", 3),
    ("dd_fwd.hip", "_ZN2dd10fwd_kernelILi64ELb1ELb0E", 1),
    ("dd_fwd.hip", "_ZN2dd10fwd_kernelILi128ELb0ELb0E", 2),
    ("dd_fwd.hip", "_ZN2dd10fwd_kernelILi128ELb0ELb1E", 2),
    ("dd_fwd.hip", "_ZN2dd10fwd_kernelILi128ELb1ELb0E", 1),
    # the forms with a transposed operand: all but A B^T
    ("dd_gemm.hip", "_ZN2dd11gemm_kernelILb0ELb0E", 6),
    ("dd_gemm.hip", "_ZN2dd11gemm_kernelILb1ELb0E", 4),
    ("dd_gemm.hip", "_ZN2dd15gemm_mid_kernelINS_8TallTileELb0ELb0E", 6),
    ("dd_gemm.hip", "_ZN2dd15gemm_mid_kernelINS_8TallTileELb1ELb0E", 4),
    ("dd_gemm.hip", "_ZN2dd15gemm_mid_kernelINS_9SmallTileELb0ELb0E", 6),
    ("dd_gemm.hip", "_ZN2dd15gemm_mid_kernelINS_9SmallTileELb1ELb0E", 4),
])
def test_no_dma_wait_before_transposed_reads(src, prefix, count):
    asm = device_asm(src)
    found = symbols(asm, prefix)
    assert len(found) == count, found
    for sym in found:
        lines = kernel_body(asm, sym)
        assert any(ln.startswith("ds_read_b64_tr_b16") for ln in lines), sym
        assert waits_before_transposed_reads(lines) == 0, sym


@pytest.mark.parametrize("src", ["dd_fwd.hip", "dd_bwd.hip", "dd_dkdv.hip", "dd_bwd_short.hip",
                                 "dd_gemm.hip"])
def test_kernels_do_not_spill(src):
    asm = device_asm(src)
    res = kernel_resources(asm)
    assert res, src
    spills = {k: v for k, v in res.items() if v[1] != 0}
    assert not spills, spills
    four_waves = {"dd_fwd.hip": "_ZN2dd10fwd_kernelILi64ELb0E",
                  "dd_bwd.hip": "_ZN2dd9dq_kernelILi64ELb0E"}
    if src in four_waves:
        for sym in symbols(asm, four_waves[src]):
            assert res[sym][0] <= 128, (sym, res[sym])


def test_large_gemm_first_refill_waits_for_the_reads():
    # The 256 x 256 GEMM kernels read A's first half before their loop, whose
    # first loads refill that half: from the first LDS read on, every wave has
    # to wait for its reads and meet the workgroup's barrier before any direct
    # global->LDS load.
    asm = device_asm("dd_gemm.hip")
    syms = symbols(asm, "_ZN2dd11gemm_kernelI")
    assert len(syms) == 16  # eight operand forms and epilogues, narrow and wide
    for sym in syms:
        lines = kernel_body(asm, sym)
        first = next(i for i, ln in enumerate(lines) if ln.startswith("ds_read"))
        load = next(i for i in range(first, len(lines)) if lines[i].startswith("global_load_lds"))
        ordered = any(a.startswith("s_waitcnt") and "lgkmcnt(0)" in a and b.startswith("s_barrier")
                      for a, b in zip(lines[first:load], lines[first + 1:load]))
        assert ordered, sym


def test_large_gemm_takes_a_single_step_without_phases():
    # K = 64 is one step: its 64 products run without a barrier in between
    # (a phase of the pipelined loop is 16).
    asm = device_asm("dd_gemm.hip")
    for sym in symbols(asm, "_ZN2dd11gemm_kernelI"):
        longest = run = 0
        for ln in kernel_body(asm, sym):
            run = 0 if ln.startswith("s_barrier") else run + ln.startswith("v_mfma")
            longest = max(longest, run)
        assert longest >= 64, (sym, longest)

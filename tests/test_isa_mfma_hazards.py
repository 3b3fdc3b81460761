"""Kernels that issue matrix products from inline asm keep the wait states that
the compiler does not insert for them.  The scan follows the control flow of the
device assembly of each such kernel (fall through, branch targets, loops; the
fewest wait states over all paths into a block) and counts wait states, one per
instruction, N + 1 for s_nop N:
  * an operand of a product (A, B, or the accumulator it reads) must not have
    been written by a vector instruction within the 2 wait states before it;
  * an accumulator in the AGPRs must not be touched by anything but another
    product within the 18 wait states after a product wrote it (16 passes of a
    32x32 product, 2 more)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2609_23153_amd import build as B
from test_isa_dot2c import _operands, _regs

KERNELS = [("fwd_bf16_wave.hip", "_ZN2sa12_GLOBAL__N_120fwd_bf16_wave_kernelENS0_6ParamsE")]
OPERAND, ACCUMULATOR = 2, 18   # wait states


def blocks(lines):
    """Basic blocks of a listing: [(instructions, successors' numbers)]."""
    out, labels = [[]], {}
    for l in lines:
        l = l.split(";")[0].strip()
        m = re.match(r"([.\w$]+):", l)
        if m:
            if out[-1]:
                out.append([])
            labels[m.group(1)] = len(out) - 1
        elif l and not l.startswith("."):
            out[-1].append(re.sub(r"\s+", " ", l))
            if l.startswith(("s_branch", "s_cbranch", "s_endpgm")):
                out.append([])
    res = []
    for n, ins in enumerate(out):
        last = ins[-1].split() if ins else [""]
        succ = []
        if last[0].startswith(("s_branch", "s_cbranch")):
            succ.append(labels[last[1]])
        if last[0] not in ("s_branch", "s_endpgm") and n + 1 < len(out):
            succ.append(n + 1)
        res.append((ins, succ))
    return res


def run_block(ins, entry, bad=None):
    """State after a block: wait states since a vector instruction wrote a
    register, and since a product wrote it, each {register: wait states}."""
    valu = {r: -a for r, a in entry[0].items()}   # -> time of the write
    product = {r: -a for r, a in entry[1].items()}
    now = 0
    for l in ins:
        op = l.split()[0]
        if op == "s_nop":
            now += int(l.split()[1]) + 1
            continue
        now += 1
        regs = [_regs(t) for t in _operands(l)] if len(l.split()) > 1 else []
        if op.startswith("v_mfma"):
            if bad is not None:
                for r in set().union(*regs[1:4]):
                    if now - valu.get(r, -99) <= OPERAND:
                        bad.append(("operand", r, l))
            for r in regs[0]:
                if r[0] == "a":
                    product[r] = now
        else:
            if bad is not None:
                for r in set().union(*regs) if regs else ():
                    if r[0] == "a" and now - product.get(r, -99) <= ACCUMULATOR:
                        bad.append(("accumulator", r, l))
            if op.startswith("v_") and regs:
                written = regs[0] | regs[1] if "swap" in op else regs[0]
                for r in written:
                    valu[r] = now
    return ({r: now - t for r, t in valu.items() if now - t < OPERAND},
            {r: now - t for r, t in product.items() if now - t < ACCUMULATOR})


def hazards(lines):
    bl = blocks(lines)
    entry = [({}, {}) for _ in bl]
    todo = list(range(len(bl)))
    while todo:
        n = todo.pop()
        after = run_block(bl[n][0], entry[n])
        for s in bl[n][1]:
            grown = False
            for have, new in zip(entry[s], after):
                for r, a in new.items():
                    if a < have.get(r, 99):
                        have[r] = a
                        grown = True
            if grown:
                todo.append(s)
    bad = []
    for (ins, _), e in zip(bl, entry):
        run_block(ins, e, bad)
    return bad


def kernel_lines(asm, sym):
    lines = asm.split("\n")
    start = next(i for i, l in enumerate(lines) if l.startswith(sym + ":"))
    end = next(i for i in range(start, len(lines)) if lines[i].startswith(".Lfunc_end"))
    return lines[start + 1:end]


M = "v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]"


@pytest.mark.parametrize("kind,listing", [
    (None, ["v_mov_b32_e32 v5, v1", "s_nop 1", M, "s_nop 15", "s_nop 2",
            "v_accvgpr_read_b32 v9, a3"]),
    ("operand", ["v_mov_b32_e32 v5, v1", "s_nop 0", M]),
    ("operand", ["v_accvgpr_write_b32 a3, v1", M]),                  # the accumulator read as C
    ("operand", ["v_permlane32_swap_b32_e32 v20, v9", "s_nop 0", M]),
    ("accumulator", [M, "s_nop 15", "v_accvgpr_read_b32 v9, a3"]),
    # across a back edge: the end of the loop writes an operand of its start
    ("operand", [".L1:", M, "s_nop 7", "v_mov_b32_e32 v8, v1", "s_cbranch_scc1 .L1", "s_endpgm"]),
    (None, [".L1:", M, "s_nop 7", "v_mov_b32_e32 v8, v1", "s_nop 0", "s_cbranch_scc1 .L1",
            "s_endpgm"]),
    # in a block placed behind the end of the kernel
    ("accumulator", [M, "s_cbranch_vccnz .L2", ".L1:", "s_endpgm", ".L2:",
                     "v_accvgpr_read_b32 v9, a3", "s_branch .L1"]),
    (None, [M, "s_cbranch_vccnz .L2", ".L1:", "s_endpgm", ".L2:", "s_nop 15", "s_nop 1",
            "v_accvgpr_read_b32 v9, a3", "s_branch .L1"]),
    # by the shorter of two paths into a block
    ("accumulator", [M, "s_cbranch_scc1 .L1", "s_nop 15", "s_nop 7", ".L1:",
                     "v_accvgpr_read_b32 v9, a3", "s_endpgm"]),
])
def test_scanner_sees_hazards_on_every_path(kind, listing):
    found = hazards(listing)
    assert [b[0] for b in found] == ([kind] if kind else []), found


@pytest.mark.skipif(not os.path.exists(B.HIPCC) and shutil.which("hipcc") is None,
                    reason="hipcc not available")
@pytest.mark.parametrize("src,kernel", KERNELS)
def test_products_from_inline_asm_keep_their_wait_states(tmp_path, src, kernel):
    out = tmp_path / "k.s"
    cmd = [B.HIPCC, *B.FLAGS, *B.EXTRA.get(src, []), "--cuda-device-only", "-S",
           os.path.join(B.CSRC, src), "-o", str(out)]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    lines = kernel_lines(out.read_text(), kernel)
    assert sum(bool(re.match(r"\s*v_mfma\S* a\[", l)) for l in lines) >= 16
    assert not hazards(lines)

"""Kernels that issue matrix products from inline asm keep the wait states that
the compiler does not insert for them.  The scan walks the device assembly of
each such kernel in program order and counts wait states (one per instruction,
N + 1 for s_nop N):
  * a product's operands must not have been written by a vector instruction
    within the 2 wait states before it;
  * an accumulator in the AGPRs must not be touched by anything but another
    product within the 18 wait states after a product wrote it (16 passes of a
    32x32 product, 2 more)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2609_23153_amd import build as B
from test_isa_dot2c import _operands, _regs, kernel_instructions

KERNELS = [("fwd_bf16_wave.hip", "_ZN2sa12_GLOBAL__N_120fwd_bf16_wave_kernelENS0_6ParamsE")]


def hazards(instrs):
    bad, now = [], 0
    valu, product = {}, {}   # register -> wait state of its last such write
    for l in instrs:
        op = l.split()[0]
        if op == "s_nop":
            now += int(l.split()[1]) + 1
            continue
        now += 1
        regs = [_regs(t) for t in _operands(l)] if len(l.split()) > 1 else []
        if op.startswith("v_mfma"):
            for r in set().union(*regs[1:3]):
                if now - valu.get(r, -99) <= 2:
                    bad.append(("operand", r, l))
            for r in regs[0]:
                if r[0] == "a":
                    product[r] = now
        else:
            for r in set().union(*regs) if regs else ():
                if r[0] == "a" and now - product.get(r, -99) <= 18:
                    bad.append(("accumulator", r, l))
            if op.startswith("v_") and regs:
                for r in regs[0]:
                    valu[r] = now
    return bad


def test_scanner_sees_both_hazards():
    m = "v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]"
    assert not hazards(["v_mov_b32_e32 v5, v1", "s_nop 1", m, "s_nop 15", "s_nop 2",
                        "v_accvgpr_read_b32 v9, a3"])
    assert hazards(["v_mov_b32_e32 v5, v1", "s_nop 0", m])[0][0] == "operand"
    assert hazards([m, "s_nop 15", "v_accvgpr_read_b32 v9, a3"])[0][0] == "accumulator"


@pytest.mark.skipif(not os.path.exists(B.HIPCC) and shutil.which("hipcc") is None,
                    reason="hipcc not available")
@pytest.mark.parametrize("src,kernel", KERNELS)
def test_products_from_inline_asm_keep_their_wait_states(tmp_path, src, kernel):
    out = tmp_path / "k.s"
    cmd = [B.HIPCC, *B.FLAGS, *B.EXTRA.get(src, []), "--cuda-device-only", "-S",
           os.path.join(B.CSRC, src), "-o", str(out)]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    instrs = [re.sub(r"\s+", " ", l) for l in kernel_instructions(out.read_text(), kernel)]
    assert sum(l.startswith("v_mfma") and " a[" in l for l in instrs) >= 16
    assert not hazards(instrs)

"""The dK/dV kernel's first products are matrix instructions in inline assembly, whose waits the compiler does not insert.
The generated code of this build is read instruction by instruction for what the source can only ask for."""
import os
import re
import subprocess

import pytest

from paper_2408_10188_amd import build

PASSES = 8                     # issue slots (of four cycles) of a 32x32x16 bf16 product
BEFORE, AFTER = 2, 19          # wait states: vector write -> operand, result -> vector instruction


def registers(text):
    """VGPRs named by an operand list, as a set of numbers."""
    out = set()
    for lo, hi in re.findall(r"(?<![\w.])v\[(\d+):(\d+)\]", text):
        out.update(range(int(lo), int(hi) + 1))
    out.update(int(n) for n in re.findall(r"(?<![\w.\[])v(\d+)", text))
    return out


def violations(lines):
    """(line, what) for every matrix instruction with a VGPR result that breaks one of the two distances."""
    code = []
    for n, line in enumerate(lines):
        m = re.match(r"\s+([a-z]\w+)\s*(.*?)(?:\s*;.*)?$", line)
        if m and not m[1].startswith("."):
            code.append((n, m[1], m[2]))

    def states(op, args):
        return int(args, 0) + 1 if op == "s_nop" else PASSES if op.startswith("v_mfma") else 1

    bad = []
    for i, (n, op, args) in enumerate(code):
        if not (op.startswith("v_mfma") and args.startswith("v")):
            continue
        result, rest = args.split(",", 1)
        result, operands = registers(result), registers(rest)
        waited = 0
        for _, o, a in reversed(code[:i]):
            if waited >= BEFORE:
                break
            if o.startswith("v_") and not o.startswith(("v_mfma", "v_cmp", "v_accvgpr_write")) and registers(a.split(",", 1)[0]) & operands:
                bad.append((n, "operand written by " + o + " " + a))
            waited += states(o, a)
        waited = 0
        for _, o, a in code[i + 1:]:
            if waited >= AFTER:
                break
            if o.startswith("v_mfma") and a.startswith("v") and registers(a.split(",", 1)[0]) == result:
                break                                    # the chain goes on: accumulating onto the result needs no wait
            if o.startswith(("v_", "ds_", "global_", "buffer_", "flat_")) and registers(a) & result:
                bad.append((n, "result touched by " + o + " " + a))
            waited += states(o, a)
    return bad


def test_reader_finds_both_kinds():
    product = "\tv_mfma_f32_32x32x16_bf16 v[0:15], v[36:39], a[0:3], v[0:15]"
    assert violations(["\tv_mov_b32_e32 v7, v50", "\ts_mov_b32 s1, s2", product])
    assert not violations(["\tv_mov_b32_e32 v7, v50", "\ts_nop 1", product])
    assert violations([product, "\ts_nop 15", "\tv_mul_f32_e32 v60, v3, v61"])
    assert not violations([product, "\ts_nop 15", "\ts_nop 7", "\tv_mul_f32_e32 v60, v3, v61"])


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no HIP compiler")
def test_first_products_of_dkdv(tmp_path):
    out = str(tmp_path / "dkdv.s")
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    subprocess.run([build.HIPCC, *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, "bwd_dkdv_bf16.hip"), "-o", out], check=True,
                   capture_output=True)
    with open(out) as f:
        lines = f.read().splitlines()
    assert sum("v_mfma_f32_32x32x16_bf16 v" in ln for ln in lines) >= 400
    assert violations(lines) == []

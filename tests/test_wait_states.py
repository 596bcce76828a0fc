"""The backward kernels issue their gradient products as assembly statements, which the compiler's insertion of wait
states does not look into.  This reads the listing of what the compiler made around them (no GPU): a vector instruction
that writes a source of a matrix product is followed by two wait states before it, and nothing but a product that goes on
with the same accumulator touches a product's result within twelve (eight passes)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2605_10905_amd import build as b


def _regs(operand):
    m = re.match(r"^-?\|?([va])(\d+)\|?$", operand.strip())
    if m:
        return {(m.group(1), int(m.group(2)))}
    m = re.match(r"^([va])\[(\d+):(\d+)\]$", operand.strip())
    return {(m.group(1), i) for i in range(int(m.group(2)), int(m.group(3)) + 1)} if m else set()


def _instructions(text):
    out = []
    for n, line in enumerate(text.splitlines(), 1):
        m = re.match(r"^\s+([a-z]\w+)\s*(.*)$", line.split(";")[0].rstrip())
        if m:
            ops = [x for x in m.group(2).split(",") if x]
            out.append((n, m.group(1), [_regs(x.split()[0]) if x.split() else set() for x in ops], m.group(2)))
    return out


def _states(op, rest):
    return int(rest, 0) + 1 if op == "s_nop" else 1


def findings(text):
    ins, bad = _instructions(text), []
    for i, (n, op, ops, _) in enumerate(ins):
        if not op.startswith("v_mfma"):
            continue
        result, sources, states = ops[0], set().union(*ops[1:4]), 0
        for m, o, p, rest in reversed(ins[max(0, i - 3):i]):
            if o.startswith("v_") and not o.startswith(("v_mfma", "v_cmp")) and p and p[0] & sources:
                bad.append((m, n))
            states += _states(o, rest)
            if states >= 2:
                break
        states = 0
        for m, o, p, rest in ins[i + 1:i + 16]:
            if o in ("s_branch", "s_endpgm"):
                break
            if o.startswith("v_mfma"):
                if set().union(*p[1:3]) & result or (p[0] & result and p[0] != result):
                    bad.append((n, m))
            elif o.startswith(("v_", "ds_", "global_")) and p and set().union(*p) & result:
                bad.append((n, m))
            states += _states(o, rest)
            if states >= 12:
                break
    return bad


def test_the_check_sees_what_it_looks_for():
    mfma = "\tv_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[4:7], a[0:15]\n"
    assert not findings("\tv_mov_b32_e32 v4, 0\n\ts_nop 1\n" + mfma + "\ts_nop 11\n\tv_accvgpr_read_b32 v8, a3\n")
    assert findings("\tv_mov_b32_e32 v4, 0\n\ts_nop 0\n" + mfma)
    assert findings(mfma + "\ts_nop 7\n\tv_accvgpr_read_b32 v8, a3\n")
    assert findings(mfma + "\tv_mfma_f32_32x32x16_bf16 a[8:23], v[0:3], v[4:7], a[8:23]\n")
    assert not findings(mfma + mfma)


@pytest.mark.skipif(shutil.which(b.HIPCC) is None, reason="needs hipcc")
def test_gradient_products_keep_their_wait_states(tmp_path):
    src, out = "attn_bwd_bf16.hip", str(tmp_path / "bwd.s")
    subprocess.run([b.HIPCC, *b.FLAGS, *b.SOURCE_FLAGS[src], "--cuda-device-only", "-S", os.path.join(b.CSRC, src), "-o", out], check=True, capture_output=True)
    text = open(out).read()
    assert text.count("v_mfma_f32_32x32x16_bf16") > 1000
    assert not findings(text)

"""The backward kernels issue their gradient products as assembly statements, which the compiler's insertion of wait
states does not look into.  This reads the listing of what the compiler made around them (no GPU): a vector instruction
that writes a source of a matrix product is followed by two wait states before it, and nothing but a product that goes on
with the same accumulator touches a product's result within twelve (eight passes).  Branches are followed to both sides,
back edges among them."""
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
    """[(line, opcode, registers of every operand, operands)], and for each the instructions that may come after it."""
    out, labels, follows = [], {}, []
    for n, line in enumerate(text.splitlines(), 1):
        line = line.split(";")[0].rstrip()
        m = re.match(r"^([.\w$]+):$", line)
        if m:
            labels[m.group(1)] = len(out)
        m = re.match(r"^\s+([a-z]\w+)\s*(.*)$", line)
        if m:
            ops = [x for x in m.group(2).split(",") if x]
            out.append((n, m.group(1), [_regs(x.split()[0]) if x.split() else set() for x in ops], m.group(2).strip()))
    for i, (_, op, _, rest) in enumerate(out):
        nxt = [i + 1] if op not in ("s_branch", "s_endpgm", "s_setpc_b64") and i + 1 < len(out) else []
        follows.append(nxt + ([labels[rest]] if op.startswith(("s_branch", "s_cbranch")) else []))
    return out, follows


def _states(op, rest):
    return int(rest, 0) + 1 if op == "s_nop" else 1


def _within(ins, edges, start, limit):
    """The instructions that some path along `edges` reaches from `start` (not itself) before `limit` wait states."""
    least, todo = {}, [(i, 0) for i in edges[start]]
    while todo:
        i, states = todo.pop()
        if states >= limit or least.get(i, limit) <= states:
            continue
        least[i] = states
        todo += [(j, states + _states(ins[i][1], ins[i][3])) for j in edges[i]]
    return least


def findings(text):
    (ins, follows), bad = _instructions(text), []
    comes_from = [[] for _ in ins]
    for i, to in enumerate(follows):
        for j in to:
            comes_from[j].append(i)
    for i, (n, op, ops, _) in enumerate(ins):
        if not op.startswith("v_mfma"):
            continue
        result, sources = ops[0], set().union(*ops[1:4])
        for j in _within(ins, comes_from, i, 2):
            m, o, p, _ = ins[j]
            written = set().union(*p[:2 if "swap" in o else 1]) if p else set()
            if o.startswith("v_") and not o.startswith(("v_mfma", "v_cmp")) and written & sources:
                bad.append((m, n))
        for j in _within(ins, follows, i, 12):
            m, o, p, _ = ins[j]
            if o.startswith("v_mfma"):
                if set().union(*p[1:3]) & result or (p[0] & result and p[0] != result):
                    bad.append((n, m))
            elif o.startswith(("v_", "ds_", "global_", "buffer_", "scratch_", "flat_")) and p and set().union(*p) & result:
                bad.append((n, m))
    return bad


def test_the_check_sees_what_it_looks_for():
    mfma = "\tv_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[4:7], a[0:15]\n"
    assert not findings("\tv_mov_b32_e32 v4, 0\n\ts_nop 1\n" + mfma + "\ts_nop 11\n\tv_accvgpr_read_b32 v8, a3\n")
    assert findings("\tv_mov_b32_e32 v4, 0\n\ts_nop 0\n" + mfma)
    assert findings(mfma + "\ts_nop 7\n\tv_accvgpr_read_b32 v8, a3\n")
    assert findings(mfma + "\tv_mfma_f32_32x32x16_bf16 a[8:23], v[0:3], v[4:7], a[8:23]\n")
    assert not findings(mfma + mfma)
    assert findings("\tv_swap_b32 v20, v4\n" + mfma) and findings(mfma + "\tscratch_store_dword off, a3, s32\n")
    # over a loop's back edge, and to a branch's target
    loop = "\ts_nop 1\n.LBB0_1:\n" + mfma + "\ts_nop 11\n%s\ts_cbranch_scc1 .LBB0_1\n\ts_endpgm\n"
    assert not findings(loop % "") and findings(loop % "\tv_mov_b32_e32 v4, 0\n")
    away = mfma + "\ts_cbranch_scc1 .LBB0_2\n\ts_nop 11\n%s\ts_endpgm\n.LBB0_2:\n%s\ts_endpgm\n"
    read = "\tv_accvgpr_read_b32 v8, a3\n"
    assert not findings(away % (read, "\ts_nop 11\n" + read)) and findings(away % (read, read))
    assert findings(mfma + "\ts_branch .LBB0_2\n\ts_nop 11\n.LBB0_2:\n" + read)


@pytest.mark.skipif(shutil.which(b.HIPCC) is None, reason="needs hipcc")
def test_gradient_products_keep_their_wait_states(tmp_path):
    src, out = "attn_bwd_bf16.hip", str(tmp_path / "bwd.s")
    subprocess.run([b.HIPCC, *b.FLAGS, *b.SOURCE_FLAGS[src], "--cuda-device-only", "-S", os.path.join(b.CSRC, src), "-o", out], check=True, capture_output=True)
    text = open(out).read()
    assert text.count("v_mfma_f32_32x32x16_bf16") > 1000
    assert not findings(text)

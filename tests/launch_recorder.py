"""Which kernels a call of the library launches, found without a GPU: the library is loaded, in a
process of its own, behind a runtime that only writes launches down (launch_recorder.cpp).

A call is a dict: op ("fwd", "fwd_variant", "fp8", "fp8_variant", "persistent", "bwd", "bwd_noalloc", "nt", "nt_variant",
"nn", "splitk"), the sizes that entry point takes, and `variant` or `splits` where it has one."""
import ctypes
import json
import os
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def routes(calls):
    """([(status, [(kernel, workgroups, threads), ...]) for every call], names of all kernels)."""
    with tempfile.TemporaryDirectory() as td:
        lib = os.path.join(td, "recorder.so")
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", os.path.join(ROOT, "tests", "launch_recorder.cpp"), "-o", lib], check=True)
        r = subprocess.run([sys.executable, os.path.abspath(__file__), lib], input=json.dumps(calls), capture_output=True, text=True,
                           cwd=ROOT, timeout=120)
        assert r.returncode == 0, r.stderr[-2000:]
        got = json.loads(r.stdout)
    return [(st, [(short(n), g, t) for n, g, t in launches]) for st, launches in got["calls"]], {short(n) for n in got["kernels"]}


def short(name):
    """attn_fwd_sp_kernel<128, true, 0, false, 2> of a demangled name."""
    name = name.replace("(anonymous namespace)::", "")
    name = name[5:] if name.startswith("void ") else name
    return name[:name.index("(")] if "(" in name else name


def _call(A, c):
    p, q = 1 << 20, dict(stream=0, check=False)  # (aligned addresses that nothing reads)
    op = c["op"]
    if op in ("nt", "nn", "nt_variant", "splitk"):
        mnk = (c["M"], c["N"], c["K"])
        if op == "nt":
            return A.gemm_bf16_nt(p, p, p, *mnk, **q)
        if op == "nn":
            return A.gemm_bf16_nn(p, p, p, *mnk, **q)
        if op == "nt_variant":
            return A.gemm_bf16_nt_variant(p, p, p, *mnk, c["variant"], **q)
        return A.gemm_bf16_nt_splitk(p, p, p, *mnk, c["splits"], p, **q)
    size = (c.get("B", 1), c["H"], c.get("Hkv", c["H"]), c["N"], c.get("d", 128), c.get("causal", False), 0.1)
    if op == "bwd":
        return A.attn_bwd(*[p] * 10, *size, A.ATTN_BF16, **q)
    if op == "bwd_noalloc":
        return A.attn_bwd_noalloc(*[p] * 9, *size, A.ATTN_BF16, **q)
    if op == "persistent":
        return A.attn_fwd_persistent(*[p] * 5, *size, A.ATTN_BF16, p, **q)
    if op == "fp8":
        return A.attn_fwd_fp8(*[p] * 5, *size, 1.0, 1.0, 1.0, **q)
    if op == "fp8_variant":
        return A.attn_fwd_fp8_variant(*[p] * 5, *size, 1.0, 1.0, 1.0, c["variant"], **q)
    if op == "fwd_variant":
        return A.attn_fwd_variant(*[p] * 5, *size, A.ATTN_BF16, c["variant"], **q)
    assert op == "fwd", op
    return A.attn_fwd(*[p] * 5, *size, A.ATTN_BF16, **q)


def _main(recorder):
    rec = ctypes.CDLL(recorder, mode=ctypes.RTLD_GLOBAL)
    rec.recorder_take.restype = rec.recorder_kernels.restype = ctypes.c_char_p
    sys.path.insert(0, ROOT)
    import paper_2605_10905_amd.binding as A

    def lines(text):
        return [(n, int(g), int(t)) for n, g, t in (x.split("\t") for x in text.decode().splitlines())]

    calls = []
    for c in json.load(sys.stdin):
        st = _call(A, c)
        calls.append((st, lines(rec.recorder_take())))
    json.dump(dict(calls=calls, kernels=[n for n, _, _ in lines(rec.recorder_kernels())]), sys.stdout)


if __name__ == "__main__":
    _main(sys.argv[1])

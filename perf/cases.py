"""Performance cases of the attention and GEMM library: what its users have it do.

listed() holds fixed cases, draw(rng) gives one more of the same ranges, prepare / run make the
inputs of a case and take ONE pass through the public entry points.  A case is a dict of plain values:

  op      "fwd" (attn_fwd / attn_fwd_fp8), "persistent" (attn_fwd_persistent), "bwd" (attn_bwd),
          "nt" (gemm_bf16_nt), "nn" (gemm_bf16_nn), "splitk" (gemm_bf16_nt_splitk with the number
          of slices that gemm_splitk_plan recommends)
  attention: B, Hq, Hkv, N, d, causal, dtype ("bf16" / "fp8"), sigma of the normal inputs
  GEMM:      M, N, K
"""
import math

import torch

import paper_2605_10905_amd as A


def _attn(name, op, B, Hq, Hkv, N, d, causal, dtype="bf16", sigma=1.0):
    c = dict(op=op, B=B, Hq=Hq, Hkv=Hkv, N=N, d=d, causal=causal, dtype=dtype, sigma=sigma)
    return dict(name=name, **c) if name else c


def _gemm(name, op, M, N, K):
    c = dict(op=op, M=M, N=N, K=K)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest call: two heads of 256 tokens; what a unit test or a tiny layer launches, all latency
        _attn("fwd_tiny", "fwd", 1, 2, 2, 256, 64, False),
        # prefill of one request of odd length in a grouped-query layer: fewer query tiles than CUs
        _attn("fwd_prefill_1000", "fwd", 1, 32, 8, 1000, 128, True),
        # an ordinary causal training batch of 2k tokens
        _attn("fwd_causal_2k", "fwd", 4, 16, 16, 2048, 128, True),
        # long bidirectional attention, the shape the library's headline figure is quoted on
        _attn("fwd_long_8k", "fwd", 2, 32, 32, 8192, 128, False, sigma=0.5),
        # quantised long-context prefill: e4m3 inputs with one scale per tensor
        _attn("fwd_fp8_16k", "fwd", 4, 16, 16, 16384, 128, True, dtype="fp8"),
        # backward of a small batch of odd length at head dimension 64
        _attn("bwd_1000_d64", "bwd", 2, 16, 16, 1000, 64, False),
        # backward of a grouped-query training layer
        _attn("bwd_gqa_4k", "bwd", 4, 64, 8, 4096, 128, True),
        # a linear layer on a handful of rows: bound by reading the weight
        _gemm("nt_33_rows", "nt", 33, 4096, 4096),
        # a product of ordinary small size, ragged in both directions, second operand [K, N]
        _gemm("nn_odd_1k", "nn", 1111, 1000, 1056),
        # large square layer, bound by the matrix cores
        _gemm("nt_8192_k4096", "nt", 8192, 8192, 4096),
        # very many rows, short contraction: bound by memory traffic
        _gemm("nt_large_m", "nt", 442368, 448, 192),
        # few output tiles, very long contraction (a weight gradient): split over k
        _gemm("splitk_large_k", "splitk", 2304, 1024, 65536),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# largest drawn work: attention forward, backward (flop), GEMM (flop; bytes of operands and result);
# each well below the largest listed case
_CAP_FWD, _CAP_BWD, _CAP_GEMM, _CAP_GEMM_BYTES = 1.5e12, 1.2e12, 5.0e11, 1.0e9


def draw(rng):
    while True:
        op = rng.choice(("fwd", "fwd", "fwd", "fp8", "persistent", "bwd", "bwd", "nt", "nt", "nt", "nn", "splitk"))
        if op in ("fwd", "fp8", "persistent", "bwd"):
            hkv, group = rng.choice((1, 2, 3, 4, 6, 8, 12, 16, 32)), rng.choice((1, 1, 2, 4, 8))
            c = _attn(None, "fwd" if op == "fp8" else op, rng.randint(1, 8), hkv * group, hkv, _log_int(rng, 100, 16384),
                      128 if op == "fp8" else rng.choice((64, 128, 128)), rng.random() < 0.6, "fp8" if op == "fp8" else "bf16",
                      rng.choice((0.5, 1.0)))
            if work(c)["flops"] <= (_CAP_BWD if op == "bwd" else _CAP_FWD):
                return c
        else:
            if op == "splitk":
                c = _gemm(None, op, _log_int(rng, 64, 4096), _log_int(rng, 64, 4096), 64 * _log_int(rng, 64, 1024))
            else:
                c = _gemm(None, op, _log_int(rng, 1, 500000), _log_int(rng, 32, 65536), 32 * _log_int(rng, 2, 512))
                if op == "nn":
                    c["N"] = (c["N"] + 7) // 8 * 8
            if work(c)["flops"] <= _CAP_GEMM and work(c)["bytes"] <= _CAP_GEMM_BYTES:
                return c


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(shape, sigma=1.0, dtype=torch.bfloat16):
        x = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)
        return (x * sigma).to(dtype)

    def empty(shape, dtype=torch.bfloat16):
        return torch.empty(shape, device="cuda", dtype=dtype)

    st = dict(case)
    if case["op"] in ("nt", "nn", "splitk"):
        M, N, K = case["M"], case["N"], case["K"]
        st.update(a=normal((M, K)), b=normal((K, N) if case["op"] == "nn" else (N, K)), c=empty((M, N)))
        if case["op"] == "splitk":
            st["splits"] = A.gemm_splitk_plan(M, N, K)
            st["ws"] = empty((max(1, A.gemm_splitk_workspace_bytes(M, N, st["splits"]) // 4),), torch.float32)
        return st
    B, Hq, Hkv, N, d = (case[k] for k in ("B", "Hq", "Hkv", "N", "d"))
    qshape, kshape = (B, Hq, N, d), (B, Hkv, N, d)
    st.update(scale=1.0 / math.sqrt(d), o=empty(qshape), lse=empty((B, Hq, N), torch.float32))
    for nm, shape in (("q", qshape), ("k", kshape), ("v", kshape)):
        if case["dtype"] == "fp8":
            # per-tensor quantisation: codes of x / s with s = amax / 448
            x = normal(shape, case["sigma"], torch.float32)
            s = float(x.abs().max()) / 448.0
            st[nm] = (x / s).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
            st["s" + nm] = s
        else:
            st[nm] = normal(shape, case["sigma"])
    if case["op"] == "persistent":
        # the 8 counters of the tile queue; rounded up to whole 128-byte lines by the allocator
        st["queue"] = empty((A.attn_persistent_queue_bytes() // 4,), torch.int32)
    if case["op"] == "bwd":
        # the forward's outputs and the gradient of o are what a training step has at this point
        st.update(dout=normal(qshape), dq=empty(qshape), dk=empty(kshape), dv=empty(kshape),
                  ws=empty((A.attn_bwd_workspace_bytes(B, Hq, N) // 4,), torch.float32))
        A.attn_fwd(st["q"], st["k"], st["v"], st["o"], st["lse"], B, Hq, Hkv, N, d, case["causal"], st["scale"], A.ATTN_BF16)
    return st


def run(state):
    s = state
    if s["op"] in ("nt", "nn", "splitk"):
        if s["op"] == "nn":
            A.gemm_bf16_nn(s["a"], s["b"], s["c"], s["M"], s["N"], s["K"])
        elif s["op"] == "splitk" and s["splits"] > 1:
            A.gemm_bf16_nt_splitk(s["a"], s["b"], s["c"], s["M"], s["N"], s["K"], s["splits"], s["ws"])
        else:
            A.gemm_bf16_nt(s["a"], s["b"], s["c"], s["M"], s["N"], s["K"])
        return s["c"]
    sizes = (s["B"], s["Hq"], s["Hkv"], s["N"], s["d"], s["causal"], s["scale"])
    if s["op"] == "bwd":
        A.attn_bwd(s["q"], s["k"], s["v"], s["o"], s["dout"], s["lse"], s["dq"], s["dk"], s["dv"], s["ws"], *sizes, A.ATTN_BF16)
        return s["dq"], s["dk"], s["dv"]
    if s["dtype"] == "fp8":
        A.attn_fwd_fp8(s["q"], s["k"], s["v"], s["o"], s["lse"], *sizes, s["sq"], s["sk"], s["sv"])
    elif s["op"] == "persistent":
        A.attn_fwd_persistent(s["q"], s["k"], s["v"], s["o"], s["lse"], *sizes, A.ATTN_BF16, s["queue"])
    else:
        A.attn_fwd(s["q"], s["k"], s["v"], s["o"], s["lse"], *sizes, A.ATTN_BF16)
    return s["o"], s["lse"]


def work(case):
    if case["op"] in ("nt", "nn", "splitk"):
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": 2 * (M * K + N * K + M * N), "flops": 2 * M * N * K}
    B, Hq, Hkv, N, d = (case[k] for k in ("B", "Hq", "Hkv", "N", "d"))
    pairs = N * (N + 1) // 2 if case["causal"] else N * N  # visible (query, key) pairs of a head
    rows_q, rows_k = B * Hq * N, B * Hkv * N
    if case["op"] == "bwd":
        # read q, o, dout, k, v, lse; write dq, dk, dv; five products
        return {"bytes": 2 * d * (4 * rows_q + 4 * rows_k) + 4 * rows_q, "flops": 10 * B * Hq * pairs * d}
    size = 1 if case["dtype"] == "fp8" else 2
    return {"bytes": d * (size * (rows_q + 2 * rows_k) + 2 * rows_q) + 4 * rows_q, "flops": 4 * B * Hq * pairs * d}


def tolerance(case):
    # About four times what the outputs differ from the same operation in float64 (measured on the listed
    # cases and eight drawn ones): GEMM 1.7e-3 and at most 3.9e-3 of an element (the rounding to bf16);
    # attention forward 2.4e-3, largest 0.038 of the root mean square (bf16 P, then bf16 O; early causal
    # rows are larger than the mean); backward 2.6e-3, largest 0.078.
    if case["op"] in ("nt", "nn", "splitk"):
        return {"rel": 6.6e-3, "max": 1.6e-2}
    return {"rel": 1e-2, "max": 0.3 if case["op"] == "bwd" else 0.15}


def exact(case, seed):
    # what run() returns, in float64 by plain torch: the definition, one query head at a time
    s = prepare(case, seed)
    if case["op"] in ("nt", "nn", "splitk"):
        return s["a"].double() @ (s["b"].double() if case["op"] == "nn" else s["b"].double().t())
    B, Hq, Hkv, N, d = (case[k] for k in ("B", "Hq", "Hkv", "N", "d"))

    def real(nm, b, h):
        x = s[nm][b, h]
        return x.view(torch.float8_e4m3fn).float().double() * s["s" + nm] if case["dtype"] == "fp8" else x.double()

    def zeros(*shape):
        return torch.zeros(shape, device="cuda", dtype=torch.float64)

    hidden = torch.ones(N, N, device="cuda", dtype=torch.bool).triu_(1) if case["causal"] else None
    bwd = case["op"] == "bwd"
    if bwd:
        dq, dk, dv = zeros(B, Hq, N, d), zeros(B, Hkv, N, d), zeros(B, Hkv, N, d)
    else:
        o, lse = zeros(B, Hq, N, d), zeros(B, Hq, N)
    for b in range(B):
        for h in range(Hq):
            g = h // (Hq // Hkv)
            q, k, v = real("q", b, h), real("k", b, g), real("v", b, g)
            sc = (q @ k.t()).mul_(s["scale"])
            if hidden is not None:
                sc.masked_fill_(hidden, -math.inf)
            row = torch.logsumexp(sc, 1)
            p = sc.sub_(row[:, None]).exp_()
            if not bwd:
                o[b, h], lse[b, h] = p @ v, row
                continue
            g_out = s["dout"][b, h].double()
            dv[b, g] += p.t() @ g_out
            dp = g_out @ v.t()
            ds = dp.sub_((p * dp).sum(1, keepdim=True)).mul_(p).mul_(s["scale"])
            dq[b, h] = ds @ k
            dk[b, g] += ds.t() @ q
    return (dq, dk, dv) if bwd else (o, lse)

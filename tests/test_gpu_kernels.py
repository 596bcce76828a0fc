"""Every kernel of the library on the GPU against the oracle, each by a call that launches it
(kernel_cases.py; test_dispatch.py holds, without a GPU, that the calls still do).  Tolerances are those of
the other parity tests (gpu_util.py, test_gpu_gemm_parity.py)."""
import numpy as np
import pytest
import torch

import workloads as wl
from tests import gpu_util as gu
from tests import kernel_cases as kc
from tests.test_gpu_gemm_parity import check, run_gemm, run_gemm_nn

pytestmark = pytest.mark.gpu


def _inputs(c, seed):
    fp8 = c["op"].startswith("fp8")
    cfg = dict(wl.CONFIGS[4 if fp8 else 1], d=c["d"], causal=c["causal"], scale=1.0 / c["d"] ** 0.5, seed=seed)
    size = dict(B=c.get("B", 1), Hq=c["H"], N=c["N"])
    return cfg, wl.make_inputs(cfg, Hkv=c.get("Hkv", c["H"]), **size), size


def _persistent(inp, split):
    """attn_fwd_persistent; the queue's counters say whether tiles were taken from it."""
    import paper_2605_10905_amd as A

    dev = gu.to_device(inp)
    B, Hq, Hkv, N, d = (inp[k] for k in ("B", "Hq", "Hkv", "N", "d"))
    o = torch.full((B, Hq, N, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, Hq, N), float("nan"), dtype=torch.float32, device="cuda")
    queue = torch.full((A.attn_persistent_queue_bytes() // 4,), -77, dtype=torch.int32, device="cuda")
    A.attn_fwd_persistent(dev["q"], dev["k"], dev["v"], o, lse, B, Hq, Hkv, N, d, inp["causal"], inp["scale"], A.ATTN_BF16, queue)
    torch.cuda.synchronize()
    taken = queue[::32].cpu()  # eight counters, a 128-byte line apart
    if split:
        assert bool((queue == -77).all())
    else:
        assert int(taken.min()) >= 0 and int(taken.sum()) >= A.attn_num_workgroups(B, Hq, N, 256), taken
    return o, lse


@pytest.mark.parametrize("names,c", kc.ATTENTION, ids=[kc.case_id(r) for r in kc.ATTENTION])
def test_attention_kernel(names, c):
    import paper_2605_10905_amd as A

    cfg, inp, size = _inputs(c, 6100 + c["H"] + c["N"] + c["d"])
    print(f"{c} launches {names}", flush=True)
    if c["op"] == "bwd":
        dob = wl.make_dout(cfg, **size)
        dq, dk, dv, _, _ = gu.run_gpu_bwd(inp, dob)
        gu.check_bwd_full(inp, dob, dq, dk, dv, str(c))
        return
    if c["op"] == "persistent":
        o, lse = _persistent(inp, split=len(names) == 1)
        o2, lse2 = gu.run_gpu(inp)  # the same results as attn_fwd, bit for bit
        assert torch.equal(o.view(torch.int16), o2.view(torch.int16)) and torch.equal(lse, lse2)
    elif c["op"] == "fwd_variant":
        o, lse = gu.run_gpu(inp, variant=c["variant"])
    elif c["op"] == "fp8_variant":
        dev, ds = gu.to_device(inp), inp["descale"]
        o = torch.full(inp["q"].shape, float("nan"), dtype=torch.bfloat16, device="cuda")
        lse = torch.full(inp["q"].shape[:3], float("nan"), dtype=torch.float32, device="cuda")
        A.attn_fwd_fp8_variant(dev["q"], dev["k"], dev["v"], o, lse, *(inp[k] for k in ("B", "Hq", "Hkv", "N", "d", "causal", "scale")), *ds,
                               c["variant"])
        torch.cuda.synchronize()
    else:
        o, lse = gu.run_gpu(inp)
    gu.check_full(inp, o, lse, str(c))


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("name", ["all_equal_scores", "dominant_key", "large_magnitude"])
def test_whole_tile_backward_on_degenerate_scores(name, causal):
    """The score patterns of test_bwd_adversarial_rows on more tiles than a split launch takes: 90 heads, each three
    query tiles and five key tiles (rows and sizes as for the whole-tile kernels above)."""
    rng = np.random.default_rng(16)
    H, N, d = 90, 513, 128
    q, k, v, do = (rng.standard_normal((1, H, N, d)).astype(np.float32) for _ in range(4))
    if name == "all_equal_scores":
        k[:] = 0.0
    elif name == "dominant_key":
        k[:, :, 5] = 32.0 * q[:, :, 300] / np.linalg.norm(q[:, :, 300], axis=-1, keepdims=True)
    else:
        q, k = q * 4, k * 4
    bits = [wl.f32_to_bf16_bits(x) for x in (q, k, v, do)]
    inp = dict(B=1, Hq=H, Hkv=H, N=N, d=d, causal=causal, scale=1.0 / d ** 0.5, dtype="bf16", q=bits[0], k=bits[1], v=bits[2], descale=(1.0, 1.0, 1.0))
    print(f"whole-tile backward {name} causal={causal}", flush=True)
    dq, dk, dv, _, _ = gu.run_gpu_bwd(inp, bits[3])
    gu.check_bwd_full(inp, bits[3], dq, dk, dv, f"whole-tile backward {name} causal={causal}", peaked=name != "all_equal_scores")


@pytest.mark.parametrize("names,c", kc.NN, ids=[kc.case_id(r) for r in kc.NN])
def test_nn_kernel(names, c):
    a, b = wl.make_gemm_inputs(6500 + c["M"] + c["N"] + c["K"], c["M"], c["N"], c["K"])
    print(f"{c} launches {names}", flush=True)
    check(run_gemm_nn(a, np.ascontiguousarray(b.T)), a, b, str(c))


def _splitk(c, a, b, poison):
    import paper_2605_10905_amd as A

    M, N, K = c["M"], c["N"], c["K"]
    out = torch.full((M, N), poison, dtype=torch.bfloat16, device="cuda")
    ws = torch.full((c["splits"], M * N), poison, dtype=torch.float32, device="cuda")
    assert ws.numel() * 4 == A.gemm_splitk_workspace_bytes(M, N, c["splits"])
    A.gemm_bf16_nt_splitk(a, b, out, M, N, K, c["splits"], ws)
    torch.cuda.synchronize()
    return out, ws


@pytest.mark.parametrize("names,c", kc.SPLITK, ids=[kc.case_id(r) for r in kc.SPLITK])
def test_splitk_kernel(names, c):
    ab, bb = wl.make_gemm_inputs(6900 + c["M"] + c["N"] + c["K"], c["M"], c["N"], c["K"])
    a, b = gu.bf16_to_device(ab), gu.bf16_to_device(bb)
    print(f"{c} launches {names}", flush=True)
    out, ws = _splitk(c, a, b, float("nan"))
    check(out, ab, bb, str(c))
    # whole slices of the workspace are written, at least two, and what lies behind them is not touched
    finite = torch.isfinite(ws)
    used = int(finite.all(dim=1).sum())
    assert used >= 2 and bool(finite[:used].all()) and not bool(finite[used:].any()), used
    again, _ = _splitk(c, a, b, 1.0e30)  # what the workspace held before is not read
    assert torch.equal(out.view(torch.int16), again.view(torch.int16))


def test_splitk_of_two_kernels_in_a_replayed_graph():
    c = next(c for names, c in kc.SPLITK if "m16" in names[0])
    ab, bb = wl.make_gemm_inputs(78, c["M"], c["N"], c["K"])
    a, b = gu.bf16_to_device(ab), gu.bf16_to_device(bb)
    import paper_2605_10905_amd as A

    want, ws = _splitk(c, a, b, float("nan"))
    out = torch.empty_like(want)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        A.gemm_bf16_nt_splitk(a, b, out, c["M"], c["N"], c["K"], c["splits"], ws)
    for rep in range(3):
        out.fill_(7.0)  # eager work between the replays
        ws.fill_(7.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), want.view(torch.int16)), f"replay {rep}"


# C of 96 MB and more is written with non-temporal stores: the row ends of an N that is no multiple of 8,
# through the library's choice and through both families of large tiles
@pytest.mark.parametrize("M,N,K,variant", [(400001, 121, 32, None), (9003, 5401, 64, None), (9003, 5401, 64, "256x256x64 ring2 mfma16x16x32"),
                                           (9003, 5401, 96, "128x256x64 ring3"), (9003, 5401, 96, "256x128x64 ring3")])
def test_nontemporal_stores_of_ragged_rows(M, N, K, variant):
    import paper_2605_10905_amd as A

    assert 2 * M * N >= 96e6
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    a, b = (torch.randn(s, generator=gen, device="cuda").bfloat16() for s in ((M, K), (N, K)))
    guard = 64
    buf = torch.full((M * N + 2 * guard,), 7.0, dtype=torch.bfloat16, device="cuda")
    c = buf[guard:guard + M * N].view(M, N)
    c.fill_(float("nan"))
    print(f"non-temporal stores {M}x{N}x{K} variant {variant}", flush=True)
    if variant is None:
        A.gemm_bf16_nt(a, b, c, M, N, K)
    else:
        A.gemm_bf16_nt_variant(a, b, c, M, N, K, next(v for v in range(A.gemm_num_variants()) if A.gemm_variant_name(v) == "bf16 nt " + variant))
    torch.cuda.synchronize()
    ref, mag = a.float() @ b.float().t(), a.float().abs() @ b.float().abs().t()  # (fp32: errs by less than the bound's second term)
    assert bool(((c.float() - ref).abs() <= 2.0 ** -8 * ref.abs() + K * 2.0 ** -22 * mag + 1e-30).all())
    assert bool((buf[:guard] == 7.0).all()) and bool((buf[guard + M * N:] == 7.0).all())


# the 16x16x32 kernels and every other variant with fewer stages than ring slots, a half last stage, ragged tiles
@pytest.mark.parametrize("M,N,K", [(257, 263, 32), (513, 259, 96), (130, 515, 160), (259, 129, 224), (300, 270, 2080)])
def test_nt_variants_with_a_half_last_stage(M, N, K):
    import paper_2605_10905_amd as A

    a, b = wl.make_gemm_inputs(7300 + K, M, N, K)
    for v in range(A.gemm_num_variants()):
        if K % A.gemm_variant_kmult(v) == 0:
            print(f"nt {M}x{N}x{K} variant {v} ({A.gemm_variant_name(v)})", flush=True)
            check(run_gemm(a, b, v), a, b, f"nt {M}x{N}x{K} variant {A.gemm_variant_name(v)}")


def test_queue_launch_in_a_replayed_graph():
    """attn_fwd_persistent with more tiles than a split launch takes: the queue is cleared by a kernel of its own,
    on every replay."""
    import paper_2605_10905_amd as A

    c = next(c for names, c in kc.ATTENTION if c["op"] == "persistent" and len(names) == 2 and c["causal"] and c["d"] == 128)
    _, inp, _ = _inputs(c, 6300)
    want, want_lse = _persistent(inp, split=False)
    dev = gu.to_device(inp)
    o, lse = torch.empty_like(want), torch.empty_like(want_lse)
    queue = torch.zeros(A.attn_persistent_queue_bytes() // 4, dtype=torch.int32, device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        A.attn_fwd_persistent(dev["q"], dev["k"], dev["v"], o, lse, *(inp[k] for k in ("B", "Hq", "Hkv", "N", "d", "causal", "scale")), A.ATTN_BF16, queue)
    for rep in range(3):
        for t in (o, lse, queue):
            t.fill_(7)  # eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(o.view(torch.int16), want.view(torch.int16)) and torch.equal(lse, want_lse), f"replay {rep}"


def _one_tile_each(run, q, k, v, limit):
    """run(q, k, v) on as many heads at a time as stay below `limit` 256-row tiles: one tile for every workgroup."""
    B, H, N, _ = q.shape
    G, T = H // k.shape[1], (N + 255) // 256
    step = max(1, (limit - 1) // (T * G))
    parts = [run(*(x[b:b + 1, i * g:(i + step) * g].contiguous() for x, g in ((q, G), (k, 1), (v, 1)))) for b in range(B) for i in range(0, k.shape[1], step)]
    return [torch.cat([p[i].flatten(0, 1) for p in parts]).view(B, H, *parts[0][i].shape[2:]) for i in range(2)]


@pytest.mark.parametrize("names,c", kc.RESIDENT, ids=[kc.case_id(r) for r in kc.RESIDENT])
def test_resident_workgroups_give_the_bytes_of_single_tiles(names, c):
    """Workgroups that take several tiles, one after the other: the same bytes as launches of one tile for every workgroup."""
    import paper_2605_10905_amd as A

    B, H, Hkv, N, d, causal, op = c.get("B", 1), c["H"], c["Hkv"], c["N"], c["d"], c["causal"], c["op"]
    whole = next(v for v in range(A.attn_num_variants()) if A.attn_variant_name(v).startswith(f"bf16 d{d} whole tiles"))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(71 + N + d)
    q, k, v = (torch.randn((B, h, N, d), generator=gen, device="cuda") for h in (H, Hkv, Hkv))
    q, k, v = (x.to(torch.float8_e4m3fn).view(torch.uint8) if op == "fp8" else x.bfloat16() for x in (q, k, v))

    def run(q, k, v, queue=None):
        o = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device="cuda")
        lse = torch.full(q.shape[:3], float("nan"), device="cuda")
        sizes = (q.shape[0], q.shape[1], k.shape[1], N, d, causal, d ** -0.5)
        if op == "fp8":
            A.attn_fwd_fp8(q, k, v, o, lse, *sizes, 1.0, 1.0, 1.0)
        elif queue is not None:
            A.attn_fwd_persistent(q, k, v, o, lse, *sizes, A.ATTN_BF16, queue)
        else:
            A.attn_fwd_variant(q, k, v, o, lse, *sizes, A.ATTN_BF16, whole)
        torch.cuda.synchronize()
        return o, lse

    print(f"{c} launches {names}", flush=True)
    queue = torch.full((A.attn_persistent_queue_bytes() // 4,), -77, dtype=torch.int32, device="cuda") if op == "persistent" else None
    o, lse = run(q, k, v, queue)
    if op == "persistent":
        assert int(queue[::32].min()) >= 0 and int(queue[::32].sum()) >= A.attn_num_workgroups(B, H, N, 256)
    want, want_lse = _one_tile_each(run, q, k, v, 768)
    assert bool(torch.isfinite(want.float()).all()) and bool(torch.isfinite(want_lse).all())
    assert torch.equal(o.view(torch.int16), want.view(torch.int16)) and torch.equal(lse, want_lse)


# Scores that rise by `step` (in powers of two) from one 32-key block to the next: which of them raise the reference, and against which one
# a block is rounded, depends on the form; all forms stay within the tolerances.
@pytest.mark.parametrize("step", [9.0, 12.0, 15.0])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d", [64, 128])
def test_forms_on_scores_that_rise_from_block_to_block(d, causal, step):
    import paper_2605_10905_amd as A

    forms = [v for v in range(A.attn_num_variants()) if A.attn_variant_name(v).startswith(f"bf16 d{d} ")]
    assert len(forms) == 4
    rng = np.random.default_rng(81 + d)
    for N in (33, 95, 96, 97, 127, 128, 129, 160, 191, 192, 224, 257, 300):
        q, k, v = (0.25 * rng.standard_normal((1, 3, N, d)).astype(np.float32) for _ in range(3))
        q[..., 0] = 8.0
        k[..., 0] = step * (np.arange(N) // 32) / (8.0 * d ** -0.5 * 1.4426950408889634)
        bits = [wl.f32_to_bf16_bits(x) for x in (q, k, v)]
        inp = dict(B=1, Hq=3, Hkv=3, N=N, d=d, causal=causal, scale=d ** -0.5, dtype="bf16", q=bits[0], k=bits[1], v=bits[2], descale=(1.0, 1.0, 1.0))
        for form in forms:
            label = f"rising scores d={d} causal={causal} step={step} N={N} {A.attn_variant_name(form)}"
            print(label, flush=True)
            o, lse = gu.run_gpu(inp, variant=form)
            gu.check_full(inp, o, lse, label)

"""For every kernel of the library a call that launches it: what test_dispatch.py (no GPU) holds against the
routes the library takes and test_gpu_kernels.py runs against the oracle.

The rules that choose between kernels depend on sizes alone, and most small shapes take the same few of them:
a size that is meant for one kernel stops reaching it when a rule changes.  Each row names what it launches, in
order, so that it then fails instead of testing something else.  Sizes are ragged on purpose."""


def _fwd(d, causal, mode, form, **size):
    call = dict(op=size.pop("op", "fwd"), d=d, causal=causal, **size)
    fp8 = "true" if call["op"] in ("fp8", "fp8_variant") else "false"
    kernel = f"attn_fwd_sp_kernel<{d}, {str(causal).lower()}, {mode}, {fp8}, {form}>"
    return ([kernel] if mode != 1 else ["attn_queue_reset_kernel", kernel]), call


def _bwd(d, causal, q, k, **size):
    """q: 1 and 2 for dQ workgroups of 128 and 64 queries, "wide" for 256; k: 1 and 2 for dK/dV workgroups of 128 and 64 keys."""
    c = str(causal).lower()
    dq = f"attn_bwd_dq_wide_kernel<{d}, {c}>" if q == "wide" else f"attn_bwd_dq_kernel<{d}, {c}, {q}>"
    return [dq, f"attn_bwd_dkv_pipe_kernel<{d}, {c}, {k}>"], dict(op="bwd", d=d, causal=causal, **size)


ATTENTION = []
for _d in (64, 128):
    ATTENTION += [
        # few tiles: two waves share 32 queries; some more: one tile a workgroup; many: paired workgroups of 128 queries
        _fwd(_d, False, 0, 2, H=6, Hkv=3, N=517), _fwd(_d, True, 0, 2, H=6, Hkv=2, N=517),
        _fwd(_d, False, 0, 1, H=70, Hkv=35, N=513), _fwd(_d, True, 0, 3, H=90, Hkv=45, N=513), _fwd(_d, True, 0, 1, H=64, Hkv=32, N=600),
        _fwd(_d, False, 0, 3, H=90, Hkv=45, N=513), _fwd(_d, False, 0, 3, B=2, H=130, Hkv=65, N=129), _fwd(_d, True, 0, 3, H=520, Hkv=260, N=300),
        # three or more 256-row tiles per CU: one workgroup per CU walks a list of them (d = 64: long launches, and here by the variant)
        _fwd(_d, True, *((2, 1) if _d == 128 else (0, 3)), H=800, Hkv=400, N=201), _fwd(_d, True, *((2, 1) if _d == 128 else (0, 3)), B=3, H=130, Hkv=65, N=430),
        *[_fwd(_d, c, 2, 1, op="fwd_variant", variant=4 if _d == 128 else 5, H=800, Hkv=400, N=201) for c in (False, True)],
        # the queue: more tiles than start at once (paired), and whole tiles; few tiles leave it alone
        _fwd(_d, False, 1, 3, op="persistent", H=520, Hkv=260, N=300), _fwd(_d, True, 1, 3, op="persistent", H=520, Hkv=260, N=300),
        _fwd(_d, False, 1, 1, op="persistent", H=64, Hkv=32, N=600), _fwd(_d, True, 1, 1, op="persistent", H=70, Hkv=35, N=513),
        _fwd(_d, False, 0, 2 if _d == 64 else 3, op="persistent", H=5, N=300), _fwd(_d, True, 0, 2, op="persistent", H=5, N=300),
        _fwd(_d, False, 0, 2, op="persistent", H=5, N=517), _fwd(_d, False, 0, 3, op="persistent", H=130, Hkv=65, N=257),
        _bwd(_d, False, 2, 2, H=6, Hkv=3, N=517), _bwd(_d, True, 2, 2, H=6, Hkv=2, N=517), _bwd(_d, False, 1, 2, H=140, Hkv=20, N=513),
    ]
# backward, the launches whose form depends on the head dimension
ATTENTION += [
    _bwd(128, False, "wide", 1, H=70, N=513), _bwd(128, False, "wide", 1, H=70, Hkv=35, N=513), _bwd(128, False, "wide", 2, H=144, Hkv=72, N=133), _bwd(128, False, 1, 1, H=90, N=513),
    _bwd(128, True, 1, 1, H=90, N=513), _bwd(128, True, "wide", 1, H=180, Hkv=90, N=300), _bwd(128, True, 1, 2, H=90, Hkv=45, N=513), _bwd(128, True, "wide", 2, H=144, Hkv=72, N=133),
    _bwd(64, False, 1, 2, H=70, N=513), _bwd(64, False, 1, 2, H=70, Hkv=35, N=513), _bwd(64, False, 1, 1, H=46, N=513), _bwd(64, False, "wide", 2, H=192, Hkv=48, N=162),
    _bwd(64, False, "wide", 2, H=234, Hkv=117, N=390), _bwd(64, True, 1, 2, H=90, N=513), _bwd(64, True, "wide", 2, H=180, Hkv=90, N=300), _bwd(64, True, 1, 2, H=90, Hkv=45, N=513),
    _bwd(64, True, "wide", 2, H=300, Hkv=75, N=133), _bwd(64, True, 1, 1, H=60, N=513),
]
ATTENTION += [
    _fwd(128, False, 0, 1, op="fp8", H=4, Hkv=2, N=517), _fwd(128, True, 0, 1, op="fp8", H=4, Hkv=2, N=517),
    _fwd(128, True, 2, 1, op="fp8", H=800, Hkv=400, N=201), _fwd(128, False, 2, 1, op="fp8", H=800, Hkv=400, N=201),
    # more than three rounds of tiles, a fifth of them light: non-causal lists would be dealt unevenly
    _fwd(128, False, 0, 1, op="fp8", B=5, H=32, Hkv=16, N=1130),
    # four tiles and more for each resident workgroup of the queue
    _fwd(128, False, 1, 1, op="persistent", H=1000, Hkv=500, N=250), _fwd(128, True, 1, 1, op="persistent", H=800, Hkv=400, N=201),
    (["attn_fwd_fp8_kernel<128, false>"], dict(op="fp8_variant", variant=3, H=4, Hkv=2, N=517, d=128, causal=False)),
    (["attn_fwd_fp8_kernel<128, true>"], dict(op="fp8_variant", variant=3, H=4, Hkv=2, N=517, d=128, causal=True)),
]


# Workgroups that stay resident and take several tiles, by the list (three or more 256-row tiles for every CU; K/V heads a multiple of
# eight and not) and from the queue (whole tiles and paired).  Lengths: an odd number of key tiles, enough of them for the
# ring's unrolled loop, last query tiles of few rows.
RESIDENT = []
for _c in (False, True):
    for _B, _H, _Hkv, _N in ((1, 256, 64, 700), (1, 300, 100, 700), (3, 24, 12, 2900)):
        RESIDENT += [_fwd(128, _c, 2, 1, op="fp8", B=_B, H=_H, Hkv=_Hkv, N=_N)]
        RESIDENT += [_fwd(_d, _c, 2, 1, op="fwd_variant", variant=4 if _d == 128 else 5, B=_B, H=_H, Hkv=_Hkv, N=_N) for _d in (64, 128)]
    for _form, _B, _H, _Hkv, _N in ((1, 1, 64, 16, 4200), (1, 1, 40, 10, 4200), (1, 3, 16, 8, 4200), (3, 1, 300, 300, 270), (3, 5, 44, 11, 530)):
        RESIDENT += [_fwd(_d, _c, 1, _form, op="persistent", B=_B, H=_H, Hkv=_Hkv, N=_N) for _d in (64, 128)]


def _nn(kernel, M, N, K):
    return [kernel], dict(op="nn", M=M, N=N, K=K)


NN = [
    _nn("gemm_bf16_kernel<1, 2, 32, 4, 3, true>", 37, 72, 32), _nn("gemm_bf16_kernel<1, 2, 32, 4, 3, true>", 1111, 1000, 1056),
    _nn("gemm_bf16_kernel<1, 4, 32, 4, 2, true>", 8413, 208, 160),
    _nn("gemm_bf16_kernel<2, 2, 32, 4, 2, true>", 2270, 920, 224),
    _nn("gemm_bf16_kernel<2, 4, 32, 3, 2, true>", 2593, 2896, 64), _nn("gemm_bf16_kernel<2, 4, 32, 3, 2, true>", 1006, 7416, 96),
    _nn("gemm_bf16_kernel<4, 2, 32, 3, 2, true>", 5757, 1384, 224),
    _nn("gemm_bf16_kernel<4, 4, 32, 4, 1, true>", 5799, 2600, 320), _nn("gemm_bf16_kernel<4, 4, 32, 4, 1, true>", 3790, 3376, 416),
    _nn("gemm_wavek_kernel<1, 2, 8, 5, true, false>", 1, 8, 256), _nn("gemm_wavek_kernel<1, 2, 8, 5, true, false>", 53, 104, 3424),
    _nn("gemm_wavek_kernel<2, 4, 8, 3, true, false>", 5722, 8, 480), _nn("gemm_wavek_kernel<4, 2, 8, 3, true, false>", 2742, 136, 992),
]


def _sk(kernel, vec, M, N, K, splits):
    return [kernel, f"gemm_splitk_sum_kernel<{vec}>"], dict(op="splitk", M=M, N=N, K=K, splits=splits)


# split-K: rows of partial tiles that start at every alignment (N not a multiple of 4), slices of which the last
# is shorter, and the sum over an element count that is or is not a multiple of four
SPLITK = [
    _sk("gemm_bf16_nt_m16_kernel<64, 2, true, true>", "false", 1413, 758, 11008, 13), _sk("gemm_bf16_nt_m16_kernel<64, 2, true, true>", "true", 2052, 523, 17856, 11),
    _sk("gemm_bf16_nt_m16_kernel<64, 2, true, true>", "true", 1413, 760, 11072, 13),
    _sk("gemm_bf16_nt_m16_kernel<64, 2, true, false>", "false", 2757, 143, 15808, 13), _sk("gemm_bf16_nt_m16_kernel<64, 2, true, false>", "true", 196, 2323, 19328, 13),
    _sk("gemm_wavek_kernel<1, 1, 4, 4, false, true>", "false", 1, 1, 6848, 11), _sk("gemm_wavek_kernel<1, 1, 4, 4, false, true>", "false", 35, 37, 9152, 13),
    _sk("gemm_wavek_kernel<1, 1, 4, 4, false, true>", "true", 21, 52, 7104, 9),
    _sk("gemm_wavek_kernel<2, 2, 4, 2, false, true>", "false", 561, 1, 15744, 13), _sk("gemm_wavek_kernel<2, 2, 4, 2, false, true>", "true", 2, 706, 8512, 9),
    _sk("gemm_wavek_kernel<2, 4, 4, 3, false, true>", "false", 3, 1515, 20160, 14), _sk("gemm_wavek_kernel<2, 4, 4, 3, false, true>", "true", 42, 814, 25664, 9),
    _sk("gemm_wavek_kernel<4, 1, 8, 2, false, true>", "false", 1025, 3, 12736, 13), _sk("gemm_wavek_kernel<4, 1, 8, 2, false, true>", "true", 1484, 5, 19136, 8),
    _sk("gemm_wavek_kernel<4, 4, 4, 2, false, true>", "false", 197, 401, 10752, 15), _sk("gemm_wavek_kernel<4, 4, 4, 2, false, true>", "true", 101, 1304, 8768, 12),
]


def case_id(row):
    c = row[1]
    size = "x".join(str(c[k]) for k in ("M", "N", "K")) if "M" in c else \
        f"{c.get('B', 1)}x{c['H']}/{c.get('Hkv', c['H'])}xN{c['N']}d{c['d']}{'c' if c['causal'] else 'n'}"
    return f"{c['op']}-{size}"

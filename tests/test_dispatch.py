"""Routes of the public calls, without a GPU: which kernels a call launches, and that no size which fits a
launch is refused."""
import ctypes
import heapq
import math
import os
import random
import subprocess

import pytest

import paper_2605_10905_amd as A
from tests import kernel_cases as kc
from tests.launch_recorder import ROOT, routes


def test_very_many_rows_are_launched():
    """Up to 2^31 - 256 rows of few columns fit one launch; so do as many columns (70 GB and 140 GB of operands)."""
    most = 2 ** 31 - 256
    calls = [dict(op="nt", M=1_100_000_000, N=32, K=32), dict(op="nn", M=1_100_000_000, N=32, K=32), dict(op="nt", M=1, N=1_100_000_000, K=32),
             dict(op="nt", M=most, N=1, K=32), dict(op="nn", M=most, N=8, K=32), dict(op="splitk", M=most, N=1, K=64, splits=2)]
    got, _ = routes(calls)
    for c, (status, launches) in zip(calls, got):
        assert status == 0 and len(launches) == 1, (c, status, launches)
        name, grid, threads = launches[0]
        assert grid * threads < 2 ** 32 and grid >= max(c["M"], c["N"]) // 256, (c, launches)


def test_every_row_of_the_kernel_cases_launches_the_kernel_it_names():
    rows = kc.ATTENTION + kc.RESIDENT + kc.NN + kc.SPLITK
    got, _ = routes([c for _, c in rows])
    wrong = [(c, names, launches) for (names, c), (st, launches) in zip(rows, got) if st != 0 or [x[0] for x in launches] != names]
    assert not wrong, "\n".join(map(str, wrong))
    for (_, c), (_, launches) in zip(rows, got):
        if c["op"] == "splitk":  # more slices than one, and a last one that is shorter
            slices = _slices(c["M"], c["N"], *launches[0][:2])
            assert 1 < slices <= c["splits"], (c, slices)


def _slices(M, N, kernel, workgroups):
    """Slices of k of a split-K launch, from its number of workgroups."""
    a = [int(x) for x in kernel[kernel.index("<") + 1:-1].split(",")[:2]]
    bm, bn = (256, 256) if "m16" in kernel else (16 * a[0], 16 * a[1])
    tiles = -(-M // bm) * -(-N // bn)
    assert workgroups % tiles == 0
    return workgroups // tiles


def _variant_calls():
    return [dict(op="nt_variant", M=300, N=520, K=3 * A.gemm_variant_kmult(v), variant=v) for v in range(A.gemm_num_variants())]


def _form_calls():
    calls = []
    for v in range(A.attn_num_variants()):
        name = A.attn_variant_name(v)
        if name.startswith("bf16"):
            calls += [dict(op="fwd_variant", variant=v, H=2, N=300, d=int(name.split(" d")[1].split()[0]), causal=c) for c in (False, True)]
    return calls


def test_a_backward_too_large_for_a_launch_launches_nothing():
    """The dQ grid counts workgroups of 128 query rows, so that heads of 129 have two: what does not fit is refused before anything is enqueued."""
    calls = [dict(op=op, H=H, Hkv=Hkv, N=N, d=d) for op, H, Hkv, N, d in (("bwd", 2 ** 30 + 8, 1, 129, 64), ("bwd", 2 ** 24, 1, 128, 64), ("bwd", 2 ** 24, 2 ** 24, 128, 128),
                                                                         ("bwd", 2 ** 23, 2 ** 23, 256, 128), ("bwd", 2 ** 31 - 1, 1, 1, 64))]
    fits = [dict(op="bwd", H=2 ** 23 - 8, Hkv=8, N=N, d=d, causal=c) for N in (1, 128, 129, 256) for d in (64, 128) for c in (False, True)]
    got, _ = routes(calls + fits)
    for c, (st, launches) in zip(calls, got):
        assert st != 0 and not launches, (c, st, launches)
    for c, (st, launches) in zip(fits, got[len(calls):]):
        assert st == 0 and len(launches) == 2, (c, st, launches)


def test_every_kernel_is_launched_by_a_case_that_a_gpu_test_runs():
    """The rows of kernel_cases.py, and every variant of gemm_bf16_nt_variant, which the GEMM's tests run one by one."""
    got, kernels = routes([c for _, c in kc.ATTENTION + kc.NN + kc.SPLITK] + _variant_calls())
    assert all(st == 0 for st, _ in got)
    missing = kernels - {x[0] for _, launches in got for x in launches}
    assert not missing, sorted(missing)


def test_what_the_nt_product_chooses_is_among_the_variants():
    rng = random.Random(20260514)

    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    chosen = [dict(op="nt", M=log(1, 600000), N=log(1, 65536), K=32 * log(1, 512)) for _ in range(4000)]
    variants = _variant_calls()
    got, _ = routes(variants + chosen)
    assert all(st == 0 and len(launches) == 1 for st, launches in got)
    names = [launches[0][0] for _, launches in got]
    assert len(set(names[:len(variants)])) >= len(variants) - 1  # (one kernel is listed twice: whole and half last stages)
    assert set(names[len(variants):]) <= set(names[:len(variants)])


def test_the_forms_of_the_forward_are_forced_by_their_variants():
    """"whole tiles", "split keys" and "paired" run that form whatever the size; "pipelined" follows the rule."""
    calls = _form_calls()
    got, _ = routes(calls)
    for c, (st, launches) in zip(calls, got):
        name = A.attn_variant_name(c["variant"])
        # (2 heads of 300 are few tiles: the rule splits their keys, or, for non-causal chains of ten steps at d = 128, pairs workgroups)
        by_rule = 3 if c["d"] == 128 and not c["causal"] else 2
        form = next((f for word, f in (("whole", 1), ("split", 2), ("paired", 3)) if word in name), by_rule)
        assert st == 0 and [x[0] for x in launches] == [f"attn_fwd_sp_kernel<{c['d']}, {str(c['causal']).lower()}, 0, false, {form}>"], (c, launches)


@pytest.mark.parametrize("tiles_m,tiles_n,splits", [(1, 1, 2), (9, 4, 7), (5, 3, 13), (63, 1, 4), (2, 17, 64), (8, 8, 3)])
def test_split_tile_map_is_a_bijection_and_keeps_an_xcd_on_few_slices(tmp_path, tiles_m, tiles_n, splits):
    """gemm_tile_coord_split, compiled from its header: every (slice, tile) once, and an XCD (workgroup ids that
    agree mod 8) takes a consecutive piece of the list of slices."""
    src, lib = tmp_path / "map.cpp", tmp_path / "map.so"
    src.write_text('#define GEMM_HD\n#include "gemm_map.h"\nextern "C" void coord(int wg, int m, int n, int splits, int* out) {\n'
                   "  const GemmTileCoord c = gemm_tile_coord_split(wg, m, n, splits, out);\n  out[1] = c.tm;\n  out[2] = c.tn;\n}\n")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2605_10905_amd", "csrc"), str(src), "-o", str(lib)], check=True)
    out, coord = (ctypes.c_int * 3)(), ctypes.CDLL(str(lib)).coord
    total = tiles_m * tiles_n * splits
    seen, slices = set(), {}
    for wg in range(total):
        coord(wg, tiles_m, tiles_n, splits, out)
        seen.add(tuple(out))
        slices.setdefault(wg % 8, set()).add(out[0])
    assert seen == {(s, i, j) for s in range(splits) for i in range(tiles_m) for j in range(tiles_n)}
    share = -(-total // 8)  # entries of the list an XCD takes
    assert all(max(s) - min(s) + 1 == len(s) <= (share - 1 + tiles_m * tiles_n - 1) // (tiles_m * tiles_n) + 1 for s in slices.values())



def test_causal_launch_model_against_a_plain_queue_of_workgroups(tmp_path):
    """attn_causal_us, by which the causal forms are weighed, keeps places that come free at the same time together; here every
    workgroup is handed out by itself, in the order that attn_tile_coord gives, to the place that is free first."""
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text("#pragma once\ntypedef void* hipStream_t;\n")
    src, lib = tmp_path / "model.cpp", tmp_path / "model.so"
    src.write_text('#define ATTN_HD\n#include "attn_kernels.h"\nextern "C" double model(int B, int Hq, int Hkv, int T, int slots, double P, double a, double b, double heaviest, double less, double top) {\n'
                   "  return attn_causal_us(AttnFormCost{0.5, P, a, b, 0.0}, attn_tile_map_make(B, Hq, Hkv, T, 1), (long long)B * Hq * T, slots, heaviest, less, top);\n}\n")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", str(tmp_path), "-I", os.path.join(ROOT, "paper_2605_10905_amd", "csrc"), str(src), "-o", str(lib)], check=True)
    model = ctypes.CDLL(str(lib)).model
    model.restype, model.argtypes = ctypes.c_double, [ctypes.c_int] * 5 + [ctypes.c_double] * 6
    rng = random.Random(7)
    b, hq, t = ctypes.c_int(), ctypes.c_int(), ctypes.c_int()
    for _ in range(60):
        B, Hkv, G, T, slots = rng.randint(1, 6), rng.choice((1, 3, 8, 12, 16)), rng.choice((1, 2, 4)), rng.randint(1, 12), rng.randint(1, 3)
        n, P, a, share, less = B * Hkv * G * T, rng.uniform(2, 8), rng.uniform(0.2, 1), rng.uniform(0, 0.4), rng.choice((2.0, 4.0, 8.0))
        heaviest = T * less - rng.choice((0.0, 1.0))
        top = heaviest - rng.choice((0.0, 1.5))
        step = a + share * (min(-(-n // 256), slots) - 1)
        lists = 8 if B * Hkv % 8 == 0 else 1
        places = [[0.0] * (256 * slots // lists) for _ in range(lists)]
        for wg in range(n):
            assert A.lib.attn_tile_coord(wg, B, Hkv * G, Hkv, T * 256, 256, 1, ctypes.byref(b), ctypes.byref(hq), ctypes.byref(t)) == 0
            heapq.heapreplace(places[wg % lists], places[wg % lists][0] + P + min(heaviest - (T - 1 - t.value) * less, top) * step)
        want = 0.5 + max(max(x) for x in places)
        got = model(B, Hkv * G, Hkv, T, slots, P, a, share, heaviest, less, top)
        assert abs(got - want) < 1e-6 * want, (B, Hkv, G, T, slots, got, want)
    assert 0 < model(8, 64, 64, 1000, 2, 5.0, 0.5, 0.2, 1000.0, 1.0, 1000.0) < 1e6  # (more ranks than are followed)


# Sizes at which the forms of the bf16 forward differ, us, all measured in turn (w: whole tiles, s: split keys, p: paired workgroups);
# (heads, N, causal, d, the forms within 7 % of the fastest)
_FORMS = [(32, 1000, False, 128, "sp"),     # w 25.8, s 20.9, p 21.3
          (34, 2048, False, 128, "p"),      # w 102.2, s 97.0, p 89.9
          (22, 4096, False, 128, "sp"),     # w 189.5, s 178.8, p 177.4
          (90, 1000, False, 128, "wp"),     # w 61.1, s 73.3, p 64.8; s: the third round costs more than the shorter chain gives
          (68, 1000, False, 128, "wp"),     # w 59.4, s 67.3, p 59.1
          (38, 1000, False, 128, "w"),      # w 28.0, s 41.2, p 34.7
          (150, 150, False, 128, "w"),      # w 10.2, s 17.5, p 12.5
          (150, 150, True, 128, "wp"),      # w 10.3, s 15.9, p 10.2; s: 300 half tiles do not start at once
          (150, 150, True, 64, "wp"),       # w 7.5, s 11.2, p 7.3
          (58, 1000, True, 128, "wp"),      # w 30.0, s 32.8, p 28.5
          (85, 513, True, 64, "wp"),        # w 13.1, s 16.5, p 12.1 (w is 8 % behind)
          (32, 1000, True, 128, "s"),       # w 25.6, s 18.7, p 20.2
          (48, 1000, True, 128, "sp"),      # w 26.2, s 25.4, p 24.5
          (16, 4096, True, 128, "s"),       # w 84.4, s 70.4, p 79.6
          (75, 300, True, 128, "sp"),       # w 13.1, s 11.1, p 10.8; s: 225 half tiles, fewer than the 300 that twice the tiles would be
          (34, 4096, True, 64, "w"),        # w 127.9, s 117.8, p 105.7 (the rule for paired workgroups leaves this one out)
          (100, 64, False, 128, "wp"),      # w 6.0, s 6.9, p 5.7; s: as many tiles, and a merge
          (2, 40, False, 128, "wp"),        # w 5.5, s 6.5, p 5.5
          (100, 90, True, 64, "wp"),        # w 6.0, s 6.3, p 5.8
          (34, 2048, False, 64, "p"),       # w 68.2, s 63.3, p 52.5
          (24, 2048, False, 64, "w"),       # w 32.5, s 39.4, p 35.4
          (128, 2048, False, 64, "wp"),     # w 148.4, s 172.0, p 142.0
          (192, 327, True, 64, "p"),        # w 16.0, s 19.8, p 13.3
          (512, 903, True, 64, "p"),        # w 100.1, s 131.8, p 91.2
          (64, 8192, True, 128, "w"),       # w 889.7, s 1017.5, p 960.7
          (64, 8192, False, 128, "w"),      # w 1711.7, s 1871.2, p 1806.2
          (128, 568, True, 128, "w"),       # w 25.6, s 33.4, p 29.8
          (72, 1050, True, 64, "w")]        # w 24.1, s 32.4, p 28.0


@pytest.mark.parametrize("op", ["fwd", "persistent"])
def test_the_forward_takes_the_faster_form(op):
    got, _ = routes([dict(op=op, H=h, N=n, causal=c, d=d) for h, n, c, d, _ in _FORMS])
    wrong = [(f, launches) for f, (st, launches) in zip(_FORMS, got) if st != 0 or "wsp"[int(launches[-1][0][-2]) - 1] not in f[4]]
    assert not wrong, wrong


# Non-causal launches of three and more 256-row tiles per CU, us, lists / one tile per workgroup (heads, K/V heads, N, d or "fp8", lists are right)
_LISTS = [(160, 160, 1138, 128, False),      # 128.1 / 119.0: 3.1 rounds, a fifth of the tiles light
          (60, 15, 3080, 64, False),         # 192.9 / 180.3
          (384, 48, 577, 128, False),        # 92.2 / 87.0
          (72, 36, 2620, "fp8", False),      # 222.5 / 204.7
          (160, 80, 1130, "fp8", False),     # 104.9 / 93.0
          (512, 512, 513, "fp8", True),      # 82.0 / 90.7
          (768, 768, 257, "fp8", True),      # 51.8 / 58.7
          (192, 192, 1500, "fp8", True),     # 175 / 184
          (64, 64, 8192, 128, True)]         # no light tiles


def test_lists_of_uneven_tiles_are_not_walked():
    call = lambda h, g, n, d: dict(op="fp8", H=h, Hkv=g, N=n) if d == "fp8" else dict(op="fwd_variant", variant=4 if d == 128 else 5, H=h, Hkv=g, N=n, d=d)
    got, _ = routes([call(h, g, n, d) for h, g, n, d, _ in _LISTS])
    wrong = [(r, launches) for r, (st, launches) in zip(_LISTS, got) if st != 0 or (", 2, " in launches[0][0]) != r[4]]
    assert not wrong, wrong


# Backward passes in which only the form of dK/dV changes, us, keys 128 a workgroup -> 64 (heads, K/V heads, N, causal, d, 64 is right)
_DKV = [(384, 96, 297, False, 64, True),     # 72.1 -> 53.9
        (192, 96, 263, False, 64, True),     # 44.2 -> 34.2
        (36, 18, 1994, False, 64, True),     # 198 -> 165
        (120, 30, 1144, False, 64, True),    # 213 -> 179
        (24, 12, 2412, True, 64, True),      # 112 -> 90
        (384, 48, 547, True, 64, True),      # 123 -> 100
        (36, 36, 925, True, 64, False),      # 37.1 -> 45.6
        (72, 72, 490, True, 64, False),      # 26.3 -> 29.8
        (1, 1, 59, True, 64, False),         # 9.8 -> 10.2
        (60, 30, 2179, True, 128, True),     # 364 -> 311
        (12, 12, 1000, False, 128, True),    # 75 -> 67
        (16, 16, 2048, False, 128, False)]   # 140 -> 151


def test_the_backward_takes_the_faster_form_of_dkv():
    got, _ = routes([dict(op="bwd", H=h, Hkv=g, N=n, causal=c, d=d) for h, g, n, c, d, _ in _DKV])
    wrong = [(r, launches) for r, (st, launches) in zip(_DKV, got) if st != 0 or (launches[1][0][-2] == "2") != r[5]]
    assert not wrong, wrong


# The same for dQ, 128 / 64 / 256 queries a workgroup (..., the forms within 4 % of the fastest)
_DQ = [(256, 128, 133, False, 128, "w"),     # 38.2 / 43.8 / 31.9
       (144, 36, 146, False, 128, "w"),      # 46.0 / 42.4 / 38.0
       (160, 160, 152, True, 128, "w"),      # 31.9 / 31.3 / 27.9
       (60, 30, 2179, True, 128, "1"),       # 364 / 396 / 421
       (20, 20, 3449, True, 128, "2w"),      # 327 / 304 / 309
       (80, 80, 22, False, 64, "w"),         # 9.1 / 9.2 / 8.7
       (320, 160, 130, False, 64, "w"),      # 35.9 / 35.5 / 32.5
       (512, 128, 132, True, 64, "w"),       # 34.1 / 38.9 / 30.7
       (128, 64, 522, True, 64, "w"),        # 48.3 / 47.0 / 41.8
       (384, 192, 23, True, 64, "12"),       # 13.4 / 13.4 / 14.2
       (2, 2, 656, True, 128, "2")]          # 41 / 38 / 49


def test_the_backward_takes_the_faster_form_of_dq():
    got, _ = routes([dict(op="bwd", H=h, Hkv=g, N=n, causal=c, d=d) for h, g, n, c, d, _ in _DQ])
    form = [("w" if "wide" in launches[0][0] else launches[0][0][-2]) for _, launches in got]
    wrong = [(r, f) for r, f in zip(_DQ, form) if f not in r[5]]
    assert not wrong, wrong

// Internal interface between the C-ABI entry points and the HIP kernels.
#pragma once
#include <hip/hip_runtime.h>

#include "tile_map.h"

struct AttnParams {
  const void* q;
  const void* k;
  const void* v;
  void* o;
  float* lse;
  int B, Hq, Hkv, N;
  int T;             // query tiles per head = ceil(N / BM)
  int causal;
  float scale_log2;  // scale * log2(e) (times q_descale*k_descale for fp8)
  float out_scale;   // multiplies O in the epilogue (v_descale and P scaling for fp8; 1 for bf16)
  int* queue = nullptr;  // persistent launch only: 8 tile-list counters, 32 ints apart
  int total = 0;         // persistent launch only: number of query tiles = B * Hq * T
  AttnTileMap map;       // attn_tile_map_make(B, Hq, Hkv, T, causal): workgroup id -> (batch, head, tile)
};

// Whether a launch of `whole` workgroups, the longest `steps` serial 32-row block steps each, is better run
// as `split` workgroups of about half the chain each, on 256 CUs with one workgroup each.  In units of a
// step of the whole form: a workgroup costs `fixed` (`fixed_split`) beside its chain (first loads, merge,
// stores), a step of the split form `slower`.
//   equal tiles: whole rounds over the CUs, the last one at `last` of its chain's cost if it is nearly empty
//     (fewer workgroups share the memory) and all of it if it is full.  Beyond one round only from 24 steps on: a
//     third round then has to pay for its fixed cost.
//   causal: only up to 256 whole tiles, where the longest of them sets the time.  The split tiles, longest
//     first, take their mean over the CUs, and `last` of a mean tile longer where they do not all start at once.
// The callers' numbers are fits to 908 launches of the forward and 1380 of the
// backward (d = 64 and 128, N = 20 .. 6000, grouped heads among them, both forms of each timed
// in turn); what the choice costs against the better form stands at the callers.  (A kernel that needs few enough
// registers for two workgroups per CU, dQ at d = 64, blurs its rounds; its fit holds that.)
struct AttnSplitCost {
  double fixed, fixed_split, slower, last;
  double least;  // steps below which the split form saves nothing: its tiles are then as many, each with a merge
};
inline bool attn_split_pays(bool causal, long long whole, long long split, int split_per_head, double steps, const AttnSplitCost& c) {
  if (steps < c.least) return false;
  double t_whole = c.fixed + steps, t_split = c.fixed_split + 0.5 * steps * c.slower;
  if (causal) {
    if (whole > 256) return false;
    if (split > 256) {
      const double mean = c.fixed_split + 0.5 * (1.0 + 1.0 / split_per_head) * 0.5 * steps * c.slower;
      const double all = ((double)split / 256.0 + c.last) * mean;
      if (all > t_split) t_split = all;
    }
  } else {
    if (whole > 65536 || (whole > 256 && steps < 24.0)) return false;  // (65536: the split grid stays in range)
    auto time = [&](long long n, double fixed, double chain) {
      const long long before = (n - 1) / 256;  // full rounds in front of the last one
      return (double)before * (fixed + chain) + fixed + chain * (c.last + (1.0 - c.last) * (double)(n - before * 256) / 256.0);
    };
    t_whole = time(whole, c.fixed, t_whole - c.fixed);
    t_split = time(split, c.fixed_split, t_split - c.fixed_split);
  }
  return t_split < t_whole;
}

// persistent bf16 forward (d = 64 or 128): workgroups that stay resident on `cus` CUs drain the tile queue
int attn_fwd_bf16_persistent_launch(const AttnParams& p, int d, int cus, hipStream_t stream);

// backward pass (bf16, head dimension 128 or 64)
struct AttnBwdParams {
  const void* q;
  const void* k;
  const void* v;
  const void* o;
  const void* dout;
  const float* lse;
  void* dq;
  void* dk;
  void* dv;
  float* ws;         // [B, Hq, 2, Npad] floats: lse * log2(e) and -delta, rows padded to whole 64-row tiles
  int B, Hq, Hkv, N;
  int T = 0;         // query tiles per head of the dQ kernel, set by the launch (128 rows each, 64 when it splits the keys)
  int Npad;          // ceil(N / 64) * 64
  int causal;
  float scale_log2;  // scale * log2(e)
  float scale;
};
int attn_bwd_launch_bf16(const AttnBwdParams& p, int d, hipStream_t stream);  // d = 128 or 64

struct AttnVariant {
  const char* name;
  int dtype;   // attn_dtype
  int d;       // head dim
  int bm;      // query rows per workgroup
  int bn;      // keys per streamed K/V tile
  int threads; // workgroup size
  int lds;     // dynamic LDS bytes
  // launches the kernel for `grid` workgroups on `stream`; returns the hipError_t as int
  int (*launch)(const AttnParams& p, int grid, hipStream_t stream);
};

// Variant tables, defined by the kernel translation units (host functions).
const AttnVariant* attn_sp_variants(int* count);   // pipelined kernel: bf16 d = 128 / 64, fp8 d = 128 (the defaults)
const AttnVariant* attn_fp8_variants(int* count);  // all products on the fp8 matrix path, P as two e4m3 terms
const AttnVariant* attn_sp_forms(int* count);      // the two forms between which the bf16 defaults choose, each by itself

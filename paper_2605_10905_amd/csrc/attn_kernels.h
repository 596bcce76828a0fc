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
// The caller's numbers are fits to 908 launches of the forward (d = 64 and 128, N = 20 .. 6000, grouped heads among them, both forms of
// each timed in turn); what the choice costs against the better form stands there.
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

// What a launch takes, us, where forms of different tiles, or workgroups that share a CU, are weighed against each other.  A
// workgroup takes P and, for each 32-row block step of its chain, a + b (k - 1) where k workgroups share the CU; the launch F beside
// them.  The numbers are the callers' fits.
struct AttnFormCost {
  double F, P, a, b;
  double t;  // equal workgroups: of a round, what the last one takes if it is nearly empty
};
inline double attn_shared_step(const AttnFormCost& c, long long n, int slots) {
  const long long rounds = (n + 255) / 256;
  return c.a + c.b * (double)((rounds < slots ? rounds : slots) - 1);
}
// n equal workgroups of `chain` steps, `slots` of them per CU: whole rounds over the CUs, the last one by what it holds
inline double attn_equal_us(const AttnFormCost& c, long long n, int slots, double chain) {
  const long long cap = 256ll * slots, rounds = (n + 255) / 256, before = (n - 1) / cap;
  const double one = c.P + chain * attn_shared_step(c, n, slots);
  if (n <= cap) return c.F + one;
  const double last = c.t + (1.0 - c.t) * (double)(n - before * cap) / (double)cap;
  return c.F + ((double)before + last) * one * slots / (double)(rounds < slots ? rounds : slots);
}
// The workgroups of a causal launch, handed out in the order of its tile map (`heaviest` steps for the first tile of a head, `less` fewer for each
// one after it; `top` is the most a tile has) to whichever place comes free first.  Tiles of equal rank in a batch are equal, and
// so are most places, which are kept as (time, how many).  A launch of very many ranks is taken as evenly spread instead.
inline double attn_causal_us(const AttnFormCost& c, const AttnTileMap& m, long long n, int slots, double heaviest, double less, double top) {
  constexpr int MAXRANKS = 256;
  const double step = attn_shared_step(c, n, slots);
  auto us = [&](int rank) {
    const double blocks = heaviest - rank * less;
    return c.P + (blocks < top ? blocks : top) * step;
  };
  if (n <= 256ll * slots) return c.F + us(0);
  if (((m.gx + m.pb - 1) / m.pb) * (long long)m.T > MAXRANKS)
    return c.F + ((double)n / (256.0 * slots) + 0.5) * 0.5 * (us(0) + us(m.T - 1));
  double free_at[MAXRANKS + 2];
  int places[MAXRANKS + 2], kinds = 1;  // earliest first
  free_at[0] = 0.0;
  places[0] = 256 * slots / m.lists;
  double end = 0.0;
  for (int first = 0; first < m.gx; first += m.pb)
    for (int rank = 0; rank < m.T; ++rank) {
      int left = (m.gx - first < m.pb ? m.gx - first : m.pb) * m.G;
      while (left > 0) {
        const int take = left < places[0] ? left : places[0];
        const double done = free_at[0] + us(rank);
        left -= take;
        places[0] -= take;
        if (done > end) end = done;
        int at = kinds;  // the new entry goes in front of this one
        while (at > 1 && free_at[at - 1] > done) --at;
        if (places[0] == 0) {  // the first entry is used up
          --at;
          for (int i = 0; i < at; ++i) {
            free_at[i] = free_at[i + 1];
            places[i] = places[i + 1];
          }
        } else {
          for (int i = kinds++; i > at; --i) {
            free_at[i] = free_at[i - 1];
            places[i] = places[i - 1];
          }
        }
        free_at[at] = done;
        places[at] = take;
      }
    }
  return c.F + end;
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
  int T = 0;         // query tiles per head of the dQ kernel, set by the launch (128 rows each, 64 when it splits the keys, 256 in wide workgroups)
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
const AttnVariant* attn_sp_forms(int* count);      // the three forms between which the bf16 defaults choose, each by itself

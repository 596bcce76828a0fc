// C-ABI entry points of the bf16 GEMM: argument checks, kernel choice, launch.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/gemm.h"
#include "gemm_kernels.h"
#include "gemm_map.h"

namespace {

bool misaligned(const void* p, uintptr_t a) { return ((uintptr_t)p & (a - 1)) != 0; }

// Tile choice: the estimated time of a launch, smallest wins.  A tile's workgroup takes
// fixed + steps * step_us microseconds (GemmTile: measured, the rates hold the LDS staging, the
// matrix work and the tile's start and end); with one workgroup per CU the launch takes whole
// rounds over the 256 CUs, with several the rounds blur (half a round is lost at the end).
// Operands and result at tb_s are the other bound, and 0.3 of the smaller of the two is not
// hidden behind the larger.  Over 72 nt shapes drawn apart from those of the fit (M 1 .. 321228, N 36 .. 63114, K 64 ..
// 15040) the choice takes 3.4 % longer on average than the fastest tile, at worst 29 % (994 x 32024 x 96: 22.3 against
// 17.3 us).  Against 256 / 128 / 64 squares by number of tiles, over 251 nt and 125 nn shapes: 1.8 x and 1.5 x faster.
double tile_cost(const GemmTile& t, int M, int N, long long K, long long splits, double bytes) {
  if (K % t.kmult != 0) return -1.0;
  const long long tiles = (long long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn) * splits;
  if (tiles * t.threads > 0xffffffffll) return -1.0;  // beyond what a launch holds
  double rounds = (double)((tiles + 255) / 256);
  if (t.per_cu > 1 && tiles >= 256ll * t.per_cu) rounds = (double)tiles / 256.0 + 0.5;
  const double work = rounds * (t.fixed_us + (double)((K + t.step - 1) / t.step) * t.step_us);
  const double mem = bytes / (t.tb_s * 1e6);
  return work > mem ? work + 0.3 * mem : mem + 0.3 * work;
}

const GemmTile* cheapest(const GemmTile* best, double* cost, const GemmTile* table, int count, int M, int N, long long K, long long splits, double bytes) {
  for (int i = 0; i < count; ++i) {
    const double c = tile_cost(table[i], M, N, K, splits, bytes);
    if (c >= 0.0 && (!best || c < *cost)) {
      best = &table[i];
      *cost = c;
    }
  }
  return best;
}

// the variant tables, concatenated
const GemmVariant* variant_at(int i) {
  if (i < 0) return nullptr;
  for (auto list : {gemm_bf16_nt_variants, gemm_wavek_nt_variants, gemm_bf16_nt_ahead_variants}) {
    int n = 0;
    const GemmVariant* const t = list(&n);
    if (i < n) return &t[i];
    i -= n;
  }
  return nullptr;
}

double gemm_bytes(int M, int N, int K) { return 2.0 * ((double)M * K + (double)N * K + (double)M * N); }

const GemmTile* choose_nt(int M, int N, int K, double* cost) {
  int n1 = 0, n2 = 0;
  const GemmTile* t1 = gemm_bf16_nt_tiles(&n1);
  const GemmTile* t2 = gemm_wavek_nt_tiles(&n2);
  const GemmTile* best = cheapest(nullptr, cost, t1, n1, M, N, K, 1, gemm_bytes(M, N, K));
  return cheapest(best, cost, t2, n2, M, N, K, 1, gemm_bytes(M, N, K));
}

const GemmTile* choose_nn(int M, int N, int K, double* cost) {
  int n1 = 0, n2 = 0;
  const GemmTile* t1 = gemm_bf16_nn_tiles(&n1);
  const GemmTile* t2 = gemm_wavek_nn_tiles(&n2);
  const GemmTile* best = cheapest(nullptr, cost, t1, n1, M, N, K, 1, gemm_bytes(M, N, K));
  return cheapest(best, cost, t2, n2, M, N, K, 1, gemm_bytes(M, N, K));
}

// Non-temporal stores of C from 96 MB on: C then does not stay in the caches and should not displace
// the operands in them.  Measured plain -> non-temporal with the tile chosen here, buffers changing from call to
// call: 442368 x 448 x 192 161.3 -> 159.9 us, 2048 x 64512 x 256 117.9 -> 102.0, 46207 x 1250 x 384 (116 MB) 77.6 -> 71.6,
// 8192 x 8192 x 1024 131.0 -> 122.7, nn 200336 x 1432 x 256 243.0 -> 220.9, 589824 x 256 x 128 97.7 -> 98.4; below the line
// 5329 x 3495 x 160 (37 MB) 18.9 -> 20.8, 300000 x 100 x 512 (60 MB) 91.1 -> 91.1, nn 2763 x 9272 x 128 (51 MB) 17.7 -> 21.1.
// (Over the same buffers again and again it gains more, 442368 x 448 x 192 to 124: half of A stays cached.)
int stream_c_pays(int M, int N) { return 2.0 * M * N >= 96e6 ? 1 : 0; }

int launch_tile(const GemmTile* t, GemmParams& p, void* stream) {
  if (!t) return ATTN_ERR_UNSUPPORTED;
  p.tiles_m = (p.M + t->bm - 1) / t->bm;
  p.tiles_n = (p.N + t->bn - 1) / t->bn;
  return t->launch(p, (hipStream_t)stream) == 0 ? ATTN_OK : ATTN_ERR_LAUNCH;
}

int run(const void* a, const void* b, void* c, int M, int N, int K, int variant, void* stream) {
  if (!a || !b || !c) return ATTN_ERR_NULL;
  if (M <= 0 || N <= 0 || K <= 0) return ATTN_ERR_SHAPE;
  if (misaligned(a, 16) || misaligned(b, 16) || misaligned(c, 16)) return ATTN_ERR_SHAPE;
  if (K % 32 != 0) return ATTN_ERR_UNSUPPORTED;
  const GemmVariant* const v = variant_at(variant);
  if (!v && variant != -1) return ATTN_ERR_UNSUPPORTED;
  // per-lane offsets inside an operand panel are 32-bit: 256 rows of K bf16
  if ((long long)K * 2 * 256 >= (1ll << 31)) return ATTN_ERR_UNSUPPORTED;
  GemmParams p;
  p.a = a; p.b = b; p.c = c;
  p.M = M; p.N = N; p.K = K;
  p.stream_c = stream_c_pays(M, N);
  if (!v) {
    double cost = 0.0;
    return launch_tile(choose_nt(M, N, K, &cost), p, stream);
  }
  if (K % v->bk != 0 || K % v->kmult != 0) return ATTN_ERR_UNSUPPORTED;
  p.tiles_m = (M + v->bm - 1) / v->bm;
  p.tiles_n = (N + v->bn - 1) / v->bn;
  if ((long long)p.tiles_m * p.tiles_n > 0x7fffffffll) return ATTN_ERR_UNSUPPORTED;
  return v->launch(p, (hipStream_t)stream) == 0 ? ATTN_OK : ATTN_ERR_LAUNCH;
}

int run_nn(const void* a, const void* b, void* c, int M, int N, int K, void* stream) {
  if (!a || !b || !c) return ATTN_ERR_NULL;
  if (M <= 0 || N <= 0 || K <= 0) return ATTN_ERR_SHAPE;
  if (misaligned(a, 16) || misaligned(b, 16) || misaligned(c, 16)) return ATTN_ERR_SHAPE;
  if (K % 32 != 0 || N % 8 != 0) return ATTN_ERR_UNSUPPORTED;
  if ((long long)K * 2 * 256 >= (1ll << 31) || (long long)N * 2 * 64 >= (1ll << 31)) return ATTN_ERR_UNSUPPORTED;
  GemmParams p;
  p.a = a; p.b = b; p.c = c;
  p.M = M; p.N = N; p.K = K;
  p.stream_c = stream_c_pays(M, N);
  double cost = 0.0;
  return launch_tile(choose_nn(M, N, K, &cost), p, stream);
}

int run_splitk(const void* a, const void* b, void* c, int M, int N, int K, int splits, float* workspace, void* stream) {
  if (!a || !b || !c || !workspace) return ATTN_ERR_NULL;
  if (M <= 0 || N <= 0 || K <= 0 || splits < 1 || splits > 64) return ATTN_ERR_SHAPE;
  if (misaligned(a, 16) || misaligned(b, 16) || misaligned(c, 16) || misaligned(workspace, 16)) return ATTN_ERR_SHAPE;
  if (K % 64 != 0) return ATTN_ERR_UNSUPPORTED;
  if ((long long)K * 2 * 256 >= (1ll << 31)) return ATTN_ERR_UNSUPPORTED;
  GemmParams p;
  p.a = a; p.b = b; p.c = c;
  p.M = M; p.N = N; p.K = K;
  // `splits` is what the workspace holds, so any smaller number may be used: the waves of the small
  // tiles split k among themselves already, and a slice more costs its partial tile twice over the
  // memory.  The same estimate as above, plus the partial tiles (written and read at 4 TB/s) and the
  // second launch (3 us), over 1, 2, 3, 4, 6, 9, ... slices and `splits` itself.  Measured, always 256 x 256
  // tiles and `splits` slices -> this: 234 x 74 x 21504 67 -> 8.1 us, 896 x 761 x 12288 72 -> 35, 84 x 3775 x 40000
  // 110 -> 79, 64 x 64 x 65536 57 -> 10; where the large tile stays, its XCD map (gemm_map.h) and the 16x16x32 kernel:
  // 2304 x 1024 x 65536 357 -> 335 -> 287 us with the sum kernel (12 us of it), 258 with operands fetched ahead.
  const int steps = K / 64;
  auto slice = [&](int s) { return ((steps + s - 1) / s) * 64; };  // whole 64-column steps, none empty
  const GemmTile large = {256, 256, 64, 1, 5.9f, 0.985f, 5.5f, gemm_bf16_nt_splitk_launch, 64};
  int nwave = 0;
  const GemmTile* const wave = gemm_wavek_nt_tiles(&nwave);
  double best_cost = 0.0;
  const GemmTile* best = choose_nt(M, N, K, &best_cost);
  int best_splits = 1;
  for (int s = 2; s <= splits; s = s == splits ? s + 1 : s + s / 2 < splits ? s + s / 2 : splits) {
    const int used = (K + slice(s) - 1) / slice(s);
    const double extra = 3.0 + 8.0 * used * M * N / 4e6;
    double cost = 0.0;
    const GemmTile* t = cheapest(nullptr, &cost, &large, 1, M, N, slice(s), used, gemm_bytes(M, N, K));
    t = cheapest(t, &cost, wave, nwave, M, N, slice(s), used, gemm_bytes(M, N, K));
    if (t && (!best || cost + extra < best_cost)) {
      best_cost = cost + extra;
      best = t;
      best_splits = s;
    }
  }
  if (best_splits == 1) {
    p.stream_c = stream_c_pays(M, N);
    return launch_tile(best, p, stream);
  }
  p.klen = slice(best_splits);
  p.splits = (K + p.klen - 1) / p.klen;
  p.partial = workspace;
  const int st = launch_tile(best, p, stream);
  if (st != ATTN_OK) return st;
  return gemm_splitk_sum_launch(p, (hipStream_t)stream) == 0 ? ATTN_OK : ATTN_ERR_LAUNCH;
}

}  // namespace

extern "C" {

int gemm_bf16_nt_splitk(const void* a, const void* b, void* c, int M, int N, int K, int splits, float* workspace, void* stream) {
  return run_splitk(a, b, c, M, N, K, splits, workspace, stream);
}

long long gemm_splitk_workspace_bytes(int M, int N, int splits) {
  if (M <= 0 || N <= 0 || splits <= 0) return 0;
  return (long long)splits * M * N * 4;
}

// Measured on the paper's large-K shapes: splitting pays when the 256 x 256 tiles leave at least half
// of the 256 CUs idle and every slice still has 2048 or more of k to amortise its prologue and the
// fp32 round trip of the partial tiles.
int gemm_splitk_plan(int M, int N, int K) {
  if (M <= 0 || N <= 0 || K <= 0 || K % 64 != 0) return 1;
  const long long tiles = (long long)((M + 255) / 256) * ((N + 255) / 256);
  if (tiles > 128) return 1;
  long long s = 256 / tiles;
  if (s > K / 2048) s = K / 2048;
  if (s > 64) s = 64;
  return s < 2 ? 1 : (int)s;
}

int gemm_bf16_nn(const void* a, const void* b, void* c, int M, int N, int K, void* stream) {
  return run_nn(a, b, c, M, N, K, stream);
}

int gemm_bf16_nt(const void* a, const void* b, void* c, int M, int N, int K, void* stream) {
  return run(a, b, c, M, N, K, -1, stream);
}

int gemm_bf16_nt_variant(const void* a, const void* b, void* c, int M, int N, int K, int variant, void* stream) {
  if (variant < 0) return ATTN_ERR_UNSUPPORTED;
  return run(a, b, c, M, N, K, variant, stream);
}

int gemm_num_variants(void) {
  int n = 0;
  while (variant_at(n)) ++n;
  return n;
}

const char* gemm_variant_name(int variant) {
  const GemmVariant* const v = variant_at(variant);
  return v ? v->name : nullptr;
}

int gemm_variant_kmult(int variant) {
  const GemmVariant* const v = variant_at(variant);
  return v ? v->kmult : 0;
}

int gemm_variant_tile(int variant) {
  const GemmVariant* const v = variant_at(variant);
  return v ? v->bm : 0;
}

int gemm_num_workgroups(int M, int N, int tile) {
  if (M <= 0 || N <= 0 || tile <= 0) return 0;
  return ((M + tile - 1) / tile) * ((N + tile - 1) / tile);
}

int gemm_tile_coord(int wg, int M, int N, int tile, int* tm, int* tn) {
  if (!tm || !tn) return ATTN_ERR_NULL;
  if (M <= 0 || N <= 0 || tile <= 0) return ATTN_ERR_SHAPE;
  const int tiles_m = (M + tile - 1) / tile, tiles_n = (N + tile - 1) / tile;
  if (wg < 0 || wg >= tiles_m * tiles_n) return ATTN_ERR_SHAPE;
  const GemmTileCoord c = gemm_tile_coord_impl(wg, tiles_m, tiles_n);
  *tm = c.tm;
  *tn = c.tn;
  return ATTN_OK;
}
}

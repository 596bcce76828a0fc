// Internal interface between the GEMM C-ABI entry points and the gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>

struct GemmParams {
  const void* a;  // bf16 [M, K]
  const void* b;  // bf16 [N, K] (nt kernels) or [K, N] (nn kernels)
  void* c;        // bf16 [M, N]
  int M, N, K;
  int tiles_m, tiles_n;
  // split-K launches only: split s of `splits` contracts k in [s * klen, min(K, (s + 1) * klen)) and
  // writes its fp32 partial tile to partial[s][M][N]; a second kernel sums the splits into c
  float* partial = nullptr;
  int splits = 1;
  int klen = 0;
  int stream_c = 0;  // non-zero: C is written with non-temporal stores (it is not read again and should not displace the operands in the L2)
};

struct GemmVariant {
  const char* name;
  int bm, bn, bk;
  int kmult;  // K must be a multiple of this (some kernels run their k-stages in pairs)
  int (*launch)(const GemmParams& p, hipStream_t stream);
};

// what gemm_bf16_nt_variant offers: every kernel that gemm_bf16_nt chooses from, and a few that it does not
const GemmVariant* gemm_bf16_nt_variants(int* count);
const GemmVariant* gemm_wavek_nt_variants(int* count);
const GemmVariant* gemm_bf16_nt_ahead_variants(int* count);  // (last, so that the others keep their numbers)
// A tile of the library's own choice (gemm_api.hip): one workgroup of it takes about
// fixed_us + ceil(K / step) * step_us, `per_cu` of them share a CU.
struct GemmTile {
  int bm, bn, step, per_cu;
  float fixed_us, step_us;
  float tb_s;  // rate at which it moves operands and result when they are the bound
  int (*launch)(const GemmParams& p, hipStream_t stream);
  int kmult = 32;  // K must be a multiple of this
  int threads = 256;
};
const GemmTile* gemm_bf16_nt_tiles(int* count);   // ring in LDS, shared by the waves of a workgroup
const GemmTile* gemm_bf16_nn_tiles(int* count);
const GemmTile* gemm_wavek_nt_tiles(int* count);  // waves split k; also writes split-K partial tiles
const GemmTile* gemm_wavek_nn_tiles(int* count);

// 256 x 256 tiles, K split over p.splits workgroups per tile (p.klen a multiple of 64), without the sum
int gemm_bf16_nt_splitk_launch(const GemmParams& p, hipStream_t stream);
// c = bf16(sum of the p.splits partial tiles)
int gemm_splitk_sum_launch(const GemmParams& p, hipStream_t stream);

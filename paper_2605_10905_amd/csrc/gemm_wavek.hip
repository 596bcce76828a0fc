// bf16 GEMM for gfx950, small outputs: the waves of a workgroup split k.
//
// The ring kernels of gemm_bf16.hip give a 64 x 64 or larger tile to a workgroup that walks the
// whole of k stage by stage behind a barrier: with few tiles most CUs idle and the launch lasts as
// long as that serial chain (33 x 4096 x 4096: 64 tiles, 128 stages, 20 us for 34 MB).  Here a
// workgroup owns a small tile and each of its WK waves contracts every WK-th chunk of k; the
// partial accumulators are added through LDS, in wave order, at the end.
//
// No operand byte is used by two waves, so every wave has a ring of its own, filled by direct-to-LDS
// loads ND chunks ahead and ordered by the wave's own load counter: no barrier until the sum.  (The
// same split with loads straight into registers moved half as much: the compiler waits for a whole
// batch of loads at every loop head, and a load instruction then covers 16 half lines instead of 8
// whole ones.)  What bounds it is the operand read, about 95 bytes per ns and CU.
//
//   nt: a chunk is 64 k, every row 128 bytes;   nn: a chunk is 32 k, the second operand's k rows
//   are gathered with the transposing LDS read.
//
// Measured, ring kernel -> this one: 33 x 4096 x 4096 20.1 -> 9.0 us, 2 x 37 x 9952 38 -> 7.6, 54 x 64 x 5696
// 22.6 -> 5.5, 300 x 300 x 16384 72 -> 17.4, 16 x 8192 x 8192 56 -> 27, nn 2 x 192 x 6016 41 -> 7.3.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "attn_device.h"
#include "gemm_kernels.h"
#include "gemm_map.h"

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

// one wave's ring of ND stages: A rows, then B rows ([K, N]: k rows), of one chunk of BK k
template <int MB, int NB, int WK, int ND, bool BKN>
struct WaveKCfg {
  static constexpr int BM = 16 * MB, BN = 16 * NB, BK = BKN ? 32 : 64, KS = BK / 32;
  static constexpr int ROWA = BK * 2, NCHA = ROWA / 16;
  static constexpr int ROWB = BKN ? BN * 2 : ROWA, NCHB = ROWB / 16;
  static constexpr int TILEA = BM * ROWA, TILEB = (BKN ? BK : BN) * ROWB, STAGEB = TILEA + TILEB;
  static constexpr int NLA = TILEA / 1024, NLB = TILEB / 1024, LPS = NLA + NLB;  // loads per stage (64 lanes x 16 bytes each)
  static constexpr int ENTRIES = MB * NB * 64;                                   // f32x4 pieces of the tile
  static constexpr int RING = WK * ND * STAGEB, RED = WK * ENTRIES * 16;
  static constexpr int LDS_BYTES = RING > RED ? RING : RED;
  static_assert(LDS_BYTES <= 160 * 1024 && (ND - 1) * LPS <= 63, "ring");
};

// chunk swizzle of a [K, N] stage: the transposing read serves two lane groups at a time, k rows
// r .. r+3 and r+8 .. r+11 of one 32-byte column piece; the XOR spreads them over the 256-byte bank line
template <int NB>
__device__ __forceinline__ constexpr int swz_kn(int r) {
  return (NB == 8 ? (r & 3) | (((r >> 3) & 1) << 2) : NB == 4 ? ((r >> 1) & 1) | (((r >> 3) & 1) << 1) : (r >> 3) & 1) << 1;
}

template <int MB, int NB, int WK, int ND, bool BKN, bool PARTIAL>
__global__ void __launch_bounds__(WK * 64) gemm_wavek_kernel(const GemmParams p) {
  using C = WaveKCfg<MB, NB, WK, ND, BKN>;
  constexpr int BM = C::BM, BN = C::BN, BK = C::BK, KS = C::KS, ENTRIES = C::ENTRIES, LPS = C::LPS, STAGEB = C::STAGEB;
  static_assert(!BKN || NB == 2 || NB == 4 || NB == 8, "[K, N] operand: k rows of 64, 128 or 256 bytes");
  __shared__ __attribute__((aligned(1024))) char smem_raw[C::LDS_BYTES];
  LDS_AS char* const smem = (LDS_AS char*)smem_raw;

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int lj = lane & 15, g = lane >> 4;

  int split = 0;
  const GemmTileCoord tc = PARTIAL ? gemm_tile_coord_split(blockIdx.x, p.tiles_m, p.tiles_n, p.splits, &split)
                                   : gemm_tile_coord_impl(blockIdx.x, p.tiles_m, p.tiles_n);
  const int m0 = tc.tm * BM, n0 = tc.tn * BN;
  const int M = p.M, N = p.N, K = p.K;
  const int kbeg = PARTIAL ? split * p.klen : 0;
  const int kcnt = PARTIAL ? min(p.klen, K - kbeg) : K;
  const size_t rowbytes = (size_t)K * 2;

  // load `it` of a stage moves 16-byte chunks it * 64 + lane of A's rows, then of B's; rows and columns
  // past the matrix re-read its last ones (their sums are not stored).  kc: the chunk's k offset in
  // bytes (what a half stage must not read beyond)
  const char* const a0 = (const char*)p.a + (size_t)m0 * rowbytes + (size_t)kbeg * 2;
  const char* const b0 = BKN ? (const char*)p.b + ((size_t)kbeg * N + n0) * 2 : (const char*)p.b + (size_t)n0 * rowbytes + (size_t)kbeg * 2;
  const size_t b_step = BKN ? (size_t)BK * N * 2 : (size_t)BK * 2;
  uint32_t off[LPS];
#pragma unroll
  for (int it = 0; it < LPS; ++it) {
    const bool is_a = it < C::NLA;
    const int s = (is_a ? it : it - C::NLA) * 64 + lane;
    if (is_a || !BKN) {
      const int r = s / C::NCHA, c = (s % C::NCHA) ^ attn_swz_k<C::ROWA>(r);
      const int row = is_a ? min(m0 + r, M - 1) - m0 : min(n0 + r, N - 1) - n0;
      off[it] = (uint32_t)row * (uint32_t)rowbytes + c * 16;
    } else {
      const int r = s / C::NCHB, c = (s % C::NCHB) ^ swz_kn<NB>(r);
      off[it] = (uint32_t)r * (uint32_t)(N * 2) + (min(n0 + c * 8, N - 8) - n0) * 2;
    }
  }
  const uint32_t ring = (uint32_t)(uintptr_t)smem + w * (ND * STAGEB);
  auto issue = [&](int c, int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int it = 0; it < LPS; ++it) {
      const char* const base = it < C::NLA ? a0 + (size_t)c * (BK * 2) : b0 + (size_t)c * b_step;
      attn_lds_dma16(base, off[it], ring + slot * STAGEB + it * 1024);
    }
  };

  // fragment addresses in slot 0: 16-row block 0, k-step s
  uint32_t ra[KS], rb[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    ra[s] = w * (ND * STAGEB) + lj * C::ROWA + (((4 * s + g) ^ attn_swz_k<C::ROWA>(lj)) << 4);
    rb[s] = ra[s] + C::TILEA;
  }
  uint32_t tb[NB][2];  // [K, N]: read e of a fragment takes k = 8 g + 4 e + (0..3), lane s16 four columns of one of these rows
  if constexpr (BKN) {
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int r = 8 * g + 4 * e + (lj >> 2);
        tb[i][e] = w * (ND * STAGEB) + C::TILEA + r * C::ROWB + (((2 * i + ((lj & 3) >> 1)) ^ swz_kn<NB>(r)) << 4) + ((lj & 1) << 3);
      }
  }

  f32x4 acc[NB][MB];  // [n block][m block]: rows of the accumulator are n (4 g + r), its column is m (lj)
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < MB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  u32x4 fa[MB][KS], fb[NB][KS];
  auto read_stage = [&](int slot) __attribute__((always_inline)) {
    const int base = slot * STAGEB;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
#pragma unroll
      for (int i = 0; i < MB; ++i) fa[i][s] = *(LDS_AS u32x4*)(smem + ra[s] + base + i * 16 * C::ROWA);
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        if constexpr (BKN) {
          const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(smem + tb[i][0] + base));
          const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(smem + tb[i][1] + base));
          s16x8 av;
          av[0] = v0[0]; av[1] = v0[1]; av[2] = v0[2]; av[3] = v0[3];
          av[4] = v1[0]; av[5] = v1[1]; av[6] = v1[2]; av[7] = v1[3];
          fb[i][s] = __builtin_bit_cast(u32x4, av);
        } else {
          fb[i][s] = *(LDS_AS u32x4*)(smem + rb[s] + base + i * 16 * C::ROWA);
        }
      }
    }
  };
  auto contract = [&](auto steps) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < decltype(steps)::value; ++s)
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fb[i][s]), __builtin_bit_cast(bf16x8, fa[j][s]), acc[i][j], 0, 0, 0);
  };

  // whole chunks w, w + WK, ...: no other wave touches this wave's ring, so its own load counter is
  // all that orders it; a slot is refilled once its fragments are in registers
  const int nchunk = kcnt / BK;
  const int n = nchunk > w ? (nchunk - w + WK - 1) / WK : 0;
#pragma unroll
  for (int d = 0; d < ND; ++d)
    if (d < n) issue(w + d * WK, d);
  int slot = 0;
  for (int i = 0; i < n; ++i) {
    if (i + ND <= n) ATTN_WAIT_VMCNT((ND - 1) * LPS);
    else ATTN_WAIT_VMCNT(0);
    __builtin_amdgcn_sched_barrier(0);
    read_stage(slot);
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
    if (i + ND < n) issue(w + (i + ND) * WK, slot);
    contract(std::integral_constant<int, KS>{});
    slot = slot == ND - 1 ? 0 : slot + 1;
  }
  if (KS == 2 && (kcnt & 32) && w == nchunk % WK) {
    // the last 32 k: the upper half of the rows' 128 bytes re-reads the lower one and is not contracted
#pragma unroll
    for (int it = 0; it < LPS; ++it) {
      const int s = (it < C::NLA ? it : it - C::NLA) * 64 + lane;
      const int c = (s % C::NCHA) ^ attn_swz_k<C::ROWA>(s / C::NCHA);
      attn_lds_dma16((it < C::NLA ? a0 : b0) + (size_t)nchunk * (BK * 2), off[it] - (c >= 4 ? 64 : 0), ring + it * 1024);
    }
    ATTN_WAIT_VMCNT(0);
    __builtin_amdgcn_sched_barrier(0);
    read_stage(0);
    contract(std::integral_constant<int, 1>{});
  }

  __syncthreads();  // the rings are done with
  LDS_AS f32x4* const part = (LDS_AS f32x4*)smem;
  // ---- sum over the waves, in wave order; a piece is four consecutive columns of one row
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int j = 0; j < MB; ++j) part[w * ENTRIES + (a * MB + j) * 64 + lane] = acc[a][j];
  __syncthreads();
  for (int e = tid; e < ENTRIES; e += WK * 64) {
    f32x4 v = part[e];
#pragma unroll
    for (int s = 1; s < WK; ++s) v += part[s * ENTRIES + e];
    const int a = e / (MB * 64), j = (e / 64) % MB;  // (lane of the piece = lane of this thread)
    const int m = m0 + 16 * j + lj;
    const int nc = n0 + 16 * a + 4 * g;
    if (m < M) {
      if constexpr (PARTIAL) {
        float* const dst = p.partial + ((size_t)split * M + m) * N + nc;
        if ((N & 3) == 0 && nc + 4 <= N) {
          *(f32x4*)dst = v;
        } else {
#pragma unroll
          for (int t = 0; t < 4; ++t)
            if (nc + t < N) dst[t] = v[t];
        }
      } else {
        __bf16* const dst = (__bf16*)p.c + (size_t)m * N + nc;
        if ((N & 3) == 0 && nc + 4 <= N) {
          *(u32x2*)dst = u32x2{attn_pack_bf16(v[0], v[1]), attn_pack_bf16(v[2], v[3])};
        } else {
#pragma unroll
          for (int t = 0; t < 4; ++t)
            if (nc + t < N) dst[t] = (__bf16)v[t];
        }
      }
    }
  }
}

template <int MB, int NB, int WK, int ND, bool BKN = false>
int launch(const GemmParams& p, hipStream_t stream) {
  const dim3 grid(p.tiles_m * p.tiles_n * p.splits), block(WK * 64);
  if (p.partial) {
    if constexpr (!BKN) hipLaunchKernelGGL((gemm_wavek_kernel<MB, NB, WK, ND, false, true>), grid, block, 0, stream, p);
  } else {
    hipLaunchKernelGGL((gemm_wavek_kernel<MB, NB, WK, ND, BKN, false>), grid, block, 0, stream, p);
  }
  return (int)hipGetLastError();
}

}  // namespace

const GemmTile* gemm_wavek_nt_tiles(int* count) {
  static const GemmTile table[] = {
      {16, 16, 256, 2, 0.4f, 0.16f, 5.5f, launch<1, 1, 4, 4>},
      {32, 32, 256, 2, 0.5f, 0.32f, 5.5f, launch<2, 2, 4, 2>},
      {64, 16, 512, 1, 1.0f, 0.78f, 5.5f, launch<4, 1, 8, 2>, 32, 512},
      {32, 64, 256, 1, 1.5f, 0.52f, 5.5f, launch<2, 4, 4, 3>},
      {64, 64, 256, 1, 2.2f, 0.68f, 5.5f, launch<4, 4, 4, 2>},
  };
  *count = (int)(sizeof(table) / sizeof(table[0]));
  return table;
}

const GemmVariant* gemm_wavek_nt_variants(int* count) {
  static const GemmVariant table[] = {
      {"bf16 nt 16x16 waves split k", 16, 16, 32, 32, launch<1, 1, 4, 4>},
      {"bf16 nt 32x32 waves split k", 32, 32, 32, 32, launch<2, 2, 4, 2>},
      {"bf16 nt 64x16 waves split k", 64, 16, 32, 32, launch<4, 1, 8, 2>},
      {"bf16 nt 32x64 waves split k", 32, 64, 32, 32, launch<2, 4, 4, 3>},
      {"bf16 nt 64x64 waves split k", 64, 64, 32, 32, launch<4, 4, 4, 2>},
  };
  *count = (int)(sizeof(table) / sizeof(table[0]));
  return table;
}

const GemmTile* gemm_wavek_nn_tiles(int* count) {
  static const GemmTile table[] = {
      {16, 32, 256, 1, 0.8f, 0.39f, 4.8f, launch<1, 2, 8, 5, true>, 32, 512},
      {32, 64, 256, 1, 1.3f, 0.50f, 4.8f, launch<2, 4, 8, 3, true>, 32, 512},
      {64, 32, 256, 1, 1.1f, 0.60f, 4.8f, launch<4, 2, 8, 3, true>, 32, 512},
  };
  *count = (int)(sizeof(table) / sizeof(table[0]));
  return table;
}

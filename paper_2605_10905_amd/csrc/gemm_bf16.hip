// bf16 GEMM for gfx950:  C[M,N] = A[M,K] * B[N,K]^T, fp32 accumulation, bf16 output.
//
// The paper's GEMM (section 6.1, GEMM paragraph; section 6.3 and appendix A for the MI350
// shapes) is a producer/consumer pipeline: loader roles stage operand tiles in swizzled shared
// memory through a ring of buffers, tensor-core roles consume them.  The gfx950 form kept here:
//
//   * a workgroup of 4 waves owns a 256 x 256 tile of C, each wave a 128 x 128 quarter: 16
//     accumulators of the 32x32x16 MFMA = 256 registers, which the MFMA reads and writes in
//     place (one wave per SIMD, the whole 512-register file).  Every operand fragment read from
//     LDS feeds four MFMAs, half the LDS bytes per MFMA of a 2-waves-per-SIMD tiling;
//   * operand tiles (256 rows x BK of A and of B) travel HBM/L2 -> LDS by direct-to-LDS loads
//     into a ring of NSTAGE slots, NSTAGE-1 stages ahead, one workgroup barrier per stage.  Every
//     wave issues its share of the loads itself: on CDNA a wave that only loads would idle a
//     SIMD, and the loads cost one issue slot each;
//   * the product is taken transposed (MFMA A operand = rows of B, B operand = rows of A), so a
//     lane owns one row m of C and, after one exchange between the lane halves, 8 consecutive n;
//     the finished tile is staged in LDS and stored along C's rows (gemm_store_staged);
//   * 16-byte chunks of a tile row are XOR-swizzled so that the 16 lanes the LDS serves together
//     hit 16 different bank groups;
//   * tiles are ordered for L2 reuse inside an XCD (gemm_map.h).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "attn_device.h"
#include "gemm_kernels.h"
#include "gemm_map.h"

// One 16-byte piece of C: plain, or non-temporal when the launch streams C (GemmParams::stream_c).
// (Written as an assembly statement: the compiler merges a plain and a non-temporal store behind a
// run-time condition into one plain store.  What it stores has been read from LDS before, and nothing reads C
// afterwards; only the elements at the row ends are stored behind it.)
#define GEMM_STORE_C(val, ptr)                                                                          \
  do {                                                                                                  \
    if (p.stream_c) asm volatile("global_store_dwordx4 %0, %1, off nt" ::"v"(ptr), "v"(val) : "memory"); \
    else *(ptr) = (val);                                                                                \
  } while (0)

namespace {

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  bf16x2 t;
  t[0] = (__bf16)a;
  t[1] = (__bf16)b;
  return __builtin_bit_cast(uint32_t, t);
}

// The last step of every tile: the finished bf16 tile lies row-major in LDS (row pitch BN * 2 + 16
// bytes) and goes to C in 16-byte pieces at 16-byte aligned addresses, consecutive lanes on
// consecutive pieces of a row.  The accumulator layout gives a lane 8 columns of a row of its own,
// i.e. a store instruction that touches 32 rows with 32 bytes each, and with N not a multiple of 8
// even that splits into 2-byte stores because the rows start at any multiple of 2 bytes.  Here the
// odd start costs a shift: the piece that begins s = (row start mod 8) elements earlier is put
// together from five LDS words by a funnel shift, and only the up to seven elements in front of the
// first and behind the last whole piece of a row are stored one by one.  Bound by memory writes for
// short contractions; measured, stores from the accumulator layout -> staged: 442368 x 448 x 192
// 165.6 -> 145.9 us (3.4 -> 3.9 TB/s), 5329 x 3495 x 160 79.5 -> 26.2 us, 27854 x 4910 x 960 457 -> 303 us,
// 794 x 58579 x 4576 601 -> 485 us, 8192 x 8192 x 4096 unchanged (457 / 458 us).
template <int BM, int BN>
__device__ __forceinline__ void gemm_store_staged(LDS_AS const char* tile, const GemmParams& p, int m0, int n0, int tid) {
  constexpr int PITCH = BN * 2 + 16, CPR = BN / 8, RPI = 256 / CPR;
  static_assert(256 % CPR == 0 && BM % RPI == 0, "whole rows per pass");
  const int rows = min(BM, p.M - m0), nv = min(BN, p.N - n0);
  const int c = tid % CPR, r0 = tid / CPR;
  __bf16* const ctile = (__bf16*)p.c + (size_t)m0 * p.N + n0;
  if ((p.N & 7) == 0) {
#pragma unroll 8
    for (int i = 0; i < BM / RPI; ++i) {
      const int r = i * RPI + r0;
      if (r < rows && c * 8 < nv) {
        const u32x4 out = *(LDS_AS const u32x4*)(tile + r * PITCH + c * 16);
        GEMM_STORE_C(out, (u32x4*)(ctile + (size_t)r * p.N + c * 8));
      }
    }
    return;
  }
#pragma unroll 4
  for (int i = 0; i < BM / RPI; ++i) {
    const int r = i * RPI + r0;
    const int s = (int)(((size_t)(m0 + r) * p.N + n0) & 7);
    const int e = 8 * (c + (s ? 1 : 0)) - s;  // first element of this lane's piece
    if (r < rows && e + 8 <= nv) {
      LDS_AS const uint32_t* const w = (LDS_AS const uint32_t*)(tile + r * PITCH) + (e >> 1);
      uint32_t d[5];
#pragma unroll
      for (int j = 0; j < 5; ++j) d[j] = w[j];  // (the fifth word of a row's last piece is row padding)
      const uint32_t sh = (e & 1) * 16;
      u32x4 out;
#pragma unroll
      for (int j = 0; j < 4; ++j) out[j] = __builtin_amdgcn_alignbit(d[j + 1], d[j], sh);
      GEMM_STORE_C(out, (u32x4*)(ctile + (size_t)r * p.N + e));
    }
  }
  // row ends: eight lanes for the elements in front of the first whole piece, eight for those behind the last
  const int j = tid & 15;
#pragma unroll 4
  for (int i = 0; i < BM / 16; ++i) {
    const int r = i * 16 + (tid >> 4);
    const int s = (int)(((size_t)(m0 + r) * p.N + n0) & 7);
    const int head = min((8 - s) & 7, nv);
    const int e = j < 8 ? j : head + ((nv - head) & ~7) + (j - 8);
    if (r < rows && e < (j < 8 ? head : nv)) ((uint16_t*)ctile)[(size_t)r * p.N + e] = *(LDS_AS const uint16_t*)(tile + r * PITCH + e * 2);
  }
}

// WM x WN 32x32 blocks per wave, 2 x 2 waves: the workgroup tile is 64 WM x 64 WN.
template <int WM, int WN, int BK, int NSTAGE>
struct GemmCfg {
  static constexpr int BM = 64 * WM, BN = 64 * WN, NT = 256;
  static constexpr int ROWB = BK * 2, NCH = ROWB / 16;
  static constexpr int TILEA = BM * ROWB, TILEB_ = BN * ROWB;
  static constexpr int STAGEB = TILEA + TILEB_;  // A tile then B tile
  static constexpr int NLDA = BM * NCH / NT, NLDB = BN * NCH / NT;  // direct-to-LDS loads per thread and stage
  static constexpr int LPS = NLDA + NLDB;
  static constexpr int NKK = BK / 16;
  static constexpr int LPP = (LPS + NKK - 1) / NKK;  // loads issued per k-step, at most
  static constexpr int PITCH = BN * 2 + 16;  // bytes per row of the finished tile staged in LDS (gemm_store_staged)
  static constexpr int LDS_BYTES = NSTAGE * STAGEB > BM * PITCH ? NSTAGE * STAGEB : BM * PITCH;
  static_assert(LDS_BYTES <= 160 * 1024, "ring does not fit the LDS");
  static_assert((NSTAGE - 1) * LPS <= 63, "vmcnt field");
  static_assert(NSTAGE >= 2 && NKK % 2 == 0 && NLDA >= 1 && NLDB >= 1, "pipeline shape");
};

// BKN: the second operand is stored [K, N] (row-major, N contiguous) instead of [N, K].  Its tile is
// then BK rows of BN columns in LDS, and the MFMA operand that needs 8 consecutive k per lane is
// gathered with the transposing LDS read, exactly as the attention kernels read V.
template <int WM, int WN, int BK, int NSTAGE, int MINW, bool BKN>
__global__ void __launch_bounds__(256, MINW) gemm_bf16_kernel(const GemmParams p) {
  using C = GemmCfg<WM, WN, BK, NSTAGE>;
  constexpr int ROWBB = C::BN * 2, NCHB = ROWBB / 16;  // [K,N] layout: bytes and 16-byte chunks per tile row
  // the four k rows that the transposing read takes together land in different 64-byte groups of the
  // 256-byte bank line (128-byte rows: two rows share a line)
  auto swz_b = [](int r) __attribute__((always_inline)) { return NCHB >= 16 ? (r & 3) << 2 : ((r >> 1) & 1) << 2; };
  constexpr int ROWB = C::ROWB, NCH = C::NCH, TILEA = C::TILEA, STAGEB = C::STAGEB, NKK = C::NKK;
  constexpr int NLDA = C::NLDA, NLDB = C::NLDB, LPS = C::LPS, LPP = C::LPP;

  __shared__ __attribute__((aligned(1024))) char smem_raw[C::LDS_BYTES];
  LDS_AS char* const smem = (LDS_AS char*)smem_raw;

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int li = lane & 31, h = lane >> 5;
  const int wm = w >> 1, wn = w & 1;

  const GemmTileCoord tc = gemm_tile_coord_impl(blockIdx.x, p.tiles_m, p.tiles_n);
  const int m0 = tc.tm * C::BM, n0 = tc.tn * C::BN;
  const int M = p.M, N = p.N, K = p.K;
  const size_t rowbytes = (size_t)K * 2;

  // ---- producer role: chunk s = it * 256 + tid of a tile is (row s / NCH, LDS chunk s % NCH) and
  // holds the row's chunk (s % NCH) ^ swizzle(row); rows past the matrix re-read its last row
  uint32_t g_off[LPS];
#pragma unroll
  for (int it = 0; it < LPS; ++it) {
    const bool is_a = it < NLDA;
    const int s = (is_a ? it : it - NLDA) * C::NT + tid;
    if (is_a || !BKN) {
      const int r = s / NCH, c = (s % NCH) ^ attn_swz_k<ROWB>(r);
      const int row = is_a ? min(m0 + r, M - 1) - m0 : min(n0 + r, N - 1) - n0;
      g_off[it] = (uint32_t)row * (uint32_t)rowbytes + c * 16;
    } else {
      // [K,N] tile: k row r, LDS chunk s % NCHB holds the row's chunk XOR swz_b(r); columns past N re-read
      // the row's last 8 (N is a multiple of 8)
      const int r = s / NCHB, c = (s % NCHB) ^ swz_b(r);
      const int col = min(n0 + c * 8, N - 8) - n0;
      g_off[it] = (uint32_t)r * (uint32_t)(N * 2) + col * 2;
    }
  }
  const char* const a_tile = (const char*)p.a + (size_t)m0 * rowbytes;
  const char* const b_tile = BKN ? (const char*)p.b + (size_t)n0 * 2 : (const char*)p.b + (size_t)n0 * rowbytes;
  const size_t b_step = BKN ? (size_t)BK * N * 2 : (size_t)ROWB;  // bytes between consecutive k-stages of the second operand
  const uint32_t lds_wave = (uint32_t)(uintptr_t)smem + w * 1024;
  // load `it` (0 .. LPS-1) of k-stage ks into ring slot `slot`
  auto issue_load = [&](int ks, int slot, int it) __attribute__((always_inline)) {
    if (it < NLDA) attn_lds_dma16(a_tile + (size_t)ks * ROWB, g_off[it], lds_wave + slot * STAGEB + it * C::NT * 16);
    else attn_lds_dma16(b_tile + (size_t)ks * b_step, g_off[it], lds_wave + slot * STAGEB + TILEA + (it - NLDA) * C::NT * 16);
  };

  // K may leave half a stage of 64 (TAIL): the upper half of its rows' 128 bytes re-reads the lower one
  // and is not contracted
  constexpr bool TAIL = BK == 64 && !BKN;
  const int nfull = K / BK;                      // whole stages
  const int nk = TAIL ? (K + BK - 1) / BK : nfull;
  auto issue_any = [&](int ks, int slot, int it) __attribute__((always_inline)) {
    if (TAIL && ks == nfull) {
      const int s = (it < NLDA ? it : it - NLDA) * C::NT + tid;
      const int c = (s % NCH) ^ attn_swz_k<ROWB>(s / NCH);
      attn_lds_dma16((it < NLDA ? a_tile : b_tile) + (size_t)ks * ROWB, g_off[it] - (c >= 4 ? 64 : 0),
                     lds_wave + slot * STAGEB + (it < NLDA ? it * C::NT * 16 : TILEA + (it - NLDA) * C::NT * 16));
    } else {
      issue_load(ks, slot, it);
    }
  };
#pragma unroll
  for (int s = 0; s < NSTAGE; ++s)
    if (s < nk) {
#pragma unroll
      for (int it = 0; it < LPS; ++it) issue_any(s, s, it);
    }

  // ---- consumer role: fragment addresses inside a stage (row block 0 of this wave's quarter)
  uint32_t ra[NKK], rb[NKK];
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) {
    const int rowa = wm * 32 * WM + li, rowb = wn * 32 * WN + li;
    ra[kk] = rowa * ROWB + (((2 * kk + h) ^ attn_swz_k<ROWB>(rowa)) << 4);
    rb[kk] = TILEA + rowb * ROWB + (((2 * kk + h) ^ attn_swz_k<ROWB>(rowb)) << 4);
  }
  // [K,N] layout: in a group of 16 lanes, lane s reads four columns of k row s / 4 and the hardware
  // hands lane t the four k of column t; read e of a fragment takes k = 8 h + 4 e + (0..3) of the k-step
  uint32_t tb[WN][2];
  {
    const int s16 = lane & 15, chalf = (lane >> 4) & 1;
#pragma unroll
    for (int nb = 0; nb < WN; ++nb)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int krow = 8 * h + 4 * e + (s16 >> 2);
        const int chunk = (wn * 32 * WN + nb * 32) / 8 + chalf * 2 + ((s16 & 3) >> 1);
        tb[nb][e] = TILEA + krow * ROWBB + ((chunk ^ swz_b(krow)) << 4) + ((s16 & 1) << 3);
      }
  }

  f32x16 acc[WN][WM];  // [n block][m block]: rows of the accumulator are n, its column is m
#pragma unroll
  for (int nb = 0; nb < WN; ++nb)
#pragma unroll
    for (int mb = 0; mb < WM; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[nb][mb][r] = 0.f;

  // Software pipeline inside the wave: the fragments of k-step kk+1 are read while the MFMAs of
  // k-step kk run.  The stage boundary (all fragments of stage ks are in registers: wait for
  // stage ks+1, barrier, first fragments of stage ks+1) sits in front of the MFMAs of a stage's
  // last k-step, so the matrix pipe has work queued across it; the slot of stage ks is free from
  // that barrier on and is refilled with stage ks+NSTAGE, LPP loads per k-step, over the k-steps
  // up to the next barrier.
  bf16x8 fa[2][WM], fb[2][WN];
  auto read_frags = [&](int buf, int base, int kk) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < WM; ++i) fa[buf][i] = *(LDS_AS bf16x8*)(smem + ra[kk] + base + i * 32 * ROWB);
    if constexpr (!BKN) {
#pragma unroll
      for (int i = 0; i < WN; ++i) fb[buf][i] = *(LDS_AS bf16x8*)(smem + rb[kk] + base + i * 32 * ROWB);
    } else {
#pragma unroll
      for (int i = 0; i < WN; ++i) {
        const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(smem + tb[i][0] + base + kk * 16 * ROWBB));
        const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(smem + tb[i][1] + base + kk * 16 * ROWBB));
        s16x8 av;
        av[0] = v0[0]; av[1] = v0[1]; av[2] = v0[2]; av[3] = v0[3];
        av[4] = v1[0]; av[5] = v1[1]; av[6] = v1[2]; av[7] = v1[3];
        fb[buf][i] = __builtin_bit_cast(bf16x8, av);
      }
    }
  };
  auto mfmas = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int nb = 0; nb < WN; ++nb)
#pragma unroll
      for (int mb = 0; mb < WM; ++mb)
        acc[nb][mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[buf][nb], fa[buf][mb], acc[nb][mb], 0, 0, 0);
  };
  // spread the WM + WN LDS reads of a k-step over its WM * WN MFMAs
  auto interleave = [&]() __attribute__((always_inline)) {
    constexpr int NR = WM + (BKN ? 2 * WN : WN), NM = WM * WN;
    constexpr int PER = NM / NR > 0 ? NM / NR : 1;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, PER, 0);
    }
  };

  if (NSTAGE <= nk) ATTN_WAIT_VMCNT((NSTAGE - 1) * LPS);
  else ATTN_WAIT_VMCNT(0);
  attn_wg_barrier();
  read_frags(0, 0, 0);

  // one k-stage; STEADY: every load and the next stage exist (no checks)
  auto stage = [&](int ks, int slot, auto steady) __attribute__((always_inline)) {
    constexpr bool STEADY = decltype(steady)::value;
    const int base = slot * STAGEB;
    const int nslot = slot == NSTAGE - 1 ? 0 : slot + 1;
    const int pslot = slot == 0 ? NSTAGE - 1 : slot - 1;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      const int cur = kk & 1, nxt = cur ^ 1;
      if (kk + 1 < NKK) {
        read_frags(nxt, base, kk + 1);
        if (STEADY || (ks >= 1 && ks - 1 + NSTAGE < nk)) {
#pragma unroll
          for (int i = 0; i < LPP; ++i)
            if ((kk + 1) * LPP + i < LPS) {
              if constexpr (STEADY) issue_load(ks - 1 + NSTAGE, pslot, (kk + 1) * LPP + i);
              else issue_any(ks - 1 + NSTAGE, pslot, (kk + 1) * LPP + i);
            }
        }
      } else if (STEADY || ks + 1 < nk) {
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wave's reads of the slot about to be refilled are done
        if (STEADY || ks + NSTAGE - 1 < nk) ATTN_WAIT_VMCNT((NSTAGE - 2) * LPS);
        else ATTN_WAIT_VMCNT(0);
        attn_wg_barrier();
        read_frags(nxt, nslot * STAGEB, 0);
        if (STEADY || ks + NSTAGE < nk) {
#pragma unroll
          for (int i = 0; i < LPP; ++i) {
            if constexpr (STEADY) issue_load(ks + NSTAGE, slot, i);
            else issue_any(ks + NSTAGE, slot, i);
          }
        }
      }
      if (STEADY || !TAIL || kk < NKK / 2 || ks < nfull) {
        mfmas(cur);
        interleave();
      }
    }
  };

  int slot = 0, ks = 0;
  if (nk > 0) {
    stage(0, 0, std::false_type{});
    ks = 1;
    slot = NSTAGE > 1 ? 1 : 0;
  }
  for (; ks + NSTAGE < nfull; ++ks) {  // (what a steady stage requests is a whole stage)
    stage(ks, slot, std::true_type{});
    slot = slot == NSTAGE - 1 ? 0 : slot + 1;
  }
  for (; ks < nk; ++ks) {
    stage(ks, slot, std::false_type{});
    slot = slot == NSTAGE - 1 ? 0 : slot + 1;
  }

  // ---- epilogue: lane (li, h) holds, for row m, the columns n = 32 nb + 8 a + 4 h + (0..3); the tile goes
  // to LDS first and from there to C
  __syncthreads();  // no wave reads the ring any more
#pragma unroll
  for (int mb = 0; mb < WM; ++mb) {
    const uint32_t row = (wm * 32 * WM + mb * 32 + li) * C::PITCH + (wn * 32 * WN + h * 8) * 2;
#pragma unroll
    for (int nb = 0; nb < WN; ++nb)
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        uint32_t x[2], y[2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          const uint32_t tx = pack_bf16(acc[nb][mb][(2 * a) * 4 + 2 * r], acc[nb][mb][(2 * a) * 4 + 2 * r + 1]);
          const uint32_t ty = pack_bf16(acc[nb][mb][(2 * a + 1) * 4 + 2 * r], acc[nb][mb][(2 * a + 1) * 4 + 2 * r + 1]);
          auto sw = __builtin_amdgcn_permlane32_swap(tx, ty, false, false);
          x[r] = sw[0];
          y[r] = sw[1];
        }
        *(LDS_AS u32x4*)(smem + row + (nb * 32 + a * 16) * 2) = u32x4{x[0], x[1], y[0], y[1]};  // this lane's 8 consecutive columns
      }
  }
  __syncthreads();
  gemm_store_staged<C::BM, C::BN>(smem, p, m0, n0, tid);
}

// The 256 x 256 tile on the 16x16x32 MFMA: each wave's 128 x 128 quarter is 8 x 8 blocks of 16 x 16
// (64 accumulators of 4 registers), a k-step is 32 wide, a fragment (16 rows x 32 k: 16 bytes per
// lane, lane (j, g) = row j, k 8g .. 8g+7) feeds eight MFMAs.  It is what large outputs run on where K is
// a multiple of 64: stages of 64 k, so that a load covers whole 128-byte lines (half the L2 requests
// of 32-wide stages), in two slots.  Bound by the board's power limit, then by the matrix pipe; the
// 32x32x16 kernel with four 32-wide stages -> this one, us, one run of the same buffers: 8192 x 8192 x 1024 134 -> 119,
// x 4096 427 -> 370, x 8192 822 -> 702, x 16384 1866 -> 1530, 4096^3 108.6 -> 94, 16384 x 4096 x 2048 229 -> 200; with changing
// buffers, on other boxes: x 4096 400 - 409 (1345 - 1374 TFLOP/s), x 8192 764, x 16384 1627, 4096^3 99, 16384 x 4096 x 2048 210.
typedef __attribute__((ext_vector_type(4))) float f32x4;

// SPLITK: the grid holds p.splits workgroups per tile; workgroup (split, tile) contracts its slice
// of k and stores the fp32 accumulators to p.partial instead of rounding them into c.
// AHEAD: operands are fetched into the L2 a few stages before they are requested.
template <int BK, int NSTAGE, bool SPLITK, bool AHEAD>
__global__ void __launch_bounds__(256, 1) gemm_bf16_nt_m16_kernel(const GemmParams p) {
  using C = GemmCfg<4, 4, BK, NSTAGE>;
  constexpr int ROWB = C::ROWB, NCH = C::NCH, TILEA = C::TILEA, STAGEB = C::STAGEB;
  constexpr int NLDA = C::NLDA, LPS = C::LPS;
  constexpr int NPH = BK / 32;       // k-steps per stage
  static_assert(BK % 32 == 0 && LPS % (8 * NPH) == 0, "k-step of 32, whole loads per row");

  __shared__ __attribute__((aligned(1024))) char smem_raw[C::LDS_BYTES];
  LDS_AS char* const smem = (LDS_AS char*)smem_raw;

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int lj = lane & 15, g = lane >> 4;
  const int wm = w >> 1, wn = w & 1;

  int split = 0;
  const GemmTileCoord tc = SPLITK ? gemm_tile_coord_split(blockIdx.x, p.tiles_m, p.tiles_n, p.splits, &split)
                                  : gemm_tile_coord_impl(blockIdx.x, p.tiles_m, p.tiles_n);
  const int m0 = tc.tm * C::BM, n0 = tc.tn * C::BN;
  const int M = p.M, N = p.N, K = p.K;
  const size_t rowbytes = (size_t)K * 2;
  const int kbeg = SPLITK ? split * p.klen : 0;            // this workgroup's slice of k
  const int kcnt = SPLITK ? min(p.klen, K - kbeg) : K;

  uint32_t g_off[LPS];
#pragma unroll
  for (int it = 0; it < LPS; ++it) {
    const bool is_a = it < NLDA;
    const int s = (is_a ? it : it - NLDA) * C::NT + tid;
    const int r = s / NCH, c = (s % NCH) ^ attn_swz_k<ROWB>(r);
    const int row = is_a ? min(m0 + r, M - 1) - m0 : min(n0 + r, N - 1) - n0;
    g_off[it] = (uint32_t)row * (uint32_t)rowbytes + c * 16;
  }
  const char* const a_tile = (const char*)p.a + (size_t)m0 * rowbytes + (size_t)kbeg * 2;
  const char* const b_tile = (const char*)p.b + (size_t)n0 * rowbytes + (size_t)kbeg * 2;
  const uint32_t lds_wave = (uint32_t)(uintptr_t)smem + w * 1024;
  auto issue_load = [&](int ks, int slot, int it) __attribute__((always_inline)) {
    if (it < NLDA) attn_lds_dma16(a_tile + (size_t)ks * ROWB, g_off[it], lds_wave + slot * STAGEB + it * C::NT * 16);
    else attn_lds_dma16(b_tile + (size_t)ks * ROWB, g_off[it], lds_wave + slot * STAGEB + TILEA + (it - NLDA) * C::NT * 16);
  };

  const int nk = kcnt / BK;
#pragma unroll
  for (int s = 0; s < NSTAGE; ++s)
    if (s < nk) {
#pragma unroll
      for (int it = 0; it < LPS; ++it) issue_load(s, s, it);
    }

  // Two slots request an operand one stage, about 1 us, before it is used: enough for what another workgroup has brought
  // into the XCD's L2, not for what comes from memory.  So the workgroups that share a panel fetch it into the L2 four stages
  // ahead between them: per stage one load of one line per lane and wave (waves 0, 1 half of the A panel's rows, waves 2, 3 of
  // B's, which half by the tile's place; written into LDS that the ring leaves over and never read).  It goes out
  // behind the stage's own loads, so that a wait for those leaves it in flight.  Where: see the launches.  Measured, without -> with,
  // buffers changing from call to call: split-K 2304 x 1024 x 65536 298 -> 258 us, x 65600 262 -> 244, 3000 x 1000 x 20480 122 -> 116.
  constexpr int DIST = 4;
  static_assert(!AHEAD || (NSTAGE == 2 && C::LDS_BYTES >= NSTAGE * STAGEB + 4096), "room for what is fetched ahead");
  const char* const pf_tile = w < 2 ? a_tile : b_tile;
  const int pf_row = (((w < 2 ? tc.tn : tc.tm) * 2 + w) & 3) * 64, pf_last = w < 2 ? M - 1 - m0 : N - 1 - n0;
  auto fetch_ahead = [&](int ks) __attribute__((always_inline)) {
    int r = lane;
    asm volatile("" : "+v"(r));  // (the offset is made here each time: no register is left to keep it in)
    attn_lds_dma16(pf_tile + (size_t)min(ks + DIST, nk - 1) * ROWB, (uint32_t)min(pf_row + r, pf_last) * (uint32_t)rowbytes, lds_wave + NSTAGE * STAGEB);
  };

  // fragment addresses: row block 0 of this wave's quarter, k-step ph
  uint32_t ra[NPH], rb[NPH];
#pragma unroll
  for (int ph = 0; ph < NPH; ++ph) {
    const int rowa = wm * 128 + lj, rowb = wn * 128 + lj;
    ra[ph] = rowa * ROWB + (((4 * ph + g) ^ attn_swz_k<ROWB>(rowa)) << 4);
    rb[ph] = TILEA + rowb * ROWB + (((4 * ph + g) ^ attn_swz_k<ROWB>(rowb)) << 4);
  }

  f32x4 acc[8][8];  // [n block][m block]: rows of the accumulator are n (4 g + r), its column is m (lj)
#pragma unroll
  for (int nb = 0; nb < 8; ++nb)
#pragma unroll
    for (int mb = 0; mb < 8; ++mb)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[nb][mb][r] = 0.f;

  bf16x8 fa[2][8], fb[2][8];
  // fragment r of a k-step in the order of first use: the first n block, the eight m blocks, the other n blocks
  auto read_frag = [&](int buf, int base, int ph, int r) __attribute__((always_inline)) {
    if (r >= 1 && r <= 8) fa[buf][r - 1] = *(LDS_AS bf16x8*)(smem + ra[ph] + base + (r - 1) * 16 * ROWB);
    else fb[buf][r ? r - 8 : 0] = *(LDS_AS bf16x8*)(smem + rb[ph] + base + (r ? r - 8 : 0) * 16 * ROWB);
  };

  if (NSTAGE <= nk) ATTN_WAIT_VMCNT((NSTAGE - 1) * LPS);
  else ATTN_WAIT_VMCNT(0);
  attn_wg_barrier();
#pragma unroll
  for (int r = 0; r < 16; ++r) read_frag(0, 0, 0, r);

  // One k-stage; PAR: which fragment buffer its first k-step uses (stages of one k-step alternate).
  // A k-step is eight rows of eight MFMAs (one n block each), fenced one by one: every row carries two
  // or three fragment reads of the next k-step and DPR direct-to-LDS loads, each behind an MFMA of its own.
  // (All loads of a stage in one go behind the barrier kept the waves from issuing MFMAs until the
  // address unit had taken them: 1.61 M cycles at 8192^3 where the matrix pipe needs 1.05 M.)  The stage
  // boundary sits behind the first row of a stage's last k-step: that k-step's fragments, requested one
  // k-step ago, have arrived by then, and the slot of the stage is free for stage ks+NSTAGE.
  auto stage = [&](int ks, int slot, auto steady, auto par) __attribute__((always_inline)) {
    constexpr bool STEADY = decltype(steady)::value;
    constexpr int PAR = decltype(par)::value;
    constexpr int DPR = NSTAGE > 2 ? LPS / (8 * NPH) : 2 * LPS / (8 * NPH);  // (two slots: early enough to arrive)
    static_assert(DPR >= 1 && DPR <= 2, "loads per row");
    const int base = slot * STAGEB;
    const int nslot = slot == NSTAGE - 1 ? 0 : slot + 1;
    const int pslot = slot == 0 ? NSTAGE - 1 : slot - 1;
    const bool more = STEADY || ks + 1 < nk;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ph = 0; ph < NPH; ++ph) {
      const int cur = (PAR + ph) & 1, nxt = cur ^ 1;
      const bool last = ph == NPH - 1;
#pragma unroll
      for (int row = 0; row < 8; ++row) {
        if (last && row == 1 && more) {
          __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wave's reads of the slot about to be refilled are done
          if (AHEAD) ATTN_WAIT_VMCNT(1);
          else if (STEADY || ks + NSTAGE - 1 < nk) ATTN_WAIT_VMCNT((NSTAGE - 2) * LPS);
          else ATTN_WAIT_VMCNT(0);
          attn_wg_barrier();
        }
        // reads of this row: first .. first + count - 1
        const int count = !last ? 2 : row == 0 ? 0 : row < 3 ? 3 : 2;
        const int first = !last ? 2 * row : row == 0 ? 0 : row < 3 ? 3 * (row - 1) : 2 * row;
        // rows since the barrier that freed the slot: behind it the loads of stage ks+NSTAGE, before it those left of the one before
        const bool behind = last && row >= 1;
        const int q = behind ? row - 1 : 7 + 8 * ph + row;
        const int dks = behind ? ks + NSTAGE : ks - 1 + NSTAGE;
        const bool load = STEADY || (dks < nk && (behind || ks >= 1));
#pragma unroll
        for (int mb = 0; mb < 8; ++mb) {
          acc[row][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[cur][row], fa[cur][mb], acc[row][mb], 0, 0, 0);
          if ((mb & 1) == 0 && mb / 2 < count) {
            if (!last) read_frag(nxt, base, ph + 1, first + mb / 2);
            else if (more) read_frag(nxt, nslot * STAGEB, 0, first + mb / 2);
          }
          if ((mb == 5 || (mb == 7 && DPR > 1)) && load) {
            const int it = q * DPR + (mb == 7 ? 1 : 0);
            if (it < LPS) issue_load(dks, behind ? slot : pslot, it);
          }
          if (AHEAD && ph == 0 && row == 2 && mb == 5) fetch_ahead(ks);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  };

  // stages of one k-step alternate between the two fragment buffers: they are run in pairs (the host
  // only picks this kernel when the number of stages is even)
  int slot = 0, ks = 0;
  auto advance = [&]() __attribute__((always_inline)) {
    slot = slot == NSTAGE - 1 ? 0 : slot + 1;
    ++ks;
  };
  auto step = [&](auto steady) __attribute__((always_inline)) {
    stage(ks, slot, steady, std::integral_constant<int, 0>{});
    advance();
    if (NPH & 1) {
      stage(ks, slot, steady, std::integral_constant<int, 1>{});
      advance();
    }
  };
  constexpr int PER_STEP = (NPH & 1) ? 2 : 1;
  if (nk > 0) step(std::false_type{});
  while (ks + PER_STEP - 1 + NSTAGE < nk) step(std::true_type{});
  while (ks < nk) step(std::false_type{});
  if (AHEAD) ATTN_WAIT_VMCNT(0);

  // ---- epilogue: lane (lj, g) holds, for row m, the columns n = 16 nb + 4 g + (0..3); a pair of
  // neighbouring n blocks is exchanged between odd and even lane groups so that every lane owns 8
  // consecutive columns: one 16-byte store each
  if (SPLITK) {
    // fp32 partial tile: every lane owns 4 consecutive columns of row m, one 16-byte store
    const bool vec4 = (N & 3) == 0;
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) {
      const int m = m0 + wm * 128 + mb * 16 + lj;
      float* const prow = p.partial + ((size_t)split * M + (size_t)min(m, M - 1)) * N;
#pragma unroll
      for (int nb = 0; nb < 8; ++nb) {
        const int n = n0 + wn * 128 + nb * 16 + 4 * g;
        if (m < M) {
          if (vec4 && n + 4 <= N) {
            *(f32x4*)(prow + n) = acc[nb][mb];
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (n + e < N) prow[n + e] = acc[nb][mb][e];
          }
        }
      }
    }
    return;
  }
  __syncthreads();  // no wave reads the ring any more
#pragma unroll
  for (int mb = 0; mb < 8; ++mb) {
    const uint32_t row = (wm * 128 + mb * 16 + lj) * C::PITCH;
#pragma unroll
    for (int nb = 0; nb < 8; nb += 2) {
      uint32_t x[2], y[2];
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const uint32_t tx = pack_bf16(acc[nb][mb][2 * r], acc[nb][mb][2 * r + 1]);
        const uint32_t ty = pack_bf16(acc[nb + 1][mb][2 * r], acc[nb + 1][mb][2 * r + 1]);
        auto sw = __builtin_amdgcn_permlane16_swap(tx, ty, false, false);
        x[r] = sw[0];
        y[r] = sw[1];
      }
      // even lane groups: own block nb, columns 4g .. 4g+7; odd ones: block nb+1, columns 4(g-1) .. 4(g-1)+7
      const int n = wn * 128 + (nb + (g & 1)) * 16 + 4 * (g & ~1);
      *(LDS_AS u32x4*)(smem + row + n * 2) = u32x4{x[0], x[1], y[0], y[1]};
    }
  }
  __syncthreads();
  gemm_store_staged<C::BM, C::BN>(smem, p, m0, n0, tid);
}

template <int BK, int NSTAGE, bool AHEAD = false>
int launch_m16(const GemmParams& p, hipStream_t stream) {
  hipLaunchKernelGGL((gemm_bf16_nt_m16_kernel<BK, NSTAGE, false, AHEAD>), dim3(p.tiles_m * p.tiles_n), dim3(256), 0, stream, p);
  return (int)hipGetLastError();
}

// Fetching ahead (see the kernel) pays where K is long and every panel has several tiles to share it; us, without -> with:
// 4000 x 4000 x 9984 237 -> 231, 4096 x 4096 x 16384 413 -> 399, 8192 x 8192 x 16384 1634 -> 1610, 4096 x 4096 x 65536 1882 -> 1582,
// 1000 x 15000 x 16384 405 -> 392; 512 x 30000 x 16384 (two tile rows) 403 -> 421, 8192 x 8192 x 4096 370 -> 385,
// 3000 x 30000 x 2752 393 -> 400.  (One kernel with a branch instead: 0.5 % slower on the launches that do not fetch ahead.)
// What it gives depends on where the operands are.  Either side of the line, from memory / from the memory-side cache: 1003 x 2609 x 7552
// 163 -> 147 / 131 -> 132, 6197 x 4606 x 7936 377 -> 349 / 332 -> 351, 1439 x 1708 x 8192 171 -> 149 / 140 -> 142, 6108 x 4303 x 8192 361 -> 348 /
// 329 -> 338, 7714 x 4385 x 8640 525 -> 522 / 510 -> 519.  So for operands from memory the line could lie lower (1585 x 1960 x 4096 88 -> 78 / 74 -> 75).
int launch_m16_by_size(const GemmParams& p, hipStream_t stream) {
  return p.K >= 8192 && p.tiles_m >= 4 && p.tiles_n >= 4 ? launch_m16<64, 2, true>(p, stream) : launch_m16<64, 2>(p, stream);
}

// c[i] = bf16(sum over splits of partial[s][i]), splits added in index order.  VEC: four consecutive
// elements per thread (total a multiple of 4: every slice starts 16-byte aligned), else four
// elements 256 apart, so that a wave reads whole lines either way; the loads of four slices are in
// flight at a time.
template <bool VEC>
__global__ void __launch_bounds__(256) gemm_splitk_sum_kernel(const float* __restrict__ partial, __bf16* __restrict__ c, size_t total, int splits) {
  const size_t i0 = (size_t)blockIdx.x * 1024 + (VEC ? threadIdx.x * 4 : threadIdx.x);
  auto load = [&](int s) __attribute__((always_inline)) {
    const float* const src = partial + (size_t)s * total;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if constexpr (VEC) {
      if (i0 < total) v = *(const f32x4*)(src + i0);
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (i0 + 256 * t < total) v[t] = src[i0 + 256 * t];
    }
    return v;
  };
  f32x4 sum = load(0);
  int s = 1;
  for (; s + 4 <= splits; s += 4) {
    const f32x4 a = load(s), b = load(s + 1), d = load(s + 2), e = load(s + 3);
    sum = (((sum + a) + b) + d) + e;
  }
  for (; s < splits; ++s) sum += load(s);
  if constexpr (VEC) {
    if (i0 < total) *(u32x2*)(c + i0) = u32x2{pack_bf16(sum[0], sum[1]), pack_bf16(sum[2], sum[3])};
  } else {
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (i0 + 256 * t < total) c[i0 + 256 * t] = (__bf16)sum[t];
  }
}

template <int WM, int WN, int BK, int NSTAGE, int MINW, bool BKN = false>
int launch(const GemmParams& p, hipStream_t stream) {
  hipLaunchKernelGGL((gemm_bf16_kernel<WM, WN, BK, NSTAGE, MINW, BKN>), dim3(p.tiles_m * p.tiles_n), dim3(256), 0, stream, p);
  return (int)hipGetLastError();
}

}  // namespace

int gemm_bf16_nt_splitk_launch(const GemmParams& p, hipStream_t stream) {
  // Fetched ahead from three rows and columns of tiles on.  Of one row or column nobody shares the panel and of the other operand only half
  // is fetched; with two, what is fetched for some twenty panels of which each has two users can outgrow an XCD's L2.  Time with over without, 2532
  // launches, operands from memory / all of them in the memory-side cache, geometric means (worst): one 1.01 / 1.01 (1.08 / 1.10: 105 x 4127 x
  // 27520 69 -> 75 us), two 0.98 / 1.00 (1.15 / 1.48: 5140 x 281 x 49344 240 -> 355, 321 x 5342 x 48960 240 -> 274), three 0.96 / 0.99 (1.04 / 1.09),
  // four and more 0.95 / 0.98 (1.03 / 1.14).
  const dim3 grid(p.tiles_m * p.tiles_n * p.splits);
  if (p.tiles_m > 2 && p.tiles_n > 2) hipLaunchKernelGGL((gemm_bf16_nt_m16_kernel<64, 2, true, true>), grid, dim3(256), 0, stream, p);
  else hipLaunchKernelGGL((gemm_bf16_nt_m16_kernel<64, 2, true, false>), grid, dim3(256), 0, stream, p);
  return (int)hipGetLastError();
}

int gemm_splitk_sum_launch(const GemmParams& p, hipStream_t stream) {
  const size_t total = (size_t)p.M * p.N;
  const dim3 grid((unsigned)((total + 1023) / 1024));
  if ((total & 3) == 0) hipLaunchKernelGGL(gemm_splitk_sum_kernel<true>, grid, dim3(256), 0, stream, p.partial, (__bf16*)p.c, total, p.splits);
  else hipLaunchKernelGGL(gemm_splitk_sum_kernel<false>, grid, dim3(256), 0, stream, p.partial, (__bf16*)p.c, total, p.splits);
  return (int)hipGetLastError();
}

const GemmVariant* gemm_bf16_nt_variants(int* count) {
  static const GemmVariant table[] = {
      {"bf16 nt 256x256x32 ring4", 256, 256, 32, 32, launch<4, 4, 32, 4, 1>},
      {"bf16 nt 256x256x64 ring2", 256, 256, 64, 64, launch<4, 4, 64, 2, 1>},
      {"bf16 nt 128x128x64 ring2", 128, 128, 64, 64, launch<2, 2, 64, 2, 2>},
      {"bf16 nt 128x128x64 ring4", 128, 128, 64, 64, launch<2, 2, 64, 4, 1>},
      {"bf16 nt 64x64x64 ring2", 64, 64, 64, 64, launch<1, 1, 64, 2, 4>},
      {"bf16 nt 64x64x32 ring4", 64, 64, 32, 32, launch<1, 1, 32, 4, 4>},
      {"bf16 nt 256x256x32 ring4 mfma16x16x32", 256, 256, 32, 64, launch_m16<32, 4>},
      {"bf16 nt 256x256x64 ring2 mfma16x16x32", 256, 256, 64, 64, launch_m16<64, 2>},
      // (64-wide stages whose last one may be half: K a multiple of 32)
      {"bf16 nt 256x128x64 ring3", 256, 128, 32, 32, launch<4, 2, 64, 3, 1>},
      {"bf16 nt 128x256x64 ring3", 128, 256, 32, 32, launch<2, 4, 64, 3, 1>},
      {"bf16 nt 128x256x32 ring3", 128, 256, 32, 32, launch<2, 4, 32, 3, 2>},
      {"bf16 nt 128x128x64 ring4 half", 128, 128, 32, 32, launch<2, 2, 64, 4, 1>},
      {"bf16 nt 64x128x64 ring3", 64, 128, 32, 32, launch<1, 2, 64, 3, 2>},
      {"bf16 nt 64x128x64 ring2", 64, 128, 32, 32, launch<1, 2, 64, 2, 3>},
      {"bf16 nt 64x128x32 ring4", 64, 128, 32, 32, launch<1, 2, 32, 4, 3>},
  };
  *count = (int)(sizeof(table) / sizeof(table[0]));
  return table;
}

const GemmVariant* gemm_bf16_nt_ahead_variants(int* count) {
  static const GemmVariant table[] = {{"bf16 nt 256x256x64 ring2 mfma16x16x32 fetched ahead", 256, 256, 64, 64, launch_m16<64, 2, true>}};
  *count = 1;
  return table;
}

// The rates (GemmTile) are a fit to about 70 shapes per layout, M 1 .. 590000, N 32 .. 65536, K 64 .. 16384.
const GemmTile* gemm_bf16_nt_tiles(int* count) {
  static const GemmTile table[] = {
      {256, 256, 64, 1, 5.9f, 0.985f, 5.5f, launch_m16_by_size, 64},
      {256, 256, 32, 1, 6.1f, 0.58f, 5.5f, launch<4, 4, 32, 4, 1>},
      {256, 128, 64, 1, 4.4f, 0.62f, 5.5f, launch<4, 2, 64, 3, 1>},
      {128, 256, 64, 1, 4.1f, 0.65f, 5.5f, launch<2, 4, 64, 3, 1>},
      {128, 256, 32, 2, 1.8f, 0.42f, 5.5f, launch<2, 4, 32, 3, 2>},
      {128, 128, 64, 1, 2.7f, 0.39f, 5.5f, launch<2, 2, 64, 4, 1>},
      {64, 128, 64, 2, 0.7f, 0.30f, 5.5f, launch<1, 2, 64, 3, 2>},
      {64, 128, 64, 3, 0.1f, 0.42f, 5.5f, launch<1, 2, 64, 2, 3>},
      {64, 128, 32, 3, 0.3f, 0.20f, 5.5f, launch<1, 2, 32, 4, 3>},
      {64, 64, 32, 5, 0.0f, 0.14f, 5.5f, launch<1, 1, 32, 4, 4>},
  };
  *count = (int)(sizeof(table) / sizeof(table[0]));
  return table;
}

const GemmTile* gemm_bf16_nn_tiles(int* count) {
  static const GemmTile table[] = {
      {256, 256, 32, 1, 5.0f, 0.55f, 5.5f, launch<4, 4, 32, 4, 1, true>},
      {256, 128, 32, 2, 2.4f, 0.35f, 5.5f, launch<4, 2, 32, 3, 2, true>},
      {128, 256, 32, 2, 1.9f, 0.34f, 5.5f, launch<2, 4, 32, 3, 2, true>},
      {128, 128, 32, 2, 1.1f, 0.22f, 5.5f, launch<2, 2, 32, 4, 2, true>},
      {64, 256, 32, 2, 0.9f, 0.25f, 5.5f, launch<1, 4, 32, 4, 2, true>},
      {64, 128, 32, 3, 0.3f, 0.16f, 5.5f, launch<1, 2, 32, 4, 3, true>},
  };
  *count = (int)(sizeof(table) / sizeof(table[0]));
  return table;
}

// Attention backward, bf16, gfx950 (head dimension 128 or 64).
//
// The paper lists the backward pass beside the forward among its attention kernels (section
// 6.1; appendix A, attention shape table, backward rows).  Given Q, K, V, the forward output O
// with its per-row logsumexp, and the output gradient dO:
//
//     P  = exp(scale Q K^T - lse)             (rebuilt from the stored statistic, no maximum needed)
//     dV = P^T dO        dP = dO V^T        delta_i = sum_d dO_id O_id
//     dS = P * (dP - delta)                 dQ = scale dS K        dK = scale dS^T Q
//
// Two kernels, neither of which uses atomics or a reduction across workgroups, so the result is
// deterministic and no gradient needs an fp32 accumulation buffer in memory:
//
//   * attn_bwd_dq_kernel: a workgroup owns 128 query rows (64 when the launch is small, 256 in attn_bwd_dq_wide_kernel, which some launches
//     take; Q and dO rows stationary in registers as MFMA B operands, one query per lane, exactly the forward layout) and streams K/V tiles:
//     S^T = K Q^T, dP^T = V dO^T, dS^T in registers, dQ^T += K^T dS^T.  It also writes the two
//     per-row vectors the other kernel needs, -delta and lse * log2(e), into the workspace.
//   * attn_bwd_dkv_pipe_kernel: a workgroup owns 128 keys (64 when the launch is small; K and V rows stationary, one key per
//     lane) and streams Q/dO tiles of every query head of its group: S = Q K^T, dP = dO V^T, P,
//     dS = P * (dP - delta), dV^T += dO^T P, dK^T += Q^T dS.
//   S and dP are therefore computed twice, 7 matrix products per tile pair instead of the minimal
//   5: the price of keeping every accumulator in registers without atomics.
//
// Both share the forward kernels' machinery: 64-row tiles streamed HBM/L2 -> LDS by
// direct-to-LDS loads into a ring of slots two tiles ahead (one workgroup barrier per tile),
// transposed products on the 32x32x16 MFMA so that the exponentiated accumulator is the next
// B operand in place, and the transposing LDS read for the operand that must be contracted
// over its row index.  Streamed tiles are read both row-wise and transposed, so their 16-byte
// chunks are swizzled with a bit-swap of the row (conflict-free for both patterns).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "attn_device.h"
#include "attn_kernels.h"
#include "tile_map.h"

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

template <int V>
using ic = std::integral_constant<int, V>;

constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  bf16x2 t;
  t[0] = (__bf16)a;
  t[1] = (__bf16)b;
  return __builtin_bit_cast(uint32_t, t);
}

// Chunk swizzle of a streamed tile.  256-byte rows (16 chunks): XOR with the bit-swapped low four
// row bits.  Row-wise operand reads (16 lanes, one chunk of 16 consecutive rows) see 16 different
// values; transposing reads (16 lanes over 4 consecutive rows x 32 bytes, two such groups on
// neighbouring chunk pairs served together) see the rows in different 64-byte groups.
// 128-byte rows (8 chunks, two rows per 256-byte bank line): rows of equal parity share a half
// line, so the XOR value is built from row bits 1-3: bit 1 selects the 64-byte group (rows r and
// r + 2, which a transposing read takes together, fall into different groups), bits 2-3 the chunk
// inside it; 16 consecutive rows then see every (half line, chunk) pair once.
template <int ROWB>
__device__ __forceinline__ constexpr int swz_rt(int row) {
  static_assert(ROWB == 256 || ROWB == 128, "row of 128 or 64 bf16");
  return ROWB == 256 ? ((row & 3) << 2) | ((row >> 2) & 3) : (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
}

template <class F, int... M>
__device__ __forceinline__ void for_each_slot(F f, std::integer_sequence<int, M...>) {
  (f(ic<M>{}), ...);
}

// store a transposed accumulator (lane (ci,h) holds rows 32cb + 8a + 4h + r of column ci) as
// row `row` of a [.., D] bf16 matrix, scaled; the two lane halves exchange so that every lane
// writes 8 consecutive columns with one 16-byte store
template <int NCB>
__device__ __forceinline__ void store_transposed(const f32x16 (&acc)[NCB], float mul, char* rowptr, int h, bool valid) {
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      uint32_t x[2], y[2];
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const uint32_t tx = pack_bf16(acc[cb][(2 * a) * 4 + 2 * r] * mul, acc[cb][(2 * a) * 4 + 2 * r + 1] * mul);
        const uint32_t ty = pack_bf16(acc[cb][(2 * a + 1) * 4 + 2 * r] * mul, acc[cb][(2 * a + 1) * 4 + 2 * r + 1] * mul);
        auto sw = __builtin_amdgcn_permlane32_swap(tx, ty, false, false);
        x[r] = sw[0];
        y[r] = sw[1];
      }
      if (valid) {
        u32x4 out = {x[0], x[1], y[0], y[1]};
        *(u32x4*)(rowptr + (cb * 32 + a * 16 + h * 8) * 2) = out;
      }
    }
}

// =====================================================================================================
// dQ (and the workspace vectors)
// Four waves, one per SIMD, each with 32 queries (Q and dO rows stationary) and up to the whole register file.  K and V
// tiles are streamed, and a step works on three 32-key blocks at once: the score products of block i+1, the
// exponentials and dS of block i, the gradient products of block i-1; none of a step's MFMAs depends on its vector
// work.  A slot is one MFMA with a share of the vector work, the LDS reads of the operand RA slots ahead and, in one step
// per tile, a load of the tile three ahead.  The gradient products come first, and all their operands were requested by
// the step before: the ring's slot of tile j-1 is free when tile j begins.
// Eight waves of 32 queries, two per SIMD, block by block without the pipeline -> this, whole backward: 2 x 1 heads x 656
// causal 49.4 -> 41.3 us (KS = 2: 37.7), 2 x 16 x 1000, d = 64 42.3 -> 40.1, 3 x 48/12 x 835 220 -> 211, 5 x 4/2 x 3220 438 -> 405 (381),
// 2 x 32 x 8192 6610 -> 6490; 4 x 16 x 2048 causal 262 -> 267 (the 256-row workgroup read K and V half as often).  Two query
// blocks per wave (half the LDS reads; a 256-row workgroup again): 4 x 64/8 x 4096 causal 3524 -> 3476, 2 x 32 x 8192 6490 -> 6540,
// and 5 - 45 % slower wherever the launch is small.
// KS = 2, for launches that leave CUs idle: the workgroup owns 64 queries, waves w and w + 2 share 32
// of them, one takes the first key block of every tile, the other the second, and the two partial dQ are added through
// LDS at the end.
// =====================================================================================================
template <int D_>
struct DqPipe {
  static constexpr int D = D_, BN = 64, NWAVES = 4, NT = NWAVES * 64;
  static constexpr int NKK = D / 16, NCB = D / 32, ROWB = D * 2, NCH = ROWB / 16;
  static constexpr int TILEB = BN * ROWB, SUBB = 32 * ROWB, NSLOT = 4;
  static constexpr int T2BASE = NSLOT * TILEB;
  static constexpr int NLD = BN * NCH / NT, LPT = 2 * NLD;  // loads per thread: of one tensor's tile, of both
  static constexpr int NS = 2 * NKK, NG = 2 * NCB;  // fragments of the score (K, V by turns) and of the gradient products of a block
  static constexpr int NM = NS + NG;                // 24 (d = 128) or 12 (d = 64)
  static constexpr int RA = NG;                     // slots 0 .. RA-1: gradient products
  static_assert(RA % 4 == 0 && NM % 4 == 0 && NM >= 2 * RA && NM / LPT >= 1, "schedule shape");
  // as in BwdPipe: groups of four slots, inside a group in the reverse of the order of use
  static constexpr int read_target(int m) { return (m / 4 + RA / 4) * 4 + 3 - m % 4; }
  static constexpr int VP0 = 3;
  static constexpr int vslot(int r) { return VP0 + (r * (NM - VP0)) / 16; }  // slot of row r's exponential
};

template <int D, bool CAUSAL, int KS>
__global__ void __launch_bounds__(256, 1) attn_bwd_dq_kernel(const AttnBwdParams p) {
  using C = DqPipe<D>;
  constexpr int NKK = C::NKK, NCB = C::NCB, ROWB = C::ROWB, NCH = C::NCH, TILEB = C::TILEB, SUBB = C::SUBB;
  constexpr int NLD = C::NLD, LPT = C::LPT, NT = C::NT, BN = C::BN, NQW = C::NWAVES / KS, BM = NQW * 32, NM = C::NM, RA = C::RA;
  static_assert(KS == 1 || KS == 2, "a tile has two key blocks");

  __shared__ __attribute__((aligned(1024))) char smem_raw[2 * C::NSLOT * TILEB];
  LDS_AS char* const smem = (LDS_AS char*)smem_raw;

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int qi = lane & 31, h = lane >> 5;

  const AttnTileCoord tc = attn_tile_coord_impl(blockIdx.x, p.B, p.Hq, p.Hkv, p.T, CAUSAL ? 1 : 0);
  const int N = p.N;
  const int hk = tc.hq / (p.Hq / p.Hkv);
  const int q0 = tc.t * BM;
  const int kg = KS == 1 ? 0 : w / NQW;  // which key block of a tile this wave computes (KS = 2)
  const int wq0 = q0 + (KS == 1 ? w : w % NQW) * 32;

  const int qrow = wq0 + qi;

  const size_t qoff = ((size_t)(tc.b * p.Hq + tc.hq) * N) * ROWB;
  const int kv_end = CAUSAL ? min(N, q0 + BM) : N;
  const int nt = (kv_end + BN - 1) / BN, nt_all = (N + BN - 1) / BN;

  uint32_t ld_off[NLD], ld_off_r[NLD];  // ("_r": inside the ragged last tile, whose rows past N-1 re-read row N-1)
#pragma unroll
  for (int it = 0; it < NLD; ++it) {
    const int s = it * NT + tid;
    const int r = s / NCH, c = s % NCH;
    ld_off[it] = r * ROWB + ((c ^ swz_rt<ROWB>(r)) << 4);
    ld_off_r[it] = ld_off[it] - (uint32_t)max(0, (N - 1) / BN * BN + r - (N - 1)) * ROWB;
  }
  const uint32_t lds_wave = (uint32_t)(uintptr_t)smem + w * 1024;
  // load i of the next tile, iss_j, into ring slot `slot`: K and V pieces by turns
  int iss_j = 0;
  const char* iss_k = (const char*)p.k + ((size_t)(tc.b * p.Hkv + hk) * N) * ROWB;
  const char* iss_v = (const char*)p.v + ((size_t)(tc.b * p.Hkv + hk) * N) * ROWB;
  auto issue_load = [&](int slot, int i) __attribute__((always_inline)) {
    const uint32_t off = iss_j == nt_all - 1 ? ld_off_r[i >> 1] : ld_off[i >> 1];
    attn_lds_dma16((i & 1) ? iss_v : iss_k, off, lds_wave + ((i & 1) ? C::T2BASE : 0) + slot * TILEB + (i >> 1) * NT * 16);
  };
  auto issue_advance = [&]() __attribute__((always_inline)) {
    ++iss_j;
    iss_k += TILEB;
    iss_v += TILEB;
  };
  auto issue_next = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < LPT; ++i) issue_load(slot, i);
    issue_advance();
  };
  issue_next(0);

  // ---- stationary operands: Q and dO rows of this lane's queries; delta from dO and O ---------------
  bf16x8 qf[NKK], dof[NKK];
  float delta;
  {
    const int row = min(qrow, N - 1);
    const char* qs = (const char*)p.q + qoff + (size_t)row * ROWB + h * 16;
    const char* ds = (const char*)p.dout + qoff + (size_t)row * ROWB + h * 16;
    const char* os = (const char*)p.o + qoff + (size_t)row * ROWB + h * 16;
    float acc = 0.f;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      qf[kk] = *(const bf16x8*)(qs + kk * 32);
      dof[kk] = *(const bf16x8*)(ds + kk * 32);
      const bf16x8 ov = *(const bf16x8*)(os + kk * 32);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc += (float)dof[kk][e] * (float)ov[e];
    }
    delta = attn_sum_halves(acc);
  }
  const float lse2 = p.lse[(size_t)(tc.b * p.Hq + tc.hq) * N + min(qrow, N - 1)] * kLog2e;
  // workspace for the key-side kernel, padded to whole 64-row tiles: rows past N get a
  // statistic of +inf (their probabilities come out as zero) and delta = 0; delta is kept negated
  if (kg == 0 && h == 0 && qrow < p.Npad) {
    float* const wsrow = p.ws + (size_t)(tc.b * p.Hq + tc.hq) * 2 * p.Npad;
    wsrow[qrow] = qrow < N ? lse2 : INFINITY;
    wsrow[p.Npad + qrow] = qrow < N ? -delta : 0.f;
  }
  if (nt > 1) issue_next(1);
  if (nt > 2) issue_next(2);

  // ---- LDS read addresses; inside the ring every offset is a compile-time immediate, V's slots lie beyond its range ----
  uint32_t raddr[2][NKK];
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) {
    raddr[0][kk] = kg * SUBB + qi * ROWB + (((2 * kk + h) ^ swz_rt<ROWB>(qi)) << 4);
    raddr[1][kk] = raddr[0][kk] + C::T2BASE;
    asm volatile("" : "+v"(raddr[1][kk]));
  }
  uint32_t taddr[NCB][2];
  {
    const int s = lane & 15, chalf = (lane >> 4) & 1;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int key = 8 * e + 4 * h + (s >> 2);
        const int chunk = cb * 4 + chalf * 2 + ((s & 3) >> 1);
        taddr[cb][e] = kg * SUBB + key * ROWB + ((chunk ^ swz_rt<ROWB>(key)) << 4) + ((s & 1) << 3);
      }
  }
  // operand of score fragment i of the block at `off`: S^T = K Q^T (even i), dP^T = V dO^T (odd i)
  auto score_operand = [&](int off, int i) __attribute__((always_inline)) { return *(LDS_AS u32x4*)(smem + raddr[i & 1][i >> 1] + off); };
  // operand of gradient fragment i of the block at `off`: dQ^T += K^T dS^T
  auto grad_operand = [&](int off, int i) __attribute__((always_inline)) {
    const int cb = i % NCB, kc = i / NCB;
    const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(smem + taddr[cb][0] + off + kc * 16 * ROWB));
    const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(smem + taddr[cb][1] + off + kc * 16 * ROWB));
    s16x8 av;
    av[0] = v0[0]; av[1] = v0[1]; av[2] = v0[2]; av[3] = v0[3];
    av[4] = v1[0]; av[5] = v1[1]; av[6] = v1[2]; av[7] = v1[3];
    return __builtin_bit_cast(u32x4, av);
  };

  f32x16 acc[NCB];  // dQ^T
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[cb][r] = 0.f;
  auto grads_settled = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) asm volatile("s_nop 15" : "+a"(acc[cb]));
  };
  grads_settled();
  // (an assembly statement for the reason, and under the conditions, given at the dK/dV kernel's)
  auto grad_mfma = [&](int i, u32x4 o, const u32x4 (&pd)[2], auto copied) __attribute__((always_inline)) {
    f32x16& sum = acc[i % NCB];
    const u32x4 ds = pd[i / NCB];
    if constexpr (decltype(copied)::value) asm volatile("s_nop 3\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(sum) : "v"(o), "v"(ds));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(sum) : "v"(o), "v"(ds));
  };

  const float c = p.scale_log2;
  f32x16 from;  // what dP starts from (instead of a subtraction per element)
#pragma unroll
  for (int r = 0; r < 16; ++r) from[r] = -delta;
  asm volatile("" : "+v"(from));

  struct Scores {
    f32x16 s, dp;
  };
  struct Packed {
    u32x4 d[2];
  };
  u32x4 pre[RA];  // operands of the next step's gradient products
  constexpr int LGAP = NM / LPT;
  // One step: scores of the block at NEXT -> out; dS of the block at CUR (scores `in`, first key key0) -> pd_out; pd_acc, the
  // block before, multiplied into dQ.  `load`: the tile iss_j is requested into slot LSLOT (-1: none)
  auto step = [&](Scores& in, Scores& out, Packed& pd_out, const Packed& pd_acc, auto CUR, auto NEXT, auto LSLOT, int key0, bool load) __attribute__((always_inline)) {
    constexpr int cur = decltype(CUR)::value, next = decltype(NEXT)::value;
    u32x4 op[NM];
#pragma unroll
    for (int m = 0; m < RA; ++m) op[m] = pre[m];
    float x[16], e[16], f[16];
    __builtin_amdgcn_sched_barrier(0);
    auto one_slot = [&](auto slot_tag) __attribute__((always_inline)) {
      constexpr int m = decltype(slot_tag)::value;
      constexpr int tgt = C::read_target(m);
      if constexpr (tgt < NM) op[tgt] = score_operand(next, tgt - RA);
      else pre[tgt - NM] = grad_operand(cur, tgt - NM);
      if constexpr (m < RA) {
        grad_mfma(m, op[m], pd_acc.d, std::false_type{});
      } else {
        constexpr int i = m - RA;
        f32x16& dst = (i & 1) ? out.dp : out.s;
        if constexpr (i < 2) {
#pragma unroll
          for (int r = 0; r < 16; ++r) dst[r] = i ? from[r] : 0.f;
        }
        dst = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, op[m]), (i & 1) ? dof[i >> 1] : qf[i >> 1], dst, 0, 0, 0);
      }
      if constexpr (decltype(LSLOT)::value >= 0 && m % LGAP == 0 && m / LGAP < LPT) {
        if (load) issue_load(decltype(LSLOT)::value, m / LGAP);
      }
      // invisible keys (causal diagonal, ragged end): a score of -inf gives P = 0 and dS = 0 (wave-uniform branch)
      if constexpr (m == C::VP0 - 2) {
        if ((CAUSAL && key0 + 31 > wq0) || key0 + 31 >= N) {
          const int limit = CAUSAL ? min(qrow, N - 1) : N - 1;
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (key0 + 4 * h + 8 * (r >> 2) + (r & 3) > limit) in.s[r] = -INFINITY;
        }
      }
      // vector work of row r, one link of its chain per slot: P = exp2(s c - lse2), dS = P (dP - delta), packs
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (C::vslot(r) - 1 == m) x[r] = __builtin_fmaf(in.s[r], c, -lse2);
        if (C::vslot(r) == m) e[r] = __builtin_amdgcn_exp2f(x[r]);
        if (C::vslot(r) + 1 == m || (m == NM - 1 && C::vslot(r) + 1 > m)) {
          f[r] = e[r] * in.dp[r];
          if (r & 1) pd_out.d[r >> 3][(r >> 1) & 3] = pack_bf16(f[r - 1], f[r]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    for_each_slot(one_slot, std::make_integer_sequence<int, NM>{});
    // (the packs are made here, not put off to where they are read)
    asm volatile("" : "+v"(pd_out.d[0]), "+v"(pd_out.d[1]), "+v"(out.s), "+v"(out.dp));
  };

  if (nt > 2) ATTN_WAIT_VMCNT(2 * LPT);
  else if (nt > 1) ATTN_WAIT_VMCNT(LPT);
  else ATTN_WAIT_VMCNT(0);
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) asm volatile("" : "+a"(qf[kk]), "+a"(dof[kk]));  // in registers from here on
  attn_wg_barrier();

  // prologue: scores of block 0
  Scores sa, sb;
  Packed pa, pb;
#pragma unroll
  for (int r = 0; r < 16; ++r) sa.s[r] = 0.f;
  sa.dp = from;
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) {
    sa.s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, score_operand(0, 2 * kk)), qf[kk], sa.s, 0, 0, 0);
    sa.dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, score_operand(0, 2 * kk + 1)), dof[kk], sa.dp, 0, 0, 0);
  }
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    pb.d[t] = u32x4{0u, 0u, 0u, 0u};
    asm volatile("s_nop 1" : "+v"(pb.d[t]));  // (not to be made again in front of the first product)
  }
#pragma unroll
  for (int m = 0; m < RA; ++m) {
    pre[m] = u32x4{0u, 0u, 0u, 0u};
    asm volatile("s_nop 1" : "+v"(pre[m]));
  }

  // Tiles that hold a block of this wave's that one of its queries sees.  Behind them (one tile at most: no loads are left) the wave only
  // keeps the barrier: a block none of its queries sees would add P = 0 times its keys and values, which is not zero where those are
  // infinite or NaN.
  const int last_block = (CAUSAL ? min(wq0 + 31, N - 1) : N - 1) >> 5;
  const int mine = (last_block + 2 - kg) >> 1;
  // tile j+1 has landed (the loads of tile j+2 stay in flight); every wave is done with tile j-1
  auto between = [&](int j) __attribute__((always_inline)) {
    if (KS == 2) __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wave's reads of tile j-1, whose slot is refilled, are done
    if (j + 2 < nt) ATTN_WAIT_VMCNT(LPT);
    else ATTN_WAIT_VMCNT(0);
    attn_wg_barrier();
  };
  // tile j lives in slot j % 4 = S
  auto tile = [&](auto S, int j) __attribute__((always_inline)) {
    constexpr int s = decltype(S)::value;
    constexpr int b0 = s * TILEB, b1 = b0 + SUBB, bn = ((s + 1) & 3) * TILEB;
    const bool load = j + 3 < nt;
    if constexpr (KS == 2) {
      between(j);
      if constexpr (s & 1) step(sb, sa, pb, pa, ic<b0>{}, ic<bn>{}, ic<(s + 3) & 3>{}, j * BN + kg * 32, load);
      else step(sa, sb, pa, pb, ic<b0>{}, ic<bn>{}, ic<(s + 3) & 3>{}, j * BN + kg * 32, load);
    } else {
      step(sa, sb, pa, pb, ic<b0>{}, ic<b1>{}, ic<-1>{}, j * BN, false);
      between(j);
      step(sb, sa, pb, pa, ic<b1>{}, ic<bn>{}, ic<(s + 3) & 3>{}, j * BN + 32, load);
    }
    if (load) issue_advance();
  };
  int j = 0;
  for (; j + 4 <= mine; j += 4) {
    tile(ic<0>{}, j);
    tile(ic<1>{}, j + 1);
    tile(ic<2>{}, j + 2);
    tile(ic<3>{}, j + 3);
  }
  if (j < mine) {
    tile(ic<0>{}, j);
    if (j + 1 < mine) {
      tile(ic<1>{}, j + 1);
      if (j + 2 < mine) tile(ic<2>{}, j + 2);
    }
  }
  if (mine < nt) between(mine);
  // the gradient products of the last block (its operands are already here), if that is a block the queries see
  if (KS == 2 && ((mine - 1) & 1) == 0) pb = pa;  // (the parity of the last step says which registers hold dS)
  if (KS == 2 || (last_block & 1)) {
#pragma unroll
    for (int i = 0; i < RA; ++i) grad_mfma(i, pre[i], pb.d, std::true_type{});
  }
  grads_settled();

  if constexpr (KS == 1) {
    store_transposed<NCB>(acc, p.scale, (char*)p.dq + qoff + (size_t)min(qrow, N - 1) * ROWB, h, qrow < N);
  } else {
    // the two waves of a query block exchange halves of their partial dQ (each gives away the columns the other one
    // finishes)
    constexpr int NH = NCB / 2;
    __syncthreads();  // no wave reads the ring any more
    LDS_AS f32x4* const give = (LDS_AS f32x4*)smem + ((kg ^ 1) * NQW + w % NQW) * (NH * 4) * 64 + lane;
    LDS_AS const f32x4* const take = (LDS_AS const f32x4*)smem + (kg * NQW + w % NQW) * (NH * 4) * 64 + lane;
    f32x16 mine[NH];
#pragma unroll
    for (int cb = 0; cb < NH; ++cb) {
      const f32x16 other = kg ? acc[cb] : acc[NH + cb];
      mine[cb] = kg ? acc[NH + cb] : acc[cb];
#pragma unroll
      for (int a = 0; a < 4; ++a) give[(cb * 4 + a) * 64] = f32x4{other[4 * a], other[4 * a + 1], other[4 * a + 2], other[4 * a + 3]};
    }
    __syncthreads();
#pragma unroll
    for (int cb = 0; cb < NH; ++cb)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const f32x4 o = take[(cb * 4 + a) * 64];
#pragma unroll
        for (int r = 0; r < 4; ++r) mine[cb][4 * a + r] += o[r];
      }
    store_transposed<NH>(mine, p.scale, (char*)p.dq + qoff + (size_t)min(qrow, N - 1) * ROWB + kg * NH * 64, h, qrow < N);
  }
}

// The same in workgroups of 256 queries: eight waves, two per SIMD, that work block by block without the pipeline.  K and V
// are read half as often, and launches of few short tiles take half the rounds over the CUs.
template <int D_>
struct DqWide {
  static constexpr int D = D_, BN = 64, NWAVES = 8, BM = NWAVES * 32, NT = NWAVES * 64;
  static constexpr int NKK = D / 16, NCB = D / 32, ROWB = D * 2, NCH = ROWB / 16;
  static constexpr int TILEB = BN * ROWB, SUBB = 32 * ROWB, NSLOT = 3;
  static constexpr int T2BASE = NSLOT * TILEB;  // V's slots
  static constexpr int NLD = BN * NCH / NT;
};

template <int D, bool CAUSAL>
__global__ void __launch_bounds__(512, 2) attn_bwd_dq_wide_kernel(const AttnBwdParams p) {
  using C = DqWide<D>;
  constexpr int NKK = C::NKK, NCB = C::NCB, ROWB = C::ROWB, NCH = C::NCH, TILEB = C::TILEB, SUBB = C::SUBB, NSLOT = C::NSLOT;
  constexpr int NLD = C::NLD, NT = C::NT, BN = C::BN, BM = C::BM;

  __shared__ __attribute__((aligned(1024))) char smem_raw[2 * NSLOT * TILEB];
  LDS_AS char* const smem = (LDS_AS char*)smem_raw;

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int qi = lane & 31, h = lane >> 5;

  const AttnTileCoord tc = attn_tile_coord_impl(blockIdx.x, p.B, p.Hq, p.Hkv, p.T, CAUSAL ? 1 : 0);
  const int N = p.N;
  const int hk = tc.hq / (p.Hq / p.Hkv);
  const int q0 = tc.t * BM;
  const int wq0 = q0 + w * 32;
  const bool wave_valid = wq0 < N;
  const int qrow = wq0 + qi;

  const size_t qoff = ((size_t)(tc.b * p.Hq + tc.hq) * N) * ROWB;
  const char* const khead = (const char*)p.k + ((size_t)(tc.b * p.Hkv + hk) * N) * ROWB;
  const char* const vhead = (const char*)p.v + ((size_t)(tc.b * p.Hkv + hk) * N) * ROWB;

  const int kv_end = CAUSAL ? min(N, q0 + BM) : N;
  const int nt = (kv_end + BN - 1) / BN;

  // ---- producer role ------------------------------------------------------------------------------
  int ld_row[NLD];
  uint32_t ld_off[NLD];
#pragma unroll
  for (int it = 0; it < NLD; ++it) {
    const int s = it * NT + tid;
    const int r = s / NCH, c = s % NCH;
    ld_row[it] = r;
    ld_off[it] = r * ROWB + ((c ^ swz_rt<ROWB>(r)) << 4);
  }
  const uint32_t lds_wave = (uint32_t)(uintptr_t)smem + w * 1024;
  auto issue_tile = [&](int j, int slot) __attribute__((always_inline)) {
    const char* const kb = khead + (size_t)j * TILEB;
    const char* const vb = vhead + (size_t)j * TILEB;
#pragma unroll
    for (int it = 0; it < NLD; ++it) {
      const uint32_t over = (uint32_t)max(0, j * BN + ld_row[it] - (N - 1)) * ROWB;  // rows past N-1 re-read row N-1
      attn_lds_dma16(kb, ld_off[it] - over, lds_wave + slot * TILEB + it * NT * 16);
      attn_lds_dma16(vb, ld_off[it] - over, lds_wave + C::T2BASE + slot * TILEB + it * NT * 16);
    }
  };
  issue_tile(0, 0);

  // ---- stationary operands: Q and dO rows of this lane's query; delta from dO and O ---------------
  bf16x8 qf[NKK], dof[NKK];
  float delta;
  {
    const int row = min(qrow, N - 1);
    const char* qs = (const char*)p.q + qoff + (size_t)row * ROWB + h * 16;
    const char* ds = (const char*)p.dout + qoff + (size_t)row * ROWB + h * 16;
    const char* os = (const char*)p.o + qoff + (size_t)row * ROWB + h * 16;
    float acc = 0.f;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      qf[kk] = *(const bf16x8*)(qs + kk * 32);
      dof[kk] = *(const bf16x8*)(ds + kk * 32);
      const bf16x8 ov = *(const bf16x8*)(os + kk * 32);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc += (float)dof[kk][e] * (float)ov[e];
    }
    delta = attn_sum_halves(acc);
  }
  const float lse2 = p.lse[(size_t)(tc.b * p.Hq + tc.hq) * N + min(qrow, N - 1)] * kLog2e;
  if (h == 0 && qrow < p.Npad) {
    float* const wsrow = p.ws + (size_t)(tc.b * p.Hq + tc.hq) * 2 * p.Npad;
    wsrow[qrow] = qrow < N ? lse2 : INFINITY;
    wsrow[p.Npad + qrow] = qrow < N ? -delta : 0.f;
  }
  if (nt > 1) issue_tile(1, 1);

  // ---- LDS read addresses (slot 0, first 32-row block) --------------------------------------------
  uint32_t raddr[NKK];  // row-wise operand: row qi, chunk 2kk + h
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) raddr[kk] = qi * ROWB + (((2 * kk + h) ^ swz_rt<ROWB>(qi)) << 4);
  uint32_t taddr[NCB][2];  // transposed operand through the transposing load
  {
    const int s = lane & 15, chalf = (lane >> 4) & 1;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int key = 8 * e + 4 * h + (s >> 2);
        const int chunk = cb * 4 + chalf * 2 + ((s & 3) >> 1);
        taddr[cb][e] = key * ROWB + ((chunk ^ swz_rt<ROWB>(key)) << 4) + ((s & 1) << 3);
      }
  }
  auto row_operand = [&](int base, int kk) __attribute__((always_inline)) { return *(LDS_AS bf16x8*)(smem + raddr[kk] + base); };
  auto tr_operand = [&](int base, int cb, int kc) __attribute__((always_inline)) {
    const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(smem + taddr[cb][0] + base + kc * 16 * ROWB));
    const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(smem + taddr[cb][1] + base + kc * 16 * ROWB));
    s16x8 av;
    av[0] = v0[0]; av[1] = v0[1]; av[2] = v0[2]; av[3] = v0[3];
    av[4] = v1[0]; av[5] = v1[1]; av[6] = v1[2]; av[7] = v1[3];
    return __builtin_bit_cast(bf16x8, av);
  };

  f32x16 acc[NCB];  // dQ^T
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[cb][r] = 0.f;
  const float c = p.scale_log2;
  const int limit = CAUSAL ? min(qrow, N - 1) : (N - 1);
  const int wlast = wq0 + 31;

  // one 32-key block: `base` = byte offset of the block inside the K slots (V: + T2BASE)
  auto block = [&](int key0, int base) __attribute__((always_inline)) {
    f32x16 s, dp;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = dp[r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(row_operand(base, kk), qf[kk], s, 0, 0, 0);
      dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(row_operand(base + C::T2BASE, kk), dof[kk], dp, 0, 0, 0);
    }
    // invisible keys (causal diagonal, ragged tail): a score of -inf gives P = 0 and dS = 0.  The
    // compare / select work sits behind a wave-uniform branch, the common case carries none of it.
    if ((CAUSAL && key0 + 31 > wq0) || key0 + 31 >= N) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (key0 + 4 * h + 8 * (r >> 2) + (r & 3) > limit) s[r] = -INFINITY;
    }
    u32x4 dsk[2];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      float e[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int r = 2 * u + t;
        const float pr = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c, -lse2));
        e[t] = pr * (dp[r] - delta);
      }
      dsk[u >> 2][u & 3] = pack_bf16(e[0], e[1]);
    }
#pragma unroll
    for (int i = 0; i < 2 * NCB; ++i) {
      const int cb = i % NCB, kc = i / NCB;
      acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(tr_operand(base, cb, kc), __builtin_bit_cast(bf16x8, dsk[kc]), acc[cb], 0, 0, 0);
    }
  };

  if (nt > 1) ATTN_WAIT_VMCNT(2 * NLD);
  else ATTN_WAIT_VMCNT(0);
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) asm volatile("" ::"v"(qf[kk]), "v"(dof[kk]));  // stationary operands are in registers
  attn_wg_barrier();

  int slot = 0;
  for (int j = 0; j < nt; ++j) {
    const int pslot = slot == 0 ? NSLOT - 1 : slot - 1;  // slot of tile j+2 = slot of tile j-1
    if (j + 2 < nt) issue_tile(j + 2, pslot);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int key0 = j * BN + i * 32;
      if (wave_valid && key0 < kv_end && (!CAUSAL || key0 <= wlast)) block(key0, slot * TILEB + i * SUBB);
    }
    if (j + 2 < nt) ATTN_WAIT_VMCNT(2 * NLD);  // tile j+1 has landed; the loads of tile j+2 stay in flight
    else ATTN_WAIT_VMCNT(0);
    attn_wg_barrier();
    slot = slot == NSLOT - 1 ? 0 : slot + 1;
  }

  store_transposed<NCB>(acc, p.scale, (char*)p.dq + qoff + (size_t)min(qrow, N - 1) * ROWB, h, qrow < N);
}

// =====================================================================================================
// dK and dV in one kernel (S and dP computed once for both).  The accumulators of both gradients
// (128 registers per 32 keys) beside the stationary K and V rows (64) leave no room for two waves
// per SIMD, so this kernel runs four waves of 32 keys, one per SIMD, with the whole register file;
// a workgroup owns 128 keys.
// With one wave per SIMD nothing else hides the vector work of a block behind matrix work, so the
// wave is software-pipelined: a step works on three 32-query blocks at once, the score products of
// block i+1, the exponentials and dS of block i, and the gradient products of block i-1.  The 32
// MFMAs of a step depend on none of its vector work.  Instruction order inside a step is fixed by
// hand (one MFMA per slot, operands requested two groups of four slots ahead, a row's vector work spread over
// three slots so that no instruction waits for the one before it, one load of the tile three ahead every few slots)
// and fenced slot by slot.  The ring has four slots because a step touches three
// tiles, and the loop is unrolled over them so that every LDS offset is an immediate.
// One wave per SIMD hides nothing it does not hide itself, so every instruction counts: the gradients and the
// stationary rows are pinned to accumulation registers, which leaves the scores in ordinary ones (the vector work had
// fetched them with 64 register moves a step), dP starts from -delta, and the loads are handed out singly (nine in a row behind the barrier stopped
// all products until the address unit had taken them).  Cycles of this kernel, 4 x 64/8 heads x 4096 causal: 4.13 M -> 3.60 M
// (matrix pipe 52 -> 60 % of them), time 2.11 -> 1.95 ms at a clock that the power limit lowers; the whole backward of
// 2 x 16 heads x 1000, d = 64 44.9 -> 43.1 us, of 3 x 48/12 x 835 232 -> 221.
// Every block of every tile is computed by every wave: a block that is invisible to the wave's keys
// (causal) or past the end (ragged) contributes exact zeros through the -inf scores and the +inf
// statistic of the padded workspace rows, and the slowest wave of the workgroup computes it anyway.
// =====================================================================================================
#ifndef ATTN_BWD_RA
#define ATTN_BWD_RA 8
#endif
template <int D_>
struct BwdPipe {
  static constexpr int D = D_, BN = 64, NWAVES = 4, BM = NWAVES * 32, NT = NWAVES * 64;
  static constexpr int NKK = D / 16, NCB = D / 32, ROWB = D * 2, NCH = ROWB / 16;
  static constexpr int TILEB = BN * ROWB, SUBB = 32 * ROWB, NSLOT = 4;
  static constexpr int T2BASE = NSLOT * TILEB;
  static constexpr int AUXBASE = 2 * NSLOT * TILEB;
  static constexpr int NLD = BN * NCH / NT;
  static constexpr int LDS_BYTES = AUXBASE + NSLOT * 512;
  static constexpr int NS = 2 * NKK;         // score products of a block: S and dP, NKK k-steps each
  static constexpr int NG = 4 * NCB;         // gradient products of a block: dV and dK, NCB column blocks x 2 k-steps
  static constexpr int NM = NS + NG;         // 32 (d = 128) or 16 (d = 64)
  static constexpr int RA = D == 128 ? ATTN_BWD_RA : 4;
  static_assert(NS == NG && RA % 4 == 0 && RA <= NS && NM % 4 == 0, "schedule shape");
  // slot p of a step: the first RA MFMAs are gradient products (their operands were requested by
  // the previous step, from a tile that is certainly resident), then score and gradient products
  // alternate, and the last RA are score products
  static constexpr bool is_score(int p) {
    if (p < RA) return false;
    const int q = p - RA, npairs = NS - RA;
    return q < 2 * npairs ? (q & 1) == 0 : true;
  }
  static constexpr int index(int p) {
    if (p < RA) return p;
    const int q = p - RA, npairs = NS - RA;
    if (q < 2 * npairs) return (q & 1) == 0 ? q / 2 : RA + q / 2;
    return npairs + (q - 2 * npairs);
  }
  // slot m requests the operand of slot read_target(m): two groups of four slots ahead, and inside
  // a group in the reverse of the order of use, so that the first product of a group waits for the
  // newest request of its batch and the other three need no wait instruction
  static constexpr int read_target(int m) { return (m / 4 + RA / 4) * 4 + 3 - m % 4; }
  static constexpr int VP0 = 6;                                                       // first slot with vector work
  static constexpr int vslot(int r) { return VP0 + (r * (NM - VP0)) / 16; }            // slot of row r's vector work
  static constexpr int dslot(int a) { return a; }  // slots that read -delta of the next block's rows 4a..4a+3 (its first dP product: slot RA + 2)
  static constexpr int aslot(int a) { return vslot(4 * a) - 6 > 0 ? vslot(4 * a) - 6 : 0; }  // slot that reads the statistics of rows 4a..4a+3
};

// QS = 1: each wave owns 32 of the workgroup's 128 keys and takes both 32-query blocks of every tile.
// QS = 2, for launches that leave CUs idle: a workgroup owns 64 keys; waves w and w + 2 share 32 of
// them, one takes the first query block of every tile, the other the second (its "previous" and
// "next" blocks are those of the neighbouring tiles), and at the end one finishes dV and the other
// dK with the partner's partial sum, exchanged through LDS.
template <int D, bool CAUSAL, int QS>
__global__ void __launch_bounds__(256, 1) attn_bwd_dkv_pipe_kernel(const AttnBwdParams p) {
  using C = BwdPipe<D>;
  constexpr int NKK = C::NKK, NCB = C::NCB, ROWB = C::ROWB, NCH = C::NCH, TILEB = C::TILEB, SUBB = C::SUBB;
  constexpr int NLD = C::NLD, NT = C::NT, BN = C::BN, NKW = C::NWAVES / QS, BM = NKW * 32, NM = C::NM, RA = C::RA;
  static_assert(QS == 1 || QS == 2, "a tile has two query blocks");

  __shared__ __attribute__((aligned(1024))) char smem_raw[C::LDS_BYTES];
  LDS_AS char* const smem = (LDS_AS char*)smem_raw;

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int ki = lane & 31, h = lane >> 5;

  const int T = (p.N + BM - 1) / BM;
  AttnTileCoord tc = attn_tile_coord_impl(blockIdx.x, p.B, p.Hkv, p.Hkv, T, CAUSAL ? 1 : 0);
  if (CAUSAL) tc.t = T - 1 - tc.t;  // key tile 0 is the heaviest: first
  const int N = p.N;
  const int G = p.Hq / p.Hkv;
  const int g = tc.hq;
  const int k0 = tc.t * BM;
  const int qg = QS == 1 ? 0 : w / NKW;                   // which query block of a tile this wave computes (QS = 2)
  const int wk0 = k0 + (QS == 1 ? w : w % NKW) * 32;  // first key of this wave
  const int krow = wk0 + ki;

  const size_t koff = ((size_t)(tc.b * p.Hkv + g) * N) * ROWB;
  const int nqt_all = (N + BN - 1) / BN;
  const int qt0 = CAUSAL ? k0 / BN : 0;
  const int nt = G * (nqt_all - qt0);

  uint32_t ld_off[NLD], ld_off_r[NLD];  // ("_r": inside the ragged last tile, whose rows past N-1 re-read row N-1)
#pragma unroll
  for (int it = 0; it < NLD; ++it) {
    const int s = it * NT + tid;
    const int r = s / NCH, c = s % NCH;
    ld_off[it] = r * ROWB + ((c ^ swz_rt<ROWB>(r)) << 4);
    ld_off_r[it] = ld_off[it] - (uint32_t)max(0, (N - 1) / BN * BN + r - (N - 1)) * ROWB;
  }
  const uint32_t lds_base = (uint32_t)(uintptr_t)smem;
  const uint32_t lds_wave = lds_base + w * 1024;
  // The next tile to request: query tile iss_qt of query head iss_h of the group, whose Q, dO and
  // workspace rows start at iss_q, iss_do, iss_ws.  Query tiles are walked from the last one down, every
  // head of the group inside a tile: the workgroups of an XCD that share a K/V head then want the same Q and
  // dO tiles at the same time whatever their first visible query is, and find them in its L2.  (Head by head
  // from the first visible tile up, 4 x 64/8 heads x 4096 causal: this kernel reads 6.8 GB from beyond the L2 and the
  // backward takes 3819 us; in this order 1.8 GB and 3669 us.)
  int iss_qt = nqt_all - 1, iss_h = 0;
  const ptrdiff_t head_bytes = (ptrdiff_t)N * ROWB;
  const ptrdiff_t wrap_bytes = -(G - 1) * head_bytes - TILEB, wrap_ws = -(G - 1) * 2 * (ptrdiff_t)p.Npad - BN;
  const char* iss_q = (const char*)p.q + (size_t)(tc.b * p.Hq + g * G) * head_bytes + (size_t)iss_qt * TILEB;
  const char* iss_do = (const char*)p.dout + (size_t)(tc.b * p.Hq + g * G) * head_bytes + (size_t)iss_qt * TILEB;
  const float* iss_ws = p.ws + (size_t)(tc.b * p.Hq + g * G) * 2 * p.Npad + (size_t)iss_qt * BN;
  const uint32_t aoff = (uint32_t)(((lane & 15) * 4 + ((lane >> 4) & 1) * p.Npad) * 4);
  // load i of that tile into ring slot `slot`: Q and dO pieces, last the workspace rows; issue_advance() goes on to
  // the tile after it
  constexpr int LPT = 2 * NLD + 1;  // loads per thread and tile
  auto issue_load = [&](int slot, int i) __attribute__((always_inline)) {
    if (i == 2 * NLD) {
      if (lane < 32) attn_lds_dma16(iss_ws, aoff, lds_base + C::AUXBASE + slot * 512);
      return;
    }
    const int it = i >> 1;
    const uint32_t off = iss_qt == nqt_all - 1 ? ld_off_r[it] : ld_off[it];
    attn_lds_dma16((i & 1) ? iss_do : iss_q, off, lds_wave + ((i & 1) ? C::T2BASE : 0) + slot * TILEB + it * NT * 16);
  };
  auto issue_advance = [&]() __attribute__((always_inline)) {
    const bool wrap = ++iss_h == G;  // back to the group's first query head, one tile down
    iss_q += wrap ? wrap_bytes : head_bytes;
    iss_do += wrap ? wrap_bytes : head_bytes;
    iss_ws += wrap ? wrap_ws : 2 * (ptrdiff_t)p.Npad;
    iss_h = wrap ? 0 : iss_h;
    iss_qt -= wrap ? 1 : 0;
  };
  auto issue_next = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < LPT; ++i) issue_load(slot, i);
    issue_advance();
  };
  issue_next(0);

  bf16x8 kf[NKK], vf[NKK];
  {
    const int row = min(krow, N - 1);
    const char* ks = (const char*)p.k + koff + (size_t)row * ROWB + h * 16;
    const char* vs = (const char*)p.v + koff + (size_t)row * ROWB + h * 16;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      kf[kk] = *(const bf16x8*)(ks + kk * 32);
      vf[kk] = *(const bf16x8*)(vs + kk * 32);
    }
  }
  if (nt > 1) issue_next(1);
  if (nt > 2) issue_next(2);

  f32x16 acc_dv[NCB], acc_dk[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc_dv[cb][r] = acc_dk[cb][r] = 0.f;
  auto grads_settled = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) asm volatile("s_nop 15" : "+a"(acc_dv[cb]), "+a"(acc_dk[cb]));
  };
  grads_settled();

  // LDS read addresses.  Inside the ring every offset (slot, 32-row half, 16-row group) is a
  // compile-time immediate of the read instruction; the second tensor's slots lie beyond the
  // immediate's range and get address registers of their own.
  uint32_t raddr[2][NKK];
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) {
    raddr[0][kk] = qg * SUBB + ki * ROWB + (((2 * kk + h) ^ swz_rt<ROWB>(ki)) << 4);
    raddr[1][kk] = raddr[0][kk] + C::T2BASE;
    asm volatile("" : "+v"(raddr[1][kk]));
  }
  uint32_t taddr[2][NCB][2];
  {
    const int s = lane & 15, chalf = (lane >> 4) & 1;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int row = 8 * e + 4 * h + (s >> 2);
        const int chunk = cb * 4 + chalf * 2 + ((s & 3) >> 1);
        taddr[0][cb][e] = qg * SUBB + row * ROWB + ((chunk ^ swz_rt<ROWB>(row)) << 4) + ((s & 1) << 3);
        taddr[1][cb][e] = taddr[0][cb][e] + C::T2BASE;
        asm volatile("" : "+v"(taddr[1][cb][e]));
      }
  }
  const uint32_t auxaddr = C::AUXBASE + qg * 128 + 16 * h;
  // `t2` selects the tensor (0: Q slots, 1: dO slots), `off` is the block's offset inside them
  auto row_operand = [&](int t2, int off, int kk) __attribute__((always_inline)) { return *(LDS_AS u32x4*)(smem + raddr[t2][kk] + off); };
  auto tr_operand = [&](int t2, int off, int cb, int kc) __attribute__((always_inline)) {
    const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(smem + taddr[t2][cb][0] + off + kc * 16 * ROWB));
    const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(smem + taddr[t2][cb][1] + off + kc * 16 * ROWB));
    s16x8 av;
    av[0] = v0[0]; av[1] = v0[1]; av[2] = v0[2]; av[3] = v0[3];
    av[4] = v1[0]; av[5] = v1[1]; av[6] = v1[2]; av[7] = v1[3];
    return __builtin_bit_cast(u32x4, av);
  };
  // operand of gradient product i of the block at `off`: dV^T += dO^T P (even i), dK^T += Q^T dS (odd i)
  auto grad_operand = [&](int off, int i) __attribute__((always_inline)) { return tr_operand((i & 1) ? 0 : 1, off, (i >> 1) % NCB, (i >> 1) / NCB); };
  // operand of score product i of the block at `off`: S += Q K^T (even i), dP += dO V^T (odd i)
  auto score_operand = [&](int off, int i) __attribute__((always_inline)) { return row_operand(i & 1, off, i >> 1); };
  // The gradients are accumulated by assembly statements that pin them to accumulation registers, which
  // the compiler's wait-state insertion does not look into.  A step packs its last P and dS in its last slot and the next step
  // reads them two slots (d = 64) or more into it: behind at least two products and their operand reads, also over the back edge of the
  // loop, where the compiler must place no move of them (a test reads the listing).  Nothing but these products touches the
  // accumulators in a step; behind the loop, `copied` covers operands that were just moved (2 wait states) and grads_settled()
  // the readers of the result (8 passes: 12).
  auto grad_mfma = [&](int i, u32x4 o, const u32x4 (&pp)[2], const u32x4 (&pd)[2], auto copied) __attribute__((always_inline)) {
    const int cb = (i >> 1) % NCB, kc = (i >> 1) / NCB;
    if constexpr (decltype(copied)::value) {
      if (i & 1) asm volatile("s_nop 3\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc_dk[cb]) : "v"(o), "v"(pd[kc]));
      else asm volatile("s_nop 3\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc_dv[cb]) : "v"(o), "v"(pp[kc]));
      return;
    }
    if (i & 1) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc_dk[cb]) : "v"(o), "v"(pd[kc]));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc_dv[cb]) : "v"(o), "v"(pp[kc]));
  };

  const float c = p.scale_log2;

  u32x4 pre[RA];  // operands of the next step's first RA MFMAs
  // slots between the loads of a tile, slot of the first one (QS = 2 waits for them one step later: as early as they go)
  constexpr int LGAP = QS == 1 ? NM / LPT : 1, LFIRST = QS == 1 ? NM - LPT * LGAP : 0;
  // One step.  (s_in, dp_in): finished scores of the block at CUR whose first query row is q0b;
  // (s_out, dp_out) <- scores of the block at NEXT; (pp_out, pd_out) <- P and dS of the block at
  // CUR; (pp_acc, pd_acc): P and dS of the block at PREV, multiplied into dV and dK.  PREV, CUR,
  // NEXT are compile-time offsets inside the ring, AUX the offset of CUR's statistics.
  auto step = [&](f32x16& s_in, f32x16& dp_in, f32x16& s_out, f32x16& dp_out, u32x4 (&pp_out)[2], u32x4 (&pd_out)[2],
                  const u32x4 (&pp_acc)[2], const u32x4 (&pd_acc)[2], auto PREV, auto CUR, auto NEXT, auto AUX, auto AUXN,
                  int q0b, bool load, auto LSLOT) __attribute__((always_inline)) {
    constexpr int prev = decltype(PREV)::value, cur = decltype(CUR)::value, next = decltype(NEXT)::value;
    constexpr int auxo = decltype(AUX)::value, auxn = decltype(AUXN)::value;
    u32x4 op[NM];
    f32x16 dn;  // -delta of the rows of the block at NEXT: dP starts from it
#pragma unroll
    for (int m = 0; m < RA; ++m) op[m] = pre[m];
    f32x4 l4[4];
    float x[16], e[16], f[16];
    __builtin_amdgcn_sched_barrier(0);
    auto one_slot = [&](auto slot_tag) __attribute__((always_inline)) {
      constexpr int m = decltype(slot_tag)::value;
      // LDS reads: the operand of slot m + RA, and the statistics of the rows handled six slots on
      {
        constexpr int t = C::read_target(m);
        if constexpr (t < NM) op[t] = C::is_score(t) ? score_operand(next, C::index(t)) : grad_operand(prev, C::index(t));
        else pre[t - NM] = grad_operand(cur, t - NM);
      }
#pragma unroll
      for (int a = 0; a < 4; ++a)
        if (C::dslot(a) == m) {
          const f32x4 t = *(const LDS_AS f32x4*)(smem + auxaddr + auxn + 256 + 32 * a);
#pragma unroll
          for (int r = 0; r < 4; ++r) dn[4 * a + r] = t[r];
        }
#pragma unroll
      for (int a = 0; a < 4; ++a)
        if (C::aslot(a) == m) {
          l4[a] = *(const LDS_AS f32x4*)(smem + auxaddr + auxo + 32 * a);
        }
      // the matrix product of this slot
      const int i = C::index(m);
      if (C::is_score(m)) {
        if (i == 0 || i == 1) {
#pragma unroll
          for (int r = 0; r < 16; ++r) (i ? dp_out : s_out)[r] = i ? dn[r] : 0.f;
        }
        if (i & 1) dp_out = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, op[m]), vf[i >> 1], dp_out, 0, 0, 0);
        else s_out = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, op[m]), kf[i >> 1], s_out, 0, 0, 0);
      } else {
        grad_mfma(i, op[m], pp_acc, pd_acc, std::false_type{});
      }
      // the next tile's loads, one at a time: all of them behind the barrier keep the wave from issuing products until
      // the address unit has taken them
      if constexpr (decltype(LSLOT)::value >= 0) {
        if constexpr (m >= LFIRST && (m - LFIRST) % LGAP == 0 && (m - LFIRST) / LGAP < LPT) {
          if (load) issue_load(decltype(LSLOT)::value, (m - LFIRST) / LGAP);
        }
      }
      // causal diagonal: -inf scores for the queries before this lane's key (wave-uniform branch)
      if (CAUSAL && m == C::VP0 - 1 && q0b < wk0 + 31) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (q0b + 8 * (r >> 2) + 4 * h + (r & 3) < krow) s_in[r] = -INFINITY;
      }
      // vector work of row r, one link of its chain per slot: P = exp2(s c - lse2), dS = P (dP - delta), packs
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (C::vslot(r) - 1 == m) x[r] = __builtin_fmaf(s_in[r], c, -l4[r >> 2][r & 3]);
        if (C::vslot(r) == m) e[r] = __builtin_amdgcn_exp2f(x[r]);
        if (C::vslot(r) + 1 == m || (m == NM - 1 && C::vslot(r) + 1 > m)) {
          f[r] = e[r] * dp_in[r];
          if (r & 1) {
            pp_out[r >> 3][(r >> 1) & 3] = pack_bf16(e[r - 1], e[r]);
            pd_out[r >> 3][(r >> 1) & 3] = pack_bf16(f[r - 1], f[r]);
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    for_each_slot(one_slot, std::make_integer_sequence<int, NM>{});
    asm volatile("" : "+v"(pp_out[0]), "+v"(pp_out[1]), "+v"(pd_out[0]), "+v"(pd_out[1]));  // (made here, not put off to where they are read)
  };

  // the block "before the first" lives in the last half of slot 3 (QS = 2: a wave's half of it):
  // zeros, so that its gradient products (with P = dS = 0) add exact zeros
  constexpr int BEFORE = 3 * TILEB + (QS == 1 ? SUBB : 0);
  {
    const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < (4 * TILEB - BEFORE) / (NT * 16); ++i) {
      *(LDS_AS u32x4*)(smem + BEFORE + (i * NT + tid) * 16) = z;
      *(LDS_AS u32x4*)(smem + C::T2BASE + BEFORE + (i * NT + tid) * 16) = z;
    }
  }
  if (nt > 2) ATTN_WAIT_VMCNT(2 * LPT);
  else if (nt > 1) ATTN_WAIT_VMCNT(LPT);
  else ATTN_WAIT_VMCNT(0);
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) asm volatile("" : "+a"(kf[kk]), "+a"(vf[kk]));
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the zero fill is written
  attn_wg_barrier();

  // prologue: scores of block 0
  f32x16 sa, dpa, sb, dpb;
  u32x4 ppa[2], pda[2], ppb[2], pdb[2];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    sa[r] = 0.f;
    dpa[r] = *(const LDS_AS float*)(smem + auxaddr + 256 + 32 * (r >> 2) + 4 * (r & 3));
  }
#pragma unroll
  for (int kk = 0; kk < NKK; ++kk) {
    sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, row_operand(0, 0, kk)), kf[kk], sa, 0, 0, 0);
    dpa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, row_operand(1, 0, kk)), vf[kk], dpa, 0, 0, 0);
  }
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    ppb[t] = pdb[t] = u32x4{0u, 0u, 0u, 0u};
    asm volatile("s_nop 1" : "+v"(ppb[t]), "+v"(pdb[t]));  // (not to be made again in front of the first product)
  }
#pragma unroll
  for (int m = 0; m < RA; ++m) pre[m] = grad_operand(BEFORE, m);

  int qt = nqt_all - 1, qh = 0;  // query tile and head of tile j
  auto next_qt = [&]() __attribute__((always_inline)) {
    if (++qh == G) {
      qh = 0;
      --qt;
    }
  };
  // QS = 2: tiles 0, 1 and 2 are requested up front.  (Behind a statement, so that no step is split off the loop: the
  // copies that takes would move the accumulators.)
  int first_load = 1;
  asm volatile("" : "+s"(first_load));
  // tile j lives in slot j % 4 = S
  auto tile = [&](auto S, int j) __attribute__((always_inline)) {
    constexpr int s = decltype(S)::value;
    if constexpr (QS == 2) {
      // one step per tile; in front of it: tile j+1 has landed, every wave is done with tile j-2
      // (tiles 0, 1 and 2 are requested by the prologue, later ones one step ahead)
      ATTN_WAIT_VMCNT(0);
      attn_wg_barrier();
      const bool load = j >= first_load && j + 2 < nt;
      constexpr int o = s * TILEB, op = ((s + 3) & 3) * TILEB, on = ((s + 1) & 3) * TILEB;
      const int q0b = qt * BN + qg * 32;
      if constexpr (s & 1) step(sb, dpb, sa, dpa, ppb, pdb, ppa, pda, ic<op>{}, ic<o>{}, ic<on>{}, ic<s * 512>{}, ic<((s + 1) & 3) * 512>{}, q0b, load, ic<(s + 2) & 3>{});
      else step(sa, dpa, sb, dpb, ppa, pda, ppb, pdb, ic<op>{}, ic<o>{}, ic<on>{}, ic<s * 512>{}, ic<((s + 1) & 3) * 512>{}, q0b, load, ic<(s + 2) & 3>{});
      if (load) issue_advance();
      next_qt();
      return;
    }
    constexpr int b0 = s * TILEB, b1 = b0 + SUBB, bp = ((s + 3) & 3) * TILEB + SUBB, bn = ((s + 1) & 3) * TILEB;
    const int q0b = qt * BN;
    step(sa, dpa, sb, dpb, ppa, pda, ppb, pdb, ic<bp>{}, ic<b0>{}, ic<b1>{}, ic<s * 512>{}, ic<s * 512 + 128>{}, q0b, false, ic<-1>{});
    // tile j+1 has landed (the loads of tile j+2 stay in flight); every wave is done with tile j-1
    if (j + 2 < nt) ATTN_WAIT_VMCNT(LPT);
    else ATTN_WAIT_VMCNT(0);
    attn_wg_barrier();
    const bool load = j + 3 < nt;
    step(sb, dpb, sa, dpa, ppb, pdb, ppa, pda, ic<b0>{}, ic<b1>{}, ic<bn>{}, ic<s * 512 + 128>{}, ic<((s + 1) & 3) * 512>{}, q0b + 32, load, ic<(s + 3) & 3>{});
    if (load) issue_advance();
    next_qt();
  };
  int j = 0;
  for (; j + 4 <= nt; j += 4) {
    tile(ic<0>{}, j);
    tile(ic<1>{}, j + 1);
    tile(ic<2>{}, j + 2);
    tile(ic<3>{}, j + 3);
  }
  if (j < nt) {
    tile(ic<0>{}, j);
    if (j + 1 < nt) {
      tile(ic<1>{}, j + 1);
      if (j + 2 < nt) tile(ic<2>{}, j + 2);
    }
  }
  // epilogue: the gradient products of the last block (its first RA operands are already here)
  if constexpr (QS == 1) {
    const int last = ((nt - 1) & 3) * TILEB + SUBB;
#pragma unroll
    for (int i = RA; i < C::NG; ++i) grad_mfma(i, grad_operand(last, i), ppb, pdb, std::true_type{});
#pragma unroll
    for (int i = 0; i < RA; ++i) grad_mfma(i, pre[i], ppb, pdb, std::true_type{});
    grads_settled();
    const size_t roff = koff + (size_t)min(krow, N - 1) * ROWB;
    store_transposed<NCB>(acc_dv, 1.0f, (char*)p.dv + roff, h, krow < N);
    store_transposed<NCB>(acc_dk, p.scale, (char*)p.dk + roff, h, krow < N);
  } else {
    const int last = ((nt - 1) & 3) * TILEB;
    const bool odd = ((nt - 1) & 1) != 0;  // (the parity of the last step says which registers hold P and dS)
    if (!odd) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        ppb[t] = ppa[t];
        pdb[t] = pda[t];
      }
    }
#pragma unroll
    for (int i = RA; i < C::NG; ++i) grad_mfma(i, grad_operand(last, i), ppb, pdb, std::true_type{});
#pragma unroll
    for (int i = 0; i < RA; ++i) grad_mfma(i, pre[i], ppb, pdb, std::true_type{});
    grads_settled();
    const size_t roff = koff + (size_t)min(krow, N - 1) * ROWB;
    __syncthreads();  // no wave reads the ring any more
    LDS_AS f32x4* const give = (LDS_AS f32x4*)smem + ((qg ^ 1) * NKW + w % NKW) * (NCB * 4) * 64 + lane;
    LDS_AS const f32x4* const take = (LDS_AS const f32x4*)smem + (qg * NKW + w % NKW) * (NCB * 4) * 64 + lane;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      const f32x16 other = qg ? acc_dv[cb] : acc_dk[cb];
      if (qg) acc_dv[cb] = acc_dk[cb];
#pragma unroll
      for (int a = 0; a < 4; ++a) give[(cb * 4 + a) * 64] = f32x4{other[4 * a], other[4 * a + 1], other[4 * a + 2], other[4 * a + 3]};
    }
    __syncthreads();
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const f32x4 o = take[(cb * 4 + a) * 64];
#pragma unroll
        for (int r = 0; r < 4; ++r) acc_dv[cb][4 * a + r] += o[r];
      }
    store_transposed<NCB>(acc_dv, qg ? p.scale : 1.0f, (char*)(qg ? p.dk : p.dv) + roff, h, krow < N);
  }
}

}  // namespace

// The forms, and which of them a launch takes: the cheapest by what attn_equal_us (not causal) and attn_causal_us make of the fitted
// costs below.  Whole backward passes in which only that kernel changes, us, heads x N (2953 random shapes, N 20 .. 6000, all forms of
// each timed in turn):
//   dQ, 128 / 64 / 256 rows: the wide form is ahead where it saves a round over the CUs or where K and V weigh more than the chain
//     d = 128  144/36 x 146 46.0 / 42.4 / 38.0; 256/128 x 133 38.2 / 43.8 / 31.9; causal 20 x 3449 327 / 304 / 309; 60/30 x 2179 364 / 396 / 421;
//              2 x 656 41 / 38 / 49
//     d = 64   80 x 22 9.1 / 9.2 / 8.7; causal 512/128 x 132 34.1 / 38.9 / 30.7; 128/64 x 522 48.3 / 47.0 / 41.8; 384/192 x 23 13.4 / 13.4 / 14.2 (no fewer
//              workgroups, and more than the CUs: not wide)
//     the choice is 0.1 % slower than the fastest form on average, at worst 3 % (non-causal), 7 % (causal); without the wide form
//     0.6 - 1.2 % and 21 %
//   dK/dV, 128 / 64 keys (at d = 64 two of the split form's workgroups share a CU, one of the whole form's)
//     d = 128  12 x 1000 75 / 67; 16 x 2048 140 / 151; causal 64 x 2048 260 / 292; 60/30 x 2179 364 / 311; 256/32 x 4096 3491 / 3687
//     d = 64   384/96 x 297 72.1 / 53.9; 36/18 x 1994 198 / 165; causal 24/12 x 2412 112 / 90; 36 x 925 37.1 / 45.6; 72 x 490 26.3 / 29.8; 1 x 59 9.8 / 10.2
//     the choice is 0.1 % slower than the faster form on average, at worst 4 %
int attn_bwd_launch_bf16(const AttnBwdParams& p, int d, hipStream_t stream) {
  auto launch = [&](auto dtag, auto causal_tag) {
    constexpr int D = decltype(dtag)::value;
    constexpr bool CAUSAL = decltype(causal_tag)::value;
    const double blocks = (p.N + 31) / 32;  // 32-row blocks of a head
    const int G = p.Hq / p.Hkv;
    auto tiles = [&](int heads, int rows) { return (long long)p.B * heads * ((p.N + rows - 1) / rows); };
    // workgroups of `rows` queries / keys, of whose blocks a wave takes `part`
    auto us_q = [&](const AttnFormCost& c, int rows, int slots, double part) {
      const long long n = tiles(p.Hq, rows);
      if (!CAUSAL) return attn_equal_us(c, n, slots, part * blocks);
      const int T = (p.N + rows - 1) / rows;
      const double tile = part * (rows / 32);
      return attn_causal_us(c, attn_tile_map_make(p.B, p.Hq, p.Hkv, T, 1), n, slots, T * tile, tile, part * blocks);
    };
    auto us_k = [&](const AttnFormCost& c, int rows, int slots, double part) {
      const long long n = tiles(p.Hkv, rows);
      const double all = part * G * blocks;
      if (!CAUSAL) return attn_equal_us(c, n, slots, all);
      return attn_causal_us(c, attn_tile_map_make(p.B, p.Hkv, p.Hkv, (p.N + rows - 1) / rows, 1), n, slots, all, part * G * (rows / 32), all);
    };
    // ---- dQ: workgroups of 128 queries, of 64 with split keys, or wide ones of 256
    static constexpr AttnFormCost cost_q[2][2][3] = {  // [d = 128][causal][128, 64, 256 rows]
        {{{-0.04, 1.84, 0.276, 0.250, 0.49}, {-0.80, 3.22, 0.229, 0.410, 0.61}, {0.53, 0.66, 0.605, 0.570, 0.42}},
         {{0.22, 3.14, 0.177, 0.049, 0.0}, {0.16, 3.52, 0.117, 0.156, 0.0}, {-0.30, 3.23, 0.476, 0.000, 0.0}}},
        {{{-0.01, 3.85, 0.517, 0.268, 1.04}, {0.02, 4.52, 0.685, 0.299, 1.32}, {0.08, 3.16, 1.056, 0.425, 0.96}},
         {{-0.06, 5.50, 0.415, 0.246, 0.0}, {0.30, 5.69, 0.550, 0.359, 0.0}, {0.10, 4.83, 0.906, 0.445, 0.0}}}};
    const AttnFormCost* const cq = cost_q[D == 128][CAUSAL];
    constexpr int slots = D == 128 ? 1 : 2;
    const double us_128 = us_q(cq[0], 128, slots, 1.0);
    const double us_64 = tiles(p.Hq, 64) <= 131072 ? us_q(cq[1], 64, slots, 0.5) : INFINITY;
    double us_256 = us_q(cq[2], 256, slots, 1.0);
    if (D == 64 && CAUSAL && p.N <= 128 && tiles(p.Hq, 256) > 256) us_256 = INFINITY;
    const int rows_q = us_256 < us_128 && us_256 < us_64 ? 256 : us_64 < us_128 ? 64 : 128;
    // ---- dK/dV: workgroups of 128 keys, or of 64 with split queries (which a head of two blocks or fewer gains nothing from)
    bool split_k = false;
    const double steps_k = blocks * G;
    if (tiles(p.Hkv, 128) <= 65536 && (D == 64 || CAUSAL || steps_k >= 4.0) && !(CAUSAL && steps_k < 3.0 && G == 1)) {
      static constexpr AttnFormCost cost_k[2][2][2] = {  // [d = 128][causal][128, 64 keys]
          {{{-0.09, 2.99, 0.420, 0.162, 0.93}, {0.26, 3.38, 0.446, 0.348, 0.35}}, {{1.30, 5.24, 0.437, 0.159, 0.0}, {-1.52, 7.62, 0.477, 0.131, 0.0}}},
          {{{-0.13, 4.19, 0.634, 0.288, 0.99}, {0.05, 5.11, 0.688, 0.292, 1.12}}, {{-0.17, 5.88, 0.618, 0.278, 0.0}, {0.02, 6.25, 0.697, 0.287, 0.0}}}};
      const AttnFormCost* const ck = cost_k[D == 128][CAUSAL];
      split_k = us_k(ck[1], 64, D == 64 ? 2 : 1, 0.5) < us_k(ck[0], 128, 1, 1.0);
    }
    const long long grid_q = tiles(p.Hq, rows_q), grid_k = tiles(p.Hkv, split_k ? 64 : 128);
    const int threads_q = rows_q == 256 ? 512 : 256;
    if (grid_q * threads_q > 0xffffffffll || grid_k * 256 > 0xffffffffll) return -1;  // beyond what a launch holds
    AttnBwdParams q = p;
    q.T = (p.N + rows_q - 1) / rows_q;
    const void* const dq = rows_q == 256  ? (const void*)attn_bwd_dq_wide_kernel<D, CAUSAL>
                           : rows_q == 64 ? (const void*)attn_bwd_dq_kernel<D, CAUSAL, 2>
                                          : (const void*)attn_bwd_dq_kernel<D, CAUSAL, 1>;
    void* args[] = {&q};
    if (hipLaunchKernel(dq, dim3((unsigned)grid_q), dim3(threads_q), args, 0, stream) != hipSuccess) {
      const int err = (int)hipGetLastError();
      return err ? err : -1;  // (dK/dV would read rows that nothing has written)
    }
    if (split_k) hipLaunchKernelGGL((attn_bwd_dkv_pipe_kernel<D, CAUSAL, 2>), dim3((unsigned)grid_k), dim3(256), 0, stream, q);
    else hipLaunchKernelGGL((attn_bwd_dkv_pipe_kernel<D, CAUSAL, 1>), dim3((unsigned)grid_k), dim3(256), 0, stream, q);
    return (int)hipGetLastError();
  };
  auto by_causal = [&](auto dtag) { return p.causal ? launch(dtag, std::true_type{}) : launch(dtag, std::false_type{}); };
  return d == 128 ? by_causal(ic<128>{}) : d == 64 ? by_causal(ic<64>{}) : -1;
}

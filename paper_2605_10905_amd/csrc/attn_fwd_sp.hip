// Fused attention forward for gfx950: the software-pipelined kernel, for bf16 inputs and for
// fp8 (e4m3) inputs.
//
// Mathematics (paper section 6.1 for the phases, appendix C.3 for the streaming-softmax state and
// the overlap of one block's QK^T product with the previous block's PV product): both products
// are taken transposed, S^T = K Q^T and O^T += V^T P^T, on the 32x32 MFMA shapes, so that a lane
// holds ONE query column and many keys: row sums are per-lane partial sums, the rescale factor
// is one scalar per lane, and the exponentiated, packed S^T accumulator IS the B operand of the
// second product (no shuffle, no LDS round trip).
//
// Orchestration.  All 8 waves of a workgroup run the same instruction stream, and that stream
// is pipelined over 32-key blocks so that the matrix pipe and the vector pipe are fed from the
// SAME wave at the same time (measured on gfx950: a wave that issues only MFMAs and a sibling
// that issues only VALU work delay each other at the shared issue port; one MFMA followed by
// three to five independent VALU instructions from the same wave is nearly free).  In the step
// that handles block u a wave
//     * exponentiates block u            (VALU:  P(u)   = exp2(c S(u) - m))
//     * computes the scores of block u+1 (MFMA:  S(u+1) = K(u+1) Q^T)
//     * accumulates block u-1            (MFMA:  O^T   += V(u-1)^T P(u-1)^T)
// The three streams are independent inside a step, which is laid out by hand in fenced slots of one MFMA each, with its
// share of the vector work and the LDS reads of the operand a few MFMAs ahead.
//
// K/V streaming (the producer role).  Block u+1 of K and block u-1 of V travel together:
// "bundle" b holds key tile b+1 and value tile b (64 keys each) and is consumed by exactly one
// loop iteration, so a three-slot LDS ring with direct-to-LDS loads issued two bundles ahead
// needs one workgroup barrier per 64 keys: it is both the "full" signal of bundle b+1 and the
// "empty" signal of bundle b-1 (stage = b mod 3).  The barrier sits between the two 32-key steps
// of an iteration so that the first K operands of the next iteration can be read one step
// early; the loads into the slot it frees are issued one at a time between the slots of the
// iteration's second step, never in a burst that keeps every wave off the matrix pipe at once.
//
// No block maximum is taken on the common path: exponentials are computed against the current
// reference maximum, and only when a lane's partial row sum comes out large (or not a number,
// as on the very first block) is the true block maximum taken, the reference raised, the
// accumulator rescaled and the block redone (exact: any reference is valid for the streaming
// softmax as long as nothing overflows).
//
// fp8 inputs (FP8 = true).  S^T = K Q^T is taken directly on the e4m3 bytes with the 32x32x64
// f8f6f4 MFMA (two MFMAs per 32-key block instead of eight bf16 ones; K tiles of half the size go
// straight from memory into the ring).  P loses too much when it is rounded to e4m3 (a single
// term measures above the 2 % Frobenius bound), so P stays bf16 and V is converted e4m3 -> bf16,
// exactly, once per tile on arrival: the fp8 value tile lands in a two-slot staging area one
// bundle early, and every thread converts the 16 bytes it staged itself with the packed
// conversion and writes them, swizzled, into the ring slot the barrier has just freed.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "attn_device.h"
#include "attn_kernels.h"
#include "tile_map.h"

namespace {

typedef __attribute__((ext_vector_type(8))) int i32x8;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr float kTau = 8.0f;
constexpr float kSumLimit = 65536.0f;  // a lane's 16-term partial sum above this redoes the block with a raised reference
// A row sum above this (of N probabilities it stays below 2^36) holds overflow: exponents are taken against the
// reference mx * c as rounded, and what that rounding leaves reaches 64 at about -2^31 and 128, i.e. infinity, at
// -2^32 (keys hidden by large negative scores).  Such a state must not outlive the reference that a visible key
// brings (infinity times alpha = 0): the first block is redone with its exponents bounded, as every redone block
// of the pipelined steps is, and the other blocks' l and O are dropped where alpha is zero.  Bounding every
// block behind a flag or by v_minimum3 cost launches of short heads 2 - 4 % (384 heads of 133: 19.5 -> 19.9 us and
// more); as it is they take 19.6, and 2 heads of 256, the smallest launch, 6.3 -> 6.5.
constexpr float kSumDrop = 1.8446744073709552e19f;  // 2^64
// Reference of a row that has seen no key: finite, so that a block whose scores are all -inf gives
// probabilities of zero (-inf + FLT_MAX) and not NaN, and far enough down that the first real score replaces it.
constexpr float kNoRef = -3.4028234663852886e38f;

template <int V>
using ic = std::integral_constant<int, V>;

enum { kWhole = 1, kSplit = 2, kPair = 3 };  // FORM of attn_fwd_sp_kernel
template <int D>
constexpr int kPairSlots = D == 64 ? 3 : 2;  // paired workgroups that share a CU

template <class F, int... M>
__device__ __forceinline__ void for_each_slot(F f, std::integer_sequence<int, M...>) {
  (f(ic<M>{}), ...);
}

// MODE says where a workgroup's query tiles come from.
//   0: one tile per workgroup (the tile the workgroup id maps to).
//   1: the launch has one workgroup per CU, and each takes tiles from a queue in device memory until
//      it is drained.  The queue is 8 counters, one per XCD list of the static tile order (a tile
//      index wg belongs to list wg % 8, the XCD the static launch would run it on, and lists are
//      consumed heaviest tile first); a workgroup serves the list of the XCD it was dispatched to
//      and, when that is empty, the lists after it, so every tile is taken exactly once whatever
//      the dispatch order was.  This is the software stand-in for the paper's cluster launch
//      control (section 4.2): dynamic assignment of tiles to resident workgroups.
//   2: one workgroup per CU again, but each walks a list fixed by arithmetic: the tiles of its XCD's
//      list are dealt to the XCD's workgroups in boustrophedon order (first to last, then last to
//      first, ...), which balances lists sorted by weight (causal inputs) without a queue, without
//      atomics and without any memory the library would have to own.
// In modes 1 and 2 consecutive tiles of a workgroup overlap at the seam: the next tile's first
// loads are requested as soon as every wave has left the ring, before the finished tile's output
// is packed, and the packed output is stored only when the next tile's loads have been waited
// for (loads and stores share one counter per wave, so a store in between would be waited for
// as well).
//
// KS = 2 (bf16, MODE 0), for launches that leave CUs idle: a workgroup owns 128 queries, and the waves
// w and w + 4 share 32 of them: one takes the first 32-key block of every 64-key tile, the other the
// second, each with a streaming softmax of its own, merged through LDS at the end.  Twice the
// workgroups, half the serial chain.  An iteration is then ONE step: bundle b holds key tile b+2 and
// value tile b, the barrier that publishes bundle b+1 and frees the slot of bundle b-1 sits in front of
// the step, and the ring has four slots so that a bundle is requested three steps ahead.  Q travels
// through LDS as well: with no load the compiler knows of, the waits are exact, and the first scores
// need only Q and key tiles 0 and 1 to have arrived, not bundles 0 and 1 requested behind them.
// FORM = kPair (bf16, MODE 0 and 1): four waves own 128 queries, key tiles of 32 and otherwise the one-step iterations of the split
// form.  The ring is 64 KB (d = 64: 32), so two (three) such workgroups share a CU, and one's first loads, first
// block, diagonal and stores run beside the other's steps.  By itself a step takes it 0.56 us (d = 128), beside another one 0.78
// (stamps of a full launch at a power-limited clock; pair_pays holds fits to whole launches, not step times).  Its results are the whole form's
// but where a row's maximum rises by more than 8 in the last block that only one of them takes through the pipelined step (the
// whole form runs an even number of blocks there): that block's probabilities are then rounded against another reference.  (The whole
// form's count here would make the bytes equal and costs paired launches 1 - 2 %.)
template <int D, bool CAUSAL, int MODE, bool FP8, int FORM = kWhole>
__global__ void __launch_bounds__(FORM == kPair ? 256 : 512, 2) attn_fwd_sp_kernel(const AttnParams p) {
  static_assert(!FP8 || (D == 128 && MODE != 1), "fp8 inputs: head dimension 128, no queue launch");
  static_assert(FORM == kWhole || !FP8, "split keys and paired workgroups: bf16");
  static_assert(FORM == kWhole || MODE == 0 || (FORM == kPair && MODE == 1), "split keys: one tile per workgroup; paired workgroups: also from the queue");
  constexpr int KS = FORM == kSplit ? 2 : 1;  // waves that share a query block
  constexpr int BN = FORM == kPair ? 32 : 64, NWAVES = FORM == kPair ? 4 : 8, NQW = NWAVES / KS, BM = NQW * 32, NT = NWAVES * 64;
  constexpr int NCB = D / 32;                // 32-row blocks of O^T
  constexpr int ROWB = D * 2;                // bytes per bf16 row: V in the ring, O
  constexpr int INB = FP8 ? D : 2 * D;       // bytes per input row (q, k, v in memory; K rows in the ring)
  constexpr int NKQ = FP8 ? D / 64 : D / 16; // MFMA k-steps of S^T = K Q^T
  constexpr int KTILEB = BN * INB;           // bytes per K tile in the ring
  constexpr int KSUBB = 32 * INB;            // bytes per 32-key block of it
  constexpr int TILEB = BN * ROWB;           // bytes per bf16 V tile in the ring
  constexpr int SUBB = 32 * ROWB;            // bytes per 32-key block of it
  constexpr int NSLOT = FORM == kWhole ? 3 : 4;     // ring depth: bundles are requested NSLOT-1 ahead
  constexpr int VBASE = NSLOT * KTILEB;      // K parts of the slots first, then the V parts
  constexpr int STGBASE = VBASE + NSLOT * TILEB;  // fp8: two staging slots of one e4m3 V tile each
  constexpr int STGTILE = BN * INB;
  constexpr int LDSB = FP8 ? STGBASE + 2 * STGTILE : STGBASE;
  constexpr int NCHI = INB / 16;             // 16-byte chunks per input row
  constexpr int NLD = BN * NCHI / NT;        // direct-to-LDS loads per thread per tile
  constexpr int QKR = FP8 ? 2 : 1;           // 128-bit LDS reads per K fragment
#ifndef ATTN_RA
#define ATTN_RA 4
#endif
  constexpr int RA = ATTN_RA;                // operands are read from LDS this many MFMAs ahead
  constexpr int NM = NKQ + 2 * NCB;          // MFMAs per 32-key step
  constexpr int STRIDE = NM / NKQ;           // MFMA m is a score product iff m % STRIDE == 0
  static_assert(BN * NCHI % NT == 0 && NLD >= 1 && (!FP8 || NLD == 1), "tile must divide evenly over the workgroup");
  static_assert(NM % NKQ == 0 && RA >= 2 && RA <= NM, "score products evenly spaced; read-ahead within a step");
  static_assert((NSLOT - 1) * TILEB + SUBB + 16 * ROWB < 65536, "ring offsets must fit the 16-bit LDS immediate");

  __shared__ __attribute__((aligned(1024))) char smem_raw[LDSB];
  LDS_AS char* const smem = (LDS_AS char*)smem_raw;
  __shared__ int next_tile;

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int qi = lane & 31;  // query column within the wave's 32-query block
  const int h = lane >> 5;   // which half of the k-slots / accumulator rows this lane holds
  const int kg = KS == 1 ? 0 : w / NQW;  // KS = 2: which key block of a tile this wave takes

  // ---- the tile this workgroup works on (re-assigned at every seam in modes 1 and 2) ------------
  const int N = p.N;
  const int G = p.Hq / p.Hkv;
  int tile_b, tile_hq;              // batch and query head
  int q0, wq0;                      // first query row of the tile / of this wave
  bool wave_valid;
  const char *qhead, *khead, *vhead;
  int kv_end, nt;                   // keys the workgroup visits; 64-key tiles = bundles
  int qrow, limit, wlast;           // this lane's query row, its last visible key, the wave's last row
  auto set_tile = [&](int wg) __attribute__((always_inline)) {
    const AttnTileCoord tc = attn_tile_coord_map(wg, p.map);
    tile_b = tc.b;
    tile_hq = tc.hq;
    const int hk = tc.hq / G;
    q0 = tc.t * BM;
    wq0 = q0 + (KS == 1 ? w : w % NQW) * 32;
    wave_valid = wq0 < N;
    qhead = (const char*)p.q + ((size_t)(tc.b * p.Hq + tc.hq) * N) * INB;
    khead = (const char*)p.k + ((size_t)(tc.b * p.Hkv + hk) * N) * INB;
    vhead = (const char*)p.v + ((size_t)(tc.b * p.Hkv + hk) * N) * INB;
    kv_end = CAUSAL ? min(N, q0 + BM) : N;
    nt = (kv_end + BN - 1) / BN;
    qrow = wq0 + qi;
    limit = CAUSAL ? min(qrow, N - 1) : (N - 1);
    wlast = wq0 + 31;
  };
  // Next tile index of this workgroup, -1 when there is none.  Every thread calls it; in mode 1
  // it contains the barrier after which no wave reads the ring of the finished tile any more.
  int lists_tried = 0;  // mode 1, thread 0 only
  int round = 0;        // mode 2: how many tiles this workgroup has taken
  auto next_tile_index = [&]() __attribute__((always_inline)) {
    if constexpr (MODE == 1) {
      if (tid == 0) {
        int t = -1;
        while (lists_tried < 8) {
          const int x = (blockIdx.x + lists_tried) & 7;
          const int s = atomicAdd(p.queue + x * 32, 1);
          if (s * 8 + x < p.total) {
            t = s * 8 + x;
            break;
          }
          ++lists_tried;  // that list is drained (its counter keeps growing, which is harmless)
        }
        next_tile = t;
      }
      __syncthreads();  // also: every wave is done with the LDS ring of the previous tile
      const int wg = __builtin_amdgcn_readfirstlane(next_tile);
      __syncthreads();
      return wg;
    } else {
      // the grid is a multiple of 8 when the tile order has 8 lists (one per XCD), any size otherwise
      const int lists = ((p.B * p.Hkv) & 7) == 0 ? 8 : 1;
      const int per = (int)gridDim.x / lists;             // workgroups per list
      const int x = (int)blockIdx.x % lists, s = (int)blockIdx.x / lists;
      const int rank = round * per + ((round & 1) ? per - 1 - s : s);
      ++round;
      return rank * lists + x < p.total ? rank * lists + x : -1;
    }
  };

  // V rows in the ring (256 bytes, 16 chunks): which physical chunk holds logical chunk `chunk`
  // (columns 8 chunk .. 8 chunk + 7) of row `row`.  bf16: the XOR swizzle of the transposing read
  // (four consecutive rows in different 64-byte groups).  fp8: the conversion pass writes the
  // tile with 128-bit stores, which the LDS serves eight lanes (= one row's eight even or eight
  // odd logical chunks) per cycle, without a second pass only if those eight lie in one 128-byte
  // half of a bank line: the even logical chunks therefore fill the first half of a row and the
  // odd ones the second, and rows are told apart inside the halves (bits 1-2), which keeps the
  // transposing read's 32 lanes (4 rows x 64 bytes) on distinct banks as well.
  auto v_chunk = [](int row, int chunk) __attribute__((always_inline)) {
    if constexpr (FP8) return ((chunk >> 1) + 8 * (chunk & 1)) ^ ((row & 3) << 1);
    else return chunk ^ attn_swz_v<ROWB>(row);
  };

  // ---- producer role: direct-to-LDS tile loads ---------------------------------------------
  // Thread tid moves chunks tid, tid + NT, ... of a tile (16 bytes each).  K goes into the ring
  // (LDS chunk c of a row holds the row's chunk c ^ swizzle; the swizzle is applied on the
  // global-address side).  V: bf16 the same; fp8 into the staging area, unswizzled.
  // The "_r" offsets are those inside the ragged last tile, where rows past N-1 re-read row N-1
  // (finite data; masked out later): a load is then one select away from the regular one.
  uint32_t ld_koff[NLD], ld_voff[NLD], ld_koff_r[NLD], ld_voff_r[NLD];
#pragma unroll
  for (int it = 0; it < NLD; ++it) {
    const int s = it * NT + tid;
    const int r = s / NCHI, c = s % NCHI;
    ld_koff[it] = r * INB + ((c ^ attn_swz_k<INB>(r)) << 4);
    ld_voff[it] = r * INB + ((FP8 ? c : v_chunk(r, c)) << 4);
    const uint32_t over = (uint32_t)max(0, (N - 1) / BN * BN + r - (N - 1)) * INB;
    ld_koff_r[it] = ld_koff[it] - over;
    ld_voff_r[it] = ld_voff[it] - over;
  }
  const uint32_t lds_wave = (uint32_t)(uintptr_t)smem + w * 1024;
  // one load of key tile t into ring slot `slot` / of value tile t into ring slot (bf16) or
  // staging slot (fp8) `slot`; only the last tile of a ragged length takes the "_r" offsets
  auto load_k = [&](int t, int slot, int it) __attribute__((always_inline)) {
    attn_lds_dma16(khead + (size_t)t * KTILEB, (t + 1) * BN > N ? ld_koff_r[it] : ld_koff[it], lds_wave + slot * KTILEB + it * NT * 16);
  };
  auto load_v = [&](int t, int slot, int it) __attribute__((always_inline)) {
    attn_lds_dma16(vhead + (size_t)t * KTILEB, (t + 1) * BN > N ? ld_voff_r[it] : ld_voff[it],
                   lds_wave + (FP8 ? STGBASE + slot * STGTILE : VBASE + slot * TILEB) + it * NT * 16);
  };
  auto issue_k = [&](int t, int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int it = 0; it < NLD; ++it) load_k(t, slot, it);
  };
  auto issue_v = [&](int t, int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int it = 0; it < NLD; ++it) load_v(t, slot, it);
  };
  // fp8: where this thread's 16 staged values (row tid / 8, bytes 16 (tid % 8) ..) go in a bf16
  // value tile: chunks 2 (tid % 8) and 2 (tid % 8) + 1 of that row
  const int st_row = tid >> 3, st_c = tid & 7;
  const uint32_t cv_v0 = VBASE + st_row * ROWB + (v_chunk(st_row, 2 * st_c) << 4);
  const uint32_t cv_v1 = VBASE + st_row * ROWB + (v_chunk(st_row, 2 * st_c + 1) << 4);
  const uint32_t st_self = STGBASE + tid * 16;  // this thread's chunk inside a staged tile
  auto staged_chunk = [&](int stg) __attribute__((always_inline)) { return *(const LDS_AS u32x4*)(smem + st_self + stg * STGTILE); };
  auto convert_store = [&](const u32x4 in, int slot) __attribute__((always_inline)) {
    // 16 e4m3 bytes -> 16 bf16 (two 16-byte chunks), exact
    uint32_t o[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[2 * i] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(in[i], 1.0f, false));
      o[2 * i + 1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(in[i], 1.0f, true));
    }
    *(LDS_AS u32x4*)(smem + cv_v0 + slot * TILEB) = u32x4{o[0], o[1], o[2], o[3]};
    *(LDS_AS u32x4*)(smem + cv_v1 + slot * TILEB) = u32x4{o[4], o[5], o[6], o[7]};
  };
  auto lds_ops_done = [&]() __attribute__((always_inline)) { __builtin_amdgcn_s_waitcnt(0xC07F); };  // lgkmcnt(0)

  // ---- first requests of a tile: key tile 0, bundle 0 and the Q operand ---------------------------
  // bundle b = key tile b+1 (the last tile again if there is none) and value tile b.
  // Q is the B operand of S^T = K Q^T: bf16: lane (qi,h) holds Q[row][16kk + 8h .. +7];
  // fp8: Q[row][64kk + 32h .. +31].
  using QFrag = std::conditional_t<FP8, i32x8, bf16x8>;
  QFrag qf[NKQ];
  auto issue_prologue = [&]() __attribute__((always_inline)) {
    issue_k(0, NSLOT - 1);  // key tile 0 borrows the K part of the last slot
    issue_k(min(1, nt - 1), 0);
    issue_v(0, 0);
    const int row = min(wq0 + qi, N - 1);
    const char* src = qhead + (size_t)row * INB + h * (FP8 ? 32 : 16);
#pragma unroll
    for (int kk = 0; kk < NKQ; ++kk) {
      if constexpr (FP8) {
        const u32x4 lo = *(const u32x4*)(src + kk * 64), hi = *(const u32x4*)(src + kk * 64 + 16);
        qf[kk] = i32x8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
      } else {
        qf[kk] = *(const bf16x8*)(src + kk * 32);
      }
    }
  };

  // ---- LDS read addresses (slot 0, first 32-key block) -----------------------------------------
  // K fragment of k-step kk: lane (qi,h) reads key row qi, chunk 2kk + h (bf16) or chunks
  // 4kk + 2h, + 1 (fp8)
  uint32_t kaddr[NKQ][QKR];
#pragma unroll
  for (int kk = 0; kk < NKQ; ++kk)
#pragma unroll
    for (int e = 0; e < QKR; ++e) kaddr[kk][e] = kg * KSUBB + qi * INB + (((QKR * (2 * kk + h) + e) ^ attn_swz_k<INB>(qi)) << 4);
  // V through the transposing load: in a group of 16 lanes, lane s reads the four columns
  // 4*(s%4).. of key row s/4 and the hardware hands lane t the four keys of column t.
  uint32_t vaddr[NCB][2];
  {
    const int s = lane & 15, chalf = (lane >> 4) & 1;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int key = 8 * e + 4 * h + (s >> 2);
        const int chunk = cb * 4 + chalf * 2 + ((s & 3) >> 1);
        vaddr[cb][e] = VBASE + kg * SUBB + key * ROWB + (v_chunk(key, chunk) << 4) + ((s & 1) << 3);
      }
  }
  // A block id names a 32-key block of the ring: 2 * slot + (which half of the slot's tiles)
  struct Operand {
    u32x4 x, y;  // K: the fragment (fp8: its low and high half); V: the fragment in x
  };
  auto k_operand = [&](auto koff, int kk) __attribute__((always_inline)) {
    Operand o;
    o.x = *(LDS_AS u32x4*)(smem + kaddr[kk][0] + koff);
    o.y = QKR > 1 ? *(LDS_AS u32x4*)(smem + kaddr[kk][QKR - 1] + koff) : o.x;
    return o;
  };
  auto v_operand = [&](auto voff, int cb, int kc) __attribute__((always_inline)) {
    const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(smem + vaddr[cb][0] + voff + kc * 16 * ROWB));
    const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(smem + vaddr[cb][1] + voff + kc * 16 * ROWB));
    s16x8 av;
    av[0] = v0[0]; av[1] = v0[1]; av[2] = v0[2]; av[3] = v0[3];
    av[4] = v1[0]; av[5] = v1[1]; av[6] = v1[2]; av[7] = v1[3];
    Operand o;
    o.x = __builtin_bit_cast(u32x4, av);
    o.y = o.x;
    return o;
  };
  auto qk_mfma = [&](const Operand& a, int kk, const f32x16& acc) __attribute__((always_inline)) {
    if constexpr (FP8) {
      const i32x8 av = i32x8{(int)a.x[0], (int)a.x[1], (int)a.x[2], (int)a.x[3], (int)a.y[0], (int)a.y[1], (int)a.y[2], (int)a.y[3]};
      // literal zero scale operands select the instruction without block scales (the scaled form
      // is not recognised as a plain matrix instruction by the compiler's scheduler and would be
      // left outside it, two dependent MFMAs back to back at the end of the step)
      return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, qf[kk], acc, 0, 0, 0, 0, 0, 0);
    } else {
      return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a.x), qf[kk], acc, 0, 0, 0);
    }
  };

  // ---- streaming-softmax state ----------------------------------------------------------------
  f32x16 oacc[NCB];
  float m_ref;            // reference maximum, scaled log2 units
  float l_run;            // this lane's share of the row sum (halves are added at the end)
  const float c = p.scale_log2;
  f32x16 s_a, s_b;        // S^T of two consecutive blocks (one consumed, one produced)
  u32x4 p_a[2], p_b[2];   // packed P^T of two consecutive blocks (one produced, one consumed)

  // true maximum of a block in scaled log2 units (both lanes of a query column agree on it)
  auto block_max = [&](const f32x16& s) __attribute__((always_inline)) {
    float mx = fmaxf(s[0], s[1]);
#pragma unroll
    for (int r = 2; r < 16; ++r) mx = fmaxf(mx, s[r]);
    return attn_max_halves(mx) * c;
  };
  // raise the reference maximum to cover mx and rescale what is relative to it: l, O and, if there is one, the
  // packed P^T that has not been multiplied into O yet; `heal`: l and O may hold overflow (kSumDrop)
  auto raise_reference = [&](float mx, u32x4* pend, auto heal) __attribute__((always_inline)) {
    const float m_new = fmaxf(m_ref, mx);
    const float alpha = __builtin_amdgcn_exp2f(m_ref - m_new);  // 0 on the first block
    m_ref = m_new;
    if constexpr (decltype(heal)::value) {
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(l_run > kSumDrop) != 0, 0)) {
        const float l_row = attn_sum_halves(l_run);  // (O holds the products of both halves' probabilities; a NaN stays one)
        if (alpha == 0.f && l_row > kSumDrop) {
          l_run = 0.f;
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[cb][r] = 0.f;
          pend[0] = pend[1] = u32x4{0, 0, 0, 0};
        }
      }
    }
    l_run *= alpha;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) oacc[cb] *= alpha;
    if (pend) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const uint32_t u = pend[i][r];
          pend[i][r] = attn_pack_bf16(__uint_as_float(u << 16) * alpha, __uint_as_float(u & 0xffff0000u) * alpha);
        }
    }
  };
  // exponentials of a whole block against the current reference, packed; returns the lane's sum
  auto exp_block = [&](const f32x16& s_in, u32x4 (&p_out)[2], auto bounded) __attribute__((always_inline)) {
    f32x16 e;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float x = __builtin_fmaf(s_in[r], c, -m_ref);
      if constexpr (decltype(bounded)::value) x = __builtin_elementwise_minimum(x, 16.0f);  // (a NaN stays one)
      e[r] = __builtin_amdgcn_exp2f(x);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) p_out[u >> 2][u & 3] = attn_pack_bf16(e[2 * u], e[2 * u + 1]);
    float ls0 = e[0], ls1 = e[1];
#pragma unroll
    for (int u = 1; u < 8; ++u) {
      ls0 += e[2 * u];
      ls1 += e[2 * u + 1];
    }
    return ls0 + ls1;
  };

  // ---- boundary-case building blocks (compiler-scheduled, not overlapped) ----------------------
  auto qk_block = [&](f32x16& s, auto koff) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < NKQ; ++kk) s = qk_mfma(k_operand(koff, kk), kk, s);
  };
  auto pv_block = [&](const u32x4 (&pk)[2], auto voff) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2 * NCB; ++i) {
      const int cb = i % NCB, kc = i / NCB;
      oacc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, v_operand(voff, cb, kc).x),
                                                         __builtin_bit_cast(bf16x8, pk[kc]), oacc[cb], 0, 0, 0);
    }
  };
  // softmax of a block that may need masking, with the block maximum taken first; `pend` is the
  // packed P^T of the block whose PV product has not been issued yet (rescaled with O)
  auto softmax_block = [&](f32x16& s, u32x4 (&pk)[2], u32x4 (&pend)[2], int key0, bool need_mask) __attribute__((always_inline)) {
    if (need_mask) {
      const int kbase = key0 + 4 * h;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (kbase + 8 * (r >> 2) + (r & 3) > limit) s[r] = -INFINITY;
    }
    const float mx = block_max(s);
    if (__builtin_amdgcn_ballot_w64(mx > m_ref + kTau) != 0) {
      raise_reference(mx, pend, std::integral_constant<bool, !FP8>{});
    }
    l_run += exp_block(s, pk, std::false_type{});
  };
  // the first block's exponentials once more, bounded, if they overflowed (kSumDrop); behind the score products
  // of the second block, which hide the look at the sum
  auto bound_first = [&]() __attribute__((always_inline)) {
    if constexpr (!FP8)
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(l_run > kSumDrop) != 0, 0)) l_run = exp_block(s_b, p_b, std::true_type{});
  };
  auto is_active = [&](int key0) __attribute__((always_inline)) {
    return wave_valid && key0 < kv_end && (!CAUSAL || key0 <= wlast);
  };
  auto needs_mask = [&](int key0) __attribute__((always_inline)) {
    return (CAUSAL && key0 + 31 > wq0) || key0 + 31 >= N;
  };

  // ---- the pipelined step on fully visible blocks ------------------------------------------------
  //   s_in  : scores of the block exponentiated now                     -> p_out
  //   s_out : scores of the next block        (K operands of block id bid)
  //   p_pv  : probabilities of the previous block, multiplied into O    (V operands of block id bid)
  // Of the NM MFMAs of a step every STRIDE-th is a score product (a dependent chain), the others
  // are PV products (independent accumulators); operands are read from LDS RA MFMAs ahead, and
  // the first RA operands of a step are requested by the previous step (bidnext = the block the
  // next step reads).  The vector work needs no block maximum: exponentials are taken against
  // the current reference and the block is redone, after raising the reference and rescaling,
  // only if a lane's partial sum comes out large or not a number (always on the very first
  // block).  A row's multiply-add, exponential, and sum and pack lie in three consecutive slots, so that none waits for the
  // one before it.  (A scheduling-group pipeline that left the order to the compiler had all three in one slot.  By itself this gives d = 64 1.5 %,
  // 2 x 32 x 8192 1095 -> 1079 us, and d = 128 nothing beyond noise; it is here because every instantiation comes out alike, the list
  // walk and the paired form too, which the compiler's solver had left half unpipelined.)
  // NSEG: between(i) runs in front of slot i * NM / NSEG, which is where the producer role's work goes.
  Operand pre[RA];
  auto koff_of = [](auto bid) __attribute__((always_inline)) { return ic<(decltype(bid)::value >> 1) * KTILEB + (decltype(bid)::value & 1) * KSUBB>{}; };
  auto voff_of = [](auto bid) __attribute__((always_inline)) { return ic<(decltype(bid)::value >> 1) * TILEB + (decltype(bid)::value & 1) * SUBB>{}; };
  auto step_operand = [&](auto bid, int m) __attribute__((always_inline)) {
    const int i = m - m / STRIDE - 1;
    return m % STRIDE == 0 ? k_operand(koff_of(bid), m / STRIDE) : v_operand(voff_of(bid), i % NCB, i / NCB);
  };
  auto step_hot = [&](f32x16& s_in, f32x16& s_out, u32x4 (&p_out)[2], u32x4 (&p_pv)[2], auto bid, auto bidnext, auto nseg_tag, auto between) __attribute__((always_inline)) {
    constexpr int NSEG = decltype(nseg_tag)::value, SEG = NM / NSEG;
    static_assert(NSEG <= 4 && NM % NSEG == 0, "whole slots");
    Operand op[NM];
#pragma unroll
    for (int m = 0; m < RA; ++m) op[m] = pre[m];
#pragma unroll
    for (int r = 0; r < 16; ++r) s_out[r] = 0.f;
    float ls0 = 0.f, ls1 = 0.f;
    float x[16], e[16];
    // the slot of row r's exponential; its multiply-add comes a slot earlier, its sum and pack a slot later
    auto eslot = [](int r) constexpr { return 1 + r * (NM - 1) / 16; };
    auto one_slot = [&](auto slot_tag) __attribute__((always_inline)) {
      constexpr int m = decltype(slot_tag)::value;
      if constexpr (m % SEG == 0) {
        between(m / SEG);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (m % STRIDE == 0) {
        s_out = qk_mfma(op[m], m / STRIDE, s_out);
      } else {
        constexpr int i = m - m / STRIDE - 1;
        oacc[i % NCB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, op[m].x), __builtin_bit_cast(bf16x8, p_pv[i / NCB]),
                                                                oacc[i % NCB], 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (eslot(r) - 1 == m) x[r] = __builtin_fmaf(s_in[r], c, -m_ref);
        if (eslot(r) == m) e[r] = __builtin_amdgcn_exp2f(x[r]);
        if (eslot(r) + 1 == m || (m == NM - 1 && eslot(r) == m)) {
          if (r & 1) {
            p_out[r >> 3][(r >> 1) & 3] = attn_pack_bf16(e[r - 1], e[r]);
            ls1 = r == 1 ? e[r] : ls1 + e[r];
          } else {
            ls0 = r == 0 ? e[r] : ls0 + e[r];
          }
        }
      }
      if constexpr (m + RA < NM) op[m + RA] = step_operand(bid, m + RA);
      else pre[m + RA - NM] = step_operand(bidnext, m + RA - NM);
      __builtin_amdgcn_sched_barrier(0);
    };
    __builtin_amdgcn_sched_barrier(0);
    for_each_slot(one_slot, std::make_integer_sequence<int, NM>{});
    ls0 += ls1;
    asm volatile("" ::"v"(p_out[0]), "v"(p_out[1]));
    float ls = ls0;
    if (__builtin_amdgcn_ballot_w64(!(ls <= kSumLimit)) != 0) {
      // the redo path "reads" the optimistic packs, so that they are computed inside the
      // pipelined step above and not sunk below this branch into the common path's tail
      asm volatile("" ::"v"(p_out[0]), "v"(p_out[1]));
      raise_reference(block_max(s_in), nullptr, std::false_type{});
      ls = exp_block(s_in, p_out, std::integral_constant<bool, !FP8>{});
    }
    l_run += ls;
  };

  // the same step for blocks that may be masked or not visible to this wave (run-time offsets)
  auto step_any = [&](bool do_sm, int key0, bool do_mm, f32x16& s_in, f32x16& s_out, u32x4 (&p_out)[2], u32x4 (&p_pv)[2], int koff,
                      int voff) __attribute__((always_inline)) {
    if (do_sm) softmax_block(s_in, p_out, p_pv, key0, needs_mask(key0));
    if (do_mm) {
      qk_block(s_out, koff);
      pv_block(p_pv, voff);
    }
  };

  // ---- main loop over bundles ------------------------------------------------------------------------
  // Iteration b: exponentiate blocks 2b+1 and 2b+2, compute the scores of blocks 2b+2 and 2b+3
  // (key tile b+1), accumulate blocks 2b and 2b+1 (value tile b).  Between its two steps bundle
  // b+1 (requested one iteration ago) is published and the slot of bundle b-1, which every wave
  // has finished reading, is handed to bundle b+2: bf16 requests its key and value tiles into it;
  // fp8 requests its key tile into it, converts its staged value tile (staging slot b mod 2) into
  // it, and stages the value tile of bundle b+3 where that of bundle b+1 was converted from.
  // A wave's LDS writes must have completed before it signals the barrier that publishes them.
  auto publish_and_free = [&](bool drain_lds) __attribute__((always_inline)) {
    ATTN_WAIT_VMCNT(0);
    if (FP8 && drain_lds) lds_ops_done();
    attn_wg_barrier();
  };
  // burst form, for the iterations that are not pipelined
  auto bundle_mid = [&](int b, int free_slot) __attribute__((always_inline)) {
    publish_and_free(true);
    if (b + 2 < nt) {
      issue_k(min(b + 3, nt - 1), free_slot);
      if constexpr (FP8) convert_store(staged_chunk(b & 1), free_slot);
      else issue_v(b + 2, free_slot);
    }
    if constexpr (FP8)
      if (b + 3 < nt) issue_v(b + 3, (b + 1) & 1);
  };
  auto nothing = [](int) __attribute__((always_inline)) {};
  // Pipelined form: the same work is handed out over the iteration's second
  // step, one piece in front of every SEG-th slot, between the operand reads.  A bundle index past the
  // end re-requests the last tiles into the free slot, which is never read again (and converts
  // whatever the staging slot holds): the loads in flight per wave are then the same in every
  // iteration.
  auto bundle_hot = [&](int b, auto slot_tag) __attribute__((always_inline)) {
    constexpr int SLOT = decltype(slot_tag)::value;
    constexpr int FREE = (SLOT + NSLOT - 1) % NSLOT;
    constexpr int NSEG = FP8 ? 2 : (2 * NLD < 2 ? 2 : 2 * NLD);
    step_hot(s_a, s_b, p_a, p_b, ic<2 * SLOT>{}, ic<2 * SLOT + 1>{}, ic<NSEG>{}, nothing);
    const int kt = min(b + 3, nt - 1), vt = min(b + 2, nt - 1);  // key and value tile of bundle b+2
    u32x4 staged;
    auto producer = [&](int sg) __attribute__((always_inline)) {
      // (the conversion's LDS writes of the previous iteration have retired: LDS operations
      // complete in order, and this wave has since waited for dozens of later operand reads)
      if (sg == 0) publish_and_free(false);
      if constexpr (FP8) {
        if (sg == 0) {
          load_k(kt, FREE, 0);
          staged = staged_chunk(b & 1);
        } else {
          convert_store(staged, FREE);
          load_v(min(b + 3, nt - 1), (b + 1) & 1, 0);
        }
      } else {
#pragma unroll
        for (int j = 0; j < 2 * NLD; ++j) {
          if ((j < NSEG ? j : NSEG - 1) != sg) continue;
          if (j < NLD) load_k(kt, FREE, j);
          else load_v(vt, FREE, j - NLD);
        }
      }
    };
    step_hot(s_b, s_a, p_b, p_a, ic<2 * SLOT + 1>{}, ic<2 * ((SLOT + 1) % NSLOT)>{}, ic<NSEG>{}, producer);
  };
  auto bundle_any = [&](int b, int slot) __attribute__((always_inline)) {
    const int k1 = (2 * b + 1) * 32, k2 = k1 + 32;
    step_any(is_active(k1), k1, is_active(k1 - 32), s_a, s_b, p_a, p_b, slot * KTILEB, slot * TILEB);
    bundle_mid(b, slot >= 1 ? slot - 1 : NSLOT - 1);
    step_any(is_active(k2), k2, is_active(k1), s_b, s_a, p_b, p_a, slot * KTILEB + KSUBB, slot * TILEB + SUBB);
  };

  // KS = 2: iteration b exponentiates this wave's block of tile b+1, computes its scores of tile b+2,
  // accumulates its block of tile b; every wave issues the loads of bundle b+3 in every iteration
  // (past the end the last tiles again, never read), so the loads in flight are always the same.
  auto split_mid = [&]() __attribute__((always_inline)) {
    ATTN_WAIT_VMCNT(2 * NLD);  // bundle b+1 has landed, bundle b+2 stays in flight
    attn_wg_barrier();
  };
  auto split_hot = [&](int b, auto slot_tag) __attribute__((always_inline)) {
    constexpr int SLOT = decltype(slot_tag)::value, FREE = (SLOT + 3) & 3, NSEG = 2 * NLD < 2 ? 2 : 2 * NLD;
    const int kt = min(b + 5, nt - 1), vt = min(b + 3, nt - 1);
    auto producer = [&](int sg) __attribute__((always_inline)) {
      if (sg == 0) split_mid();
#pragma unroll
      for (int j = 0; j < 2 * NLD; ++j) {
        if (j != sg) continue;
        if (j < NLD) load_k(kt, FREE, j);
        else load_v(vt, FREE, j - NLD);
      }
    };
    if constexpr (SLOT & 1) step_hot(s_b, s_a, p_b, p_a, ic<2 * SLOT>{}, ic<2 * ((SLOT + 1) & 3)>{}, ic<NSEG>{}, producer);
    else step_hot(s_a, s_b, p_a, p_b, ic<2 * SLOT>{}, ic<2 * ((SLOT + 1) & 3)>{}, ic<NSEG>{}, producer);
  };
  auto hand_on = [&]() __attribute__((always_inline)) {  // what an even step leaves becomes the next even step's input
    s_a = s_b;
#pragma unroll
    for (int i = 0; i < 2; ++i) p_b[i] = p_a[i];
  };
  auto split_any = [&](int b) __attribute__((always_inline)) {
    const int slot = b & 3, k1 = (b + 1) * BN + kg * 32;
    split_mid();
    issue_k(min(b + 5, nt - 1), (slot + 3) & 3);
    issue_v(min(b + 3, nt - 1), (slot + 3) & 3);
    step_any(is_active(k1), k1, is_active(k1 - BN), s_a, s_b, p_a, p_b, slot * KTILEB, slot * TILEB);
    hand_on();
  };
  if constexpr (FORM != kWhole) {
    for (;;) {
      if constexpr (MODE == 1) {
        // (holds the barrier behind which no wave reads the finished tile's ring; nothing of the next tile is requested before it, the
        // workgroups beside this one fill the seam)
        const int wg = next_tile_index();
        if (wg < 0) return;
        set_tile(wg);
      } else {
        set_tile((int)blockIdx.x);
      }
      if constexpr (FORM == kPair) {
        const char* src = qhead + (size_t)min(qrow, N - 1) * INB + h * 16;
#pragma unroll
        for (int kk = 0; kk < NKQ; ++kk)
          if constexpr (!FP8) qf[kk] = *(const bf16x8*)(src + kk * 32);
      }
      // KS = 2: Q (128 rows, swizzled like a K tile) borrows the V parts of slots 2 and 3; key tiles 0 and 1 the K
      // parts of slots 3 and 2
      constexpr int QBASE = VBASE + 2 * TILEB;
      if constexpr (KS == 2) {
#pragma unroll
        for (int it = 0; it < 2 * NLD; ++it) {
          const int s = it * NT + tid, r = s / NCHI, ch = (s % NCHI) ^ attn_swz_k<INB>(r);
          attn_lds_dma16(qhead, (uint32_t)min(q0 + r, N - 1) * INB + (ch << 4), lds_wave + QBASE + it * NT * 16);
        }
      }
      issue_k(0, 3);
      issue_k(min(1, nt - 1), 2);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        issue_k(min(b + 2, nt - 1), b);
        issue_v(min(b, nt - 1), b);
      }
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[cb][r] = 0.f;
      m_ref = kNoRef;
      l_run = 0.f;
#pragma unroll
      for (int i = 0; i < 2; ++i) p_a[i] = p_b[i] = u32x4{0, 0, 0, 0};
      ATTN_WAIT_VMCNT(4 * NLD);  // Q and key tiles 0 and 1 have landed
      attn_wg_barrier();
      if constexpr (KS == 2) {
        const int qr = (w % NQW) * 32 + qi;
#pragma unroll
        for (int kk = 0; kk < NKQ; ++kk) {
          // (kaddr's row qi and this row agree in the bits the swizzle uses)
          const u32x4 x = *(LDS_AS const u32x4*)(smem + QBASE + qr * INB + (((2 * kk + h) ^ attn_swz_k<INB>(qr)) << 4));
          if constexpr (!FP8) qf[kk] = __builtin_bit_cast(bf16x8, x);
        }
      }
      // (a wave whose first block is invisible sees no key at all: l and O stay zero)
      if (is_active(kg * 32)) {
        // Both waves start from the reference maximum of keys 0 .. 31, all of which this wave's queries see,
        // as the unsplit form does: blocks far below it (masked keys, down to -inf) get probabilities of zero
        // instead of a reference of their own against which they would overflow, and P is rounded as there.
        // (Measured, without -> with: 2 heads of 256 6.23 -> 6.31 us, 32 of 1000 causal 18.2 -> 18.4.)
        if (kg) {
          qk_block(s_b, 3 * KTILEB - KSUBB);
          m_ref = fmaxf(m_ref, block_max(s_b));
        }
        qk_block(s_b, 3 * KTILEB);
        softmax_block(s_b, p_b, p_a, kg * 32, needs_mask(kg * 32));
        qk_block(s_a, 2 * KTILEB);
        bound_first();
      }
#pragma unroll
      for (int kk = 0; kk < NKQ; ++kk) asm volatile("" ::"v"(qf[kk]));  // (read by every wave before the barrier, too)
      lds_ops_done();
      ATTN_WAIT_VMCNT(2 * NLD);
      attn_wg_barrier();  // bundle 0 is full; slots 2 and 3 are free
      issue_k(min(4, nt - 1), 2);
      issue_v(min(2, nt - 1), 2);
#pragma unroll
      for (int m = 0; m < RA; ++m) pre[m] = step_operand(ic<0>{}, m);
      const int vis = (CAUSAL ? min(wq0, N - 1) : N - 1) - kg * 32;
      constexpr int LAST1 = BN + 31;  // last key of this wave's block of tile 1 (kg = 0)
      const int n_hot = (wave_valid && vis >= LAST1) ? (vis - LAST1) / BN + 1 : 0;  // bundles whose block of tile b+1 every query sees in full
      int b = 0;
      for (; b < (n_hot & ~3); b += 4) {
        split_hot(b, ic<0>{});
        split_hot(b + 1, ic<1>{});
        split_hot(b + 2, ic<2>{});
        split_hot(b + 3, ic<3>{});
      }
      if (b < n_hot) { split_hot(b, ic<0>{}); ++b; }
      if (b < n_hot) { split_hot(b, ic<1>{}); ++b; }
      if (b < n_hot) { split_hot(b, ic<2>{}); ++b; }
      if (b & 1) hand_on();
      for (; b < nt; ++b) split_any(b);

      if constexpr (KS == 1) {
        ATTN_WAIT_VMCNT(0);  // no load writes the LDS any more
        const float l = attn_sum_halves(l_run);
        u32x4 out[2 * NCB];
        attn_pack_o_rows<NCB>(oacc, p.out_scale / l, out);
        if (qrow < N) {
          const size_t row = (size_t)(tile_b * p.Hq + tile_hq) * N + qrow;
          if (h == 0) p.lse[row] = (m_ref + __builtin_amdgcn_logf(l)) * 0.6931471805599453f;
          attn_store_packed_o<NCB>(out, (char*)p.o + row * ROWB + h * 16);
        }
        if constexpr (MODE == 1) continue;
        else return;
      }
      // ---- merge: each of the two waves gives away the columns the other one finishes ------------------
      float l = attn_sum_halves(l_run);
      ATTN_WAIT_VMCNT(0);
      attn_wg_barrier();  // no load is in flight and no wave reads the ring any more
      constexpr int NH = NCB / 2, MLBASE = NWAVES * NH * 4096;
      static_assert(MLBASE + NWAVES * 512 <= STGBASE, "the exchanged halves fit the ring");
      const int wq = w % NQW;
      LDS_AS f32x4* const give = (LDS_AS f32x4*)smem + ((kg ^ 1) * NQW + wq) * NH * 256 + lane;
      LDS_AS f32x4* const take = (LDS_AS f32x4*)smem + w * NH * 256 + lane;
      f32x16 mine[NH];
#pragma unroll
      for (int cb = 0; cb < NH; ++cb) {
        const f32x16 other = kg ? oacc[cb] : oacc[NH + cb];
        mine[cb] = kg ? oacc[NH + cb] : oacc[cb];
#pragma unroll
        for (int a = 0; a < 4; ++a) give[(cb * 4 + a) * 64] = f32x4{other[4 * a], other[4 * a + 1], other[4 * a + 2], other[4 * a + 3]};
      }
      ((LDS_AS f32x2*)(smem + MLBASE))[((kg ^ 1) * NQW + wq) * 64 + lane] = f32x2{m_ref, l};
      __syncthreads();
      f32x2 ml = ((LDS_AS const f32x2*)(smem + MLBASE))[w * 64 + lane];
      const float m = fmaxf(m_ref, ml[0]);
      const float a_mine = __builtin_amdgcn_exp2f(m_ref - m), a_other = __builtin_amdgcn_exp2f(ml[0] - m);
      const bool drop_mine = a_mine == 0.f && l > kSumDrop, drop_other = a_other == 0.f && ml[1] > kSumDrop;
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(drop_mine || drop_other) != 0, 0)) {
        // (as in raise_reference)
        if (drop_mine) l = 0.f;
        if (drop_other) ml[1] = 0.f;
#pragma unroll
        for (int cb = 0; cb < NH; ++cb)
#pragma unroll
          for (int a = 0; a < 4; ++a) {
            if (drop_other) take[(cb * 4 + a) * 64] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (drop_mine) mine[cb][4 * a + r] = 0.f;
          }
      }
      const float l_all = l * a_mine + ml[1] * a_other;
#pragma unroll
      for (int cb = 0; cb < NH; ++cb)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const f32x4 o = take[(cb * 4 + a) * 64];
#pragma unroll
          for (int r = 0; r < 4; ++r) mine[cb][4 * a + r] = mine[cb][4 * a + r] * a_mine + o[r] * a_other;
        }
      u32x4 out[2 * NH];
      attn_pack_o_rows<NH>(mine, p.out_scale / l_all, out);
      if (qrow < N) {
        const size_t row = (size_t)(tile_b * p.Hq + tile_hq) * N + qrow;
        if (kg == 0 && h == 0) p.lse[row] = (m + __builtin_amdgcn_logf(l_all)) * 0.6931471805599453f;
        attn_store_packed_o<NH>(out, (char*)p.o + row * ROWB + kg * NH * 64 + h * 16);
      }
      return;
    }
  }

  // ---- the tiles of this workgroup -----------------------------------------------------------------
  int wg = (int)blockIdx.x;
  if constexpr (MODE != 0) {
    wg = next_tile_index();
    if (wg < 0) return;
  }
  set_tile(wg);
  issue_prologue();
  // output of the previous tile, packed, waiting to be stored (modes 1 and 2)
  u32x4 pend_o[2 * NCB];
  float pend_lse = 0.f;
  char* pend_o_ptr = nullptr;   // this lane's output row (null: row past the end)
  float* pend_lse_ptr = nullptr;  // this lane's lse element (null: not this lane's to write)
  bool pending = false;
  for (;;) {
    // fresh streaming-softmax state
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[cb][r] = 0.f;
    m_ref = kNoRef;
    l_run = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i) p_a[i] = p_b[i] = u32x4{0, 0, 0, 0};

    // ---- prologue: block 0 ---------------------------------------------------------------------------
    if constexpr (FP8) {
      // everything requested so far has landed: convert value tile 0 into slot 0, request key tile 2
      // and stage value tiles 1 and 2
      ATTN_WAIT_VMCNT(0);
  #pragma unroll
      for (int kk = 0; kk < NKQ; ++kk)
  #pragma unroll
        for (int i = 0; i < 8; ++i) asm volatile("" ::"v"(qf[kk][i]));  // Q is in registers from here on
      convert_store(staged_chunk(0), 0);
      lds_ops_done();
      if (nt > 1) {
        issue_k(min(2, nt - 1), 1);
        issue_v(1, 1);
      }
      if (nt > 2) issue_v(2, 0);
    } else {
      // Q is in registers from here on.  The compiler waits for Q with the counter that the
      // direct-to-LDS loads share and cannot see them, so this is a wait for every load issued
      // so far: bundle 1 is therefore requested only behind the barrier.
      ATTN_WAIT_VMCNT(0);
  #pragma unroll
      for (int kk = 0; kk < NKQ; ++kk) asm volatile("" ::"v"(qf[kk]));
    }
    attn_wg_barrier();
    if constexpr (!FP8) {
      if (nt > 1) {
        issue_k(min(2, nt - 1), 1);
        issue_v(1, 1);
      }
    }
    if (wave_valid) {
      qk_block(s_b, (NSLOT - 1) * KTILEB);             // S(0)
      softmax_block(s_b, p_b, p_a, 0, needs_mask(0));  // P(0) -> p_b (nothing pending yet)
      qk_block(s_a, (NSLOT - 1) * KTILEB + KSUBB);     // S(1); ignored if block 1 is not visible
      bound_first();
    }
    if constexpr (FP8) {
      // bundle 1 has arrived once only value tile 2's load is outstanding: convert its value tile into slot 1
      if (nt > 1) {
        if (nt > 2) ATTN_WAIT_VMCNT(1);
        else ATTN_WAIT_VMCNT(0);
        convert_store(staged_chunk(1), 1);
        lds_ops_done();
      }
    } else {
      if (nt > 1) ATTN_WAIT_VMCNT(2 * NLD);
      else ATTN_WAIT_VMCNT(0);
    }
    attn_wg_barrier();  // bundle 0 is full; the K part of the last slot is empty again
    if constexpr (MODE != 0) {
      // every load of this tile's prologue has been waited for: the previous tile's output may go
      if (pending) {
        if (pend_lse_ptr) *pend_lse_ptr = pend_lse;
        if (pend_o_ptr) attn_store_packed_o<NCB>(pend_o, pend_o_ptr);
      }
    }
  #pragma unroll
    for (int m = 0; m < RA; ++m) pre[m] = step_operand(ic<0>{}, m);  // first operands of the first pipelined step (block id 0)


    // bundles 0 .. n_hot-1 touch only blocks (up to 2b+2) that every query of this wave sees in full
    const int vis = CAUSAL ? min(wq0, N - 1) : N - 1;  // last key every query of the wave can see
    const int n_hot = (wave_valid && vis >= 95) ? (vis - 95) / 64 + 1 : 0;
    const int n_ring = n_hot - n_hot % NSLOT;  // whole turns of the ring, slot offsets as immediates
    int b = 0;
    for (; b < n_ring; b += NSLOT) {
      bundle_hot(b, ic<0>{});
      bundle_hot(b + 1, ic<1>{});
      bundle_hot(b + 2, ic<2>{});
    }
    // the last fully visible bundles (fewer than a turn), then the masked / partly visible ones
    int slot = 0;
    if (b < n_hot) { bundle_hot(b, ic<0>{}); ++b; slot = 1; }
    if (b < n_hot) { bundle_hot(b, ic<1>{}); ++b; slot = 2; }
    for (; b < nt; ++b) {
      bundle_any(b, slot);
      slot = slot == NSLOT - 1 ? 0 : slot + 1;
    }


    // ---- epilogue: O = acc / l (bf16), lse = (m + log2 l) * ln 2 ----------------------------------
    const float l = attn_sum_halves(l_run);
    const float lse_val = (m_ref + __builtin_amdgcn_logf(l)) * 0.6931471805599453f;
    float* const lse_ptr = (qrow < N && h == 0) ? p.lse + (size_t)(tile_b * p.Hq + tile_hq) * N + qrow : nullptr;
    char* const o_ptr = qrow < N ? (char*)p.o + ((size_t)(tile_b * p.Hq + tile_hq) * N + qrow) * ROWB : nullptr;
    if constexpr (MODE == 0) {
      if (lse_ptr) *lse_ptr = lse_val;
      attn_pack_o_rows<NCB>(oacc, p.out_scale / l, pend_o);
      if (o_ptr) attn_store_packed_o<NCB>(pend_o, o_ptr + h * 16);
      break;
    } else {
      // seam: once no wave reads the ring any more, request the next tile's first loads, then
      // pack this tile's output; it is stored when those loads have been waited for
      if constexpr (MODE == 2) attn_wg_barrier();
      const int nwg = next_tile_index();
      if (nwg >= 0) {
        set_tile(nwg);
        issue_prologue();
      }
      attn_pack_o_rows<NCB>(oacc, p.out_scale / l, pend_o);
      pend_lse = lse_val;
      pend_lse_ptr = lse_ptr;
      pend_o_ptr = o_ptr ? o_ptr + h * 16 : nullptr;
      pending = true;
      if (nwg < 0) {
        if (pend_lse_ptr) *pend_lse_ptr = pend_lse;
        if (pend_o_ptr) attn_store_packed_o<NCB>(pend_o, pend_o_ptr);
        break;
      }
    }
  }  // tile loop
}

// resident workgroups of the list-walking launch: one per CU, rounded down to whole XCD shares
int resident_workgroups() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  return cus - cus % 8;
}

// Launches with at least three tiles per CU walk static tile lists (mode 2): the seams
// between a workgroup's tiles hide part of what a workgroup pays per tile outside its main loop
// (measured: causal +0.5 .. +4.5 %; with two tiles per CU the plain launch is 1 % faster; non-causal 0.93 - 0.97 of the plain launch's time on
// average, fp8, us: 512 heads x 513 90.7 -> 82.0, 768 x 257 58.7 -> 51.8, 192 x 1500 184 -> 175, 64 x 8192 1380 / 1378).
// A non-causal list is dealt as if its tiles were equal, but a ragged head's last tile is light (its waves past the end do nothing), which
// tiles handed out one by one level out.  Up to eight rounds, beyond which that drowns, both are followed on the host (1 - 6 us; a light tile
// takes 0.35, and 0.65 of the waves it uses), and lists are walked if they end earlier with the 5 % that their seams save.  us, lists / one by
// one: 160 heads x 1138 128.1 / 119.0, 60 x 3080 at d = 64 192.9 / 180.3, fp8 72 x 2620 222.5 / 204.7, 160 x 1130 104.9 / 93.0.  Over 429 launches
// this is 0.2 % slower than the faster way on average, at worst 6 %, where lists always are 0.5 % and 9 %, never 3.5 % and 29 %.
bool lists_pay(const AttnParams& p, int tiles, int resident) {
  if (tiles < 3 * resident) return false;
  const int waves = (p.N - 1) % 256 / 32 + 1;  // of a head's last tile
  if (p.causal || waves == 8 || tiles > 8 * resident || resident > 256) return true;
  const double weight[2] = {1.0, 0.35 + 0.65 * waves / 8.0};
  const int lists = p.map.lists, per = resident / lists, n = tiles / lists, full = p.map.G * (p.map.T - 1);
  double dealt[256] = {}, free_at[2][256];  // per workgroup; when the workgroups that run a full / a light tile come free, in order
  int first[2] = {0, 0}, count[2] = {per, 0};
  for (int s = 0; s < per; ++s) free_at[0][s] = 0.0;
  double most_dealt = 0.0, most = 0.0;
  for (int rank = 0, inner = 0, s = 0, down = 0; rank < n; ++rank) {
    const int light = inner >= full;
    if (++inner == p.map.W) inner = 0;
    dealt[s] += weight[light];
    if (dealt[s] > most_dealt) most_dealt = dealt[s];
    if (down ? s == 0 : s == per - 1) down ^= 1;
    else s += down ? -1 : 1;
    const int from = count[1] && (!count[0] || free_at[1][first[1]] < free_at[0][first[0]]);
    const double end = free_at[from][first[from]] + weight[light];
    first[from] = (first[from] + 1) & 255;
    --count[from];
    free_at[light][(first[light] + count[light]++) & 255] = end;
    if (end > most) most = end;
  }
  return 0.95 * most_dealt < most;
}

// bf16 launches of few tiles (`tiles` of 256 queries) split the keys (KS = 2); the plain and the queue
// launch follow the same rule, so that both give the same bytes.  us, whole tiles -> split keys, d = 128, heads x N:
//   non-causal  32 x 1000 25.8 -> 20.3; 16 x 2048 42.0 -> 34.2; 34 x 2048 100.4 -> 92.0; 22 x 4096 186.1 -> 172.7;
//               100 x 64 5.9 -> 7.0; 150 x 150 10.5 -> 17.7; 38 x 1000 26.7 -> 40.5; 90 x 1000 60.6 -> 69.8; 40 x 4096 291.9 -> 301.0
//   causal      32 x 1000 25.8 -> 18.0; 48 x 1000 26.3 -> 24.3; 32 x 2048 47.3 -> 40.5; 16 x 4096 84.9 -> 69.4;
//               150 x 150 10.5 -> 16.1; 58 x 1000 28.7 -> 31.2; 85 x 513 20.0 -> 25.4
// and d = 64: non-causal 34 x 2048 67.8 -> 60.2, 90 x 1000 39.2 -> 40.7; causal 48 x 1000 19.4 -> 16.8, 64 x 513 12.7 -> 12.9.
bool split_pays(const AttnParams& p, long long tiles) {
  const int per_head = (p.N + 127) / 128;
  const AttnSplitCost cost = p.causal ? AttnSplitCost{7.6, 10.0, 0.82, 0.75, 5.0} : AttnSplitCost{14.7, 12.9, 1.07, 0.66, 5.0};
  return attn_split_pays(p.causal != 0, tiles, (long long)p.B * p.Hq * per_head, per_head, (p.N + 31) / 32, cost);
}

// What a launch of one form takes, us (see AttnFormCost): n workgroups, the longest and the mean of their chains in 32-key steps.  A causal
// launch, longest first, lasts as long as its longest workgroup, or as all of them take evenly spread and half of t workgroups more.
double form_us(const AttnFormCost& c, bool causal, double n, int slots, double longest, double mean) {
  const long long groups = (long long)n, rounds = (groups + 255) / 256;
  if (!causal) return attn_equal_us(c, groups, slots, longest);
  const double step = attn_shared_step(c, groups, slots), k = (double)(rounds < slots ? rounds : slots);
  const double chain = c.P + longest * step, work = groups > 256ll * slots ? n / 256.0 + 0.5 * c.t : (double)rounds;
  const double all = work * (c.P + mean * step) / k;
  return c.F + (chain > all ? chain : all);
}

// Paired workgroups (kPair) against the form that the launch would take otherwise.  The numbers are fits to 1609 random launches (heads
// 1 .. 2000, N 60 .. 5000), all forms of each timed.  Over 5616 other launches (N from 20) the choice is 4 - 5 % faster than the choice without this
// form, causal at d = 128 2.4 %; 7 of them are more than 3 % slower, at worst 9 % (1792/224 causal heads x 245), and up to 2.4 % more could
// be had.  It pays where the launch has more tiles than CUs and short to middling
// chains, whose first loads, first block and stores then run beside another workgroup's steps; us, otherwise -> paired:
// d = 64 causal 192 heads x 327 16.0 -> 10.9, 512 x 903 110 -> 86; few tiles (32 heads x 1000, keys split) 13.6 -> 15.6;
// d = 128 384 x 400 47.2 -> 48.9, 96 x 1962 causal 105.1 -> 110.7, and long launches
// up to 8 % slower (every workgroup reads K and V for 128 queries instead of 256): those keep their form, as do causal launches like
// 128/64 x 568 25.6 -> 29.8, d = 64 72/36 x 1050 24.1 -> 28.0.
bool pair_pays(const AttnParams& p, int d, bool split) {
  static const AttnFormCost cost[2][2][3] = {  // [d = 128][causal][whole, split, paired]
      {{{0.98, 3.44, 0.469, 0.100, 1.00}, {0.85, 4.00, 0.496, 0.300, 1.00}, {0.67, 3.89, 0.319, 0.220, 0.24}},
       {{1.70, 3.01, 0.433, 0.300, 1.13}, {1.16, 3.98, 0.466, 0.200, 0.94}, {1.51, 3.39, 0.316, 0.140, 4.44}}},
      {{{0.36, 4.88, 0.730, 0.200, 1.00}, {0.00, 6.01, 0.762, 0.300, 1.00}, {0.33, 5.35, 0.413, 0.420, 0.38}},
       {{0.18, 5.60, 0.628, 0.300, 1.08}, {0.00, 6.58, 0.651, 0.093, 1.08}, {0.00, 6.05, 0.406, 0.182, 3.44}}}};
  const AttnFormCost* const c = cost[d == 128][p.causal != 0];
  const double heads = (double)p.B * p.Hq, steps = (p.N + 31) / 32;
  auto us = [&](const AttnFormCost& f, int bm, int slots, double part) {
    const double T = (p.N + bm - 1) / bm;
    const double mean = p.causal ? ((T - 1.0) * 0.5 * (bm / 32) + steps / T) : steps;
    return form_us(f, p.causal != 0, heads * T, slots, part < 1.0 ? 0.5 * (steps + 1.0) : steps, part * mean);
  };
  const double n = heads * ((p.N + 127) / 128);
  if (n > (1 << 22) || (p.causal && n <= 256.0) || steps > (d == 64 ? 128 : 64)) return false;
  const double other = split ? us(c[1], 128, 1, 0.5) : us(c[0], 256, 1, 1.0), whole = heads * ((p.N + 255) / 256);
  // (a causal launch of 1.35 - 2 rounds of whole tiles is better than the model says: the light tiles of the second round
  // fill up behind the heavy ones of the first)
  const double margin = !p.causal ? 0.97 : whole > 345.0 && whole <= 512.0 ? 0.90 : d == 64 ? 0.94 : 0.95;
  return us(c[2], 128, d == 64 ? kPairSlots<64> : kPairSlots<128>, 1.0) < margin * other;
}

// the launch in tiles of 128 queries
AttnParams in_tiles_of_128(const AttnParams& p) {
  AttnParams q = p;
  q.T = (p.N + 127) / 128;
  q.total = p.B * p.Hq * q.T;
  q.map = attn_tile_map_make(p.B, p.Hq, p.Hkv, q.T, p.causal);
  return q;
}

template <int D, int FORM>
int launch_128(const AttnParams& p, int, hipStream_t stream) {
  const AttnParams q = in_tiles_of_128(p);
  const dim3 grid(q.total), block(FORM == kPair ? 256 : 512);
  if (p.causal) hipLaunchKernelGGL((attn_fwd_sp_kernel<D, true, 0, false, FORM>), grid, block, 0, stream, q);
  else hipLaunchKernelGGL((attn_fwd_sp_kernel<D, false, 0, false, FORM>), grid, block, 0, stream, q);
  return (int)hipGetLastError();
}

template <int D, bool FP8>
int launch_whole(const AttnParams& p, int grid, hipStream_t stream) {
  const int resident = resident_workgroups();
  if (resident >= 8 && lists_pay(p, grid, resident)) {
    AttnParams q = p;
    q.total = grid;
    if (p.causal) hipLaunchKernelGGL((attn_fwd_sp_kernel<D, true, 2, FP8>), dim3(resident), dim3(512), 0, stream, q);
    else hipLaunchKernelGGL((attn_fwd_sp_kernel<D, false, 2, FP8>), dim3(resident), dim3(512), 0, stream, q);
  } else if (p.causal) {
    hipLaunchKernelGGL((attn_fwd_sp_kernel<D, true, 0, FP8>), dim3(grid), dim3(512), 0, stream, p);
  } else {
    hipLaunchKernelGGL((attn_fwd_sp_kernel<D, false, 0, FP8>), dim3(grid), dim3(512), 0, stream, p);
  }
  return (int)hipGetLastError();
}

template <int D, bool FP8>
int launch_sp(const AttnParams& p, int grid, hipStream_t stream) {
  if constexpr (!FP8) {
    const bool split = split_pays(p, grid);
    if (pair_pays(p, D, split)) return launch_128<D, kPair>(p, grid, stream);
    if (split) return launch_128<D, kSplit>(p, grid, stream);
  }
  return launch_whole<D, FP8>(p, grid, stream);
}

// zero the 8 list counters (a kernel, not a memset, so that the pair can be captured in a graph)
__global__ void attn_queue_reset_kernel(int* queue) {
  if (threadIdx.x < 8) queue[threadIdx.x * 32] = 0;
}

template <int D, int FORM>
void launch_resident(const AttnParams& p, int workgroups, hipStream_t stream) {
  const dim3 grid(workgroups < p.total ? workgroups : p.total), block(FORM == kPair ? 256 : 512);
  if (p.causal) hipLaunchKernelGGL((attn_fwd_sp_kernel<D, true, 1, false, FORM>), grid, block, 0, stream, p);
  else hipLaunchKernelGGL((attn_fwd_sp_kernel<D, false, 1, false, FORM>), grid, block, 0, stream, p);
}

// The form is the one that attn_fwd takes.  Launches that are few enough tiles for split keys (run paired where that is faster
// still) leave the queue alone, all others drain it: one whole-tile workgroup per CU, or as many paired ones as share a CU.
template <int D>
int launch_queue(const AttnParams& p, int cus, hipStream_t stream) {
  const bool split = split_pays(p, p.total), pair = pair_pays(p, D, split);
  if (pair && (split || in_tiles_of_128(p).total <= cus * kPairSlots<D>)) return launch_128<D, kPair>(p, 0, stream);
  if (split) return launch_128<D, kSplit>(p, 0, stream);
  hipLaunchKernelGGL(attn_queue_reset_kernel, dim3(1), dim3(64), 0, stream, p.queue);
  if (pair) launch_resident<D, kPair>(in_tiles_of_128(p), cus * kPairSlots<D>, stream);
  else launch_resident<D, kWhole>(p, cus, stream);
  return (int)hipGetLastError();
}

}  // namespace

int attn_fwd_bf16_persistent_launch(const AttnParams& p, int d, int cus, hipStream_t stream) {
  if (!p.queue || p.total <= 0 || cus <= 0 || (d != 128 && d != 64)) return -1;
  return d == 128 ? launch_queue<128>(p, cus, stream) : launch_queue<64>(p, cus, stream);
}

const AttnVariant* attn_sp_variants(int* count) {
  static const AttnVariant table[] = {
      {"bf16 d128 pipelined BM256 BN64", 0, 128, 256, 64, 512, 2 * 3 * 64 * 128 * 2, launch_sp<128, false>},
      {"bf16 d64 pipelined BM256 BN64", 0, 64, 256, 64, 512, 2 * 3 * 64 * 64 * 2, launch_sp<64, false>},
      {"fp8 d128 fp8-QK bf16-PV pipelined BM256 BN64", 1, 128, 256, 64, 512, 3 * 64 * 128 + 3 * 64 * 256 + 2 * 64 * 128, launch_sp<128, true>},
  };
  *count = (int)(sizeof(table) / sizeof(table[0]));
  return table;
}

const AttnVariant* attn_sp_forms(int* count) {
  static const AttnVariant table[] = {
      {"bf16 d128 whole tiles BM256 BN64", 0, 128, 256, 64, 512, 2 * 3 * 64 * 128 * 2, launch_whole<128, false>},
      {"bf16 d64 whole tiles BM256 BN64", 0, 64, 256, 64, 512, 2 * 3 * 64 * 64 * 2, launch_whole<64, false>},
      {"bf16 d128 split keys BM128 BN64", 0, 128, 128, 64, 512, 2 * 4 * 64 * 128 * 2, launch_128<128, kSplit>},
      {"bf16 d64 split keys BM128 BN64", 0, 64, 128, 64, 512, 2 * 4 * 64 * 64 * 2, launch_128<64, kSplit>},
      {"bf16 d128 paired BM128 BN32", 0, 128, 128, 32, 256, 2 * 4 * 32 * 128 * 2, launch_128<128, kPair>},
      {"bf16 d64 paired BM128 BN32", 0, 64, 128, 32, 256, 2 * 4 * 32 * 64 * 2, launch_128<64, kPair>},
  };
  *count = (int)(sizeof(table) / sizeof(table[0]));
  return table;
}

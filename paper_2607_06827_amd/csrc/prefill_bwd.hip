// Backward of the attention over the compressed cache (arXiv 2607.06827,
// Sec. III-B, Eq. 5 under the causal mask over compressed positions; Sec.
// III-C: training runs the pooling inside the forward pass and optimises it
// jointly, so the gradient reaches Q, the pooled K^/V^ and, through them, the
// raw K/V and the gate).
//
// With P = softmax(scale Q K^T) under the mask, O = P V and the gradient dO:
//   dP      = dO V^T,   Delta_p = sum_c P_pc dP_pc  (= dO_p . O_p exactly)
//   dZ      = P o (dP - Delta)
//   dQ      = scale dZ K^,   dK^ = scale dZ^T Q,   dV^ = P^T dO
// Delta is formed from P and dP in fp32, not from the stored output: a row
// that sees few keys has dZ = P (dP - Delta) nearly cancelling, and the bf16
// rounding of O would otherwise dominate its dQ.
// P is recomputed from the forward's log-sum-exp, so nothing of size
// queries x keys is stored.  Two kernels, each owning its output so that
// nothing is accumulated across blocks:
//
// dQ kernel - the forward's tiling: a block owns one (sequence, KV head) and
//   32*RB query rows for the G query heads; per 32-key tile
//     S^T = K Q^T,  dP^T = V dO^T          (keys x queries, one query per lane)
//     dQ^T += K^T dZ0^T,  Kbar^T += K^T P^T (K^T read transposed from the K tile)
//   in one pass, with dZ0 = P o (dP - Delta0) for Delta0 = dO . O from the
//   stored output; the exact Delta accumulates beside it, and at the end
//   dQ = scale (dZ0 K^ + (Delta0 - Delta) Kbar), Kbar = P K^.  It saves
//   Delta for:
// dK/dV kernel - a block owns a few keys (16 in fp32, 64 or 32 in bf16) of one
//   (sequence, KV head) and walks the (query head, query tile) steps that see
//   them; each step's Q / dO tile is staged in LDS by direct loads, K and V
//   held in registers
//     S = Q K^T,  dP = dO V^T               (queries x keys, one key per lane)
//     dV^T += dO^T P,  dK^T += Q^T dZ        (dO^T, Q^T read transposed)
//   starting S and dP from -LSE/scale and -Delta of their rows.
// The fp32 dK/dV kernel runs every product on the 16x16x4 fp32 MFMA (the fp32
// dQ kernel is in prefill_f32.hip).  The bf16 kernels keep this split and these
// formulas on the 16x16x32 bf16 MFMA with small per-wave tiles (16 query rows,
// or 16 keys, a wave), so that three waves or more share each SIMD (two in the
// dK/dV blocks of 32 keys at d = 128, whose buffers fill the LDS); P and dZ are
// rounded to bf16 as MFMA operands, every product accumulates in fp32, and
// dK^ and dV^ are written in fp32.
// The mask's visibility rule comes from the span view (spans.hpp): one run
// per sequence, or the runs of a segment table (kRuns).
#include <climits>
#include <type_traits>

#include "attn_mfma.hpp"
#include "kernels.hpp"
#include "kernels_bwd.hpp"

namespace skv {

namespace {

constexpr float kLog2eF = 1.4426950408889634f;

__device__ __forceinline__ float frag_dot(bf16x8_t x, bf16x8_t y) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) s = __builtin_fmaf((float)x[i], (float)y[i], s);
  return s;
}

// --------------------------------------------------------------- dK / dV

// bf16 tiles (Q and dO in dK/dV, K and V in dQ): 32 unpadded rows in LDS, filled by
// direct loads (global_load_lds: a wave-wide load writes 64 x 16 bytes in
// lane order), 16-byte chunks XOR-swizzled within a row: chunk c of row r sits
// at position c ^ swz(r), so the operand reads of 16 rows at one chunk hit
// distinct banks.
template <int D>
struct QTile {
  static constexpr int kChunks = D / 8;                     // 16-byte chunks per row
  static constexpr int kRowsPerLoad = 64 / kChunks;         // rows per wave-wide load
  static constexpr int kLoads = 32 / kRowsPerLoad;          // wave-wide loads per tile
  static constexpr int kElems = 32 * D;
  // XOR swizzle of the 16-byte chunks of row r.  With 16 chunks per row
  // (D = 128: a row spans the 64 banks once) the tile is read both
  // transposed (ds_read_b64_tr_b16: 8 consecutive rows x 2 neighbouring
  // chunks per 32 lanes, so bits 1-3 differ over 8 consecutive rows) and
  // row-wise (16x16x32 A operands: lane group g reads rows 0-15 at chunk 4c +
  // g).  A 16-byte read takes 16 lanes at a time, lanes 0-3, 12-15 of one group
  // with lanes 4-11 of the next: rows 0-3, 12-15 at one chunk with rows 4-11
  // at its neighbour.  So the rows whose swizzles differ in bit 0 only are r
  // and r ^ 12, both of one of these sets, and the 16 positions stay
  // distinct.  (Paired r with r ^ 8, every row-wise read was a 2-way
  // conflict: 2.0 conflict cycles per LDS instruction in dQ.)
  static __device__ __forceinline__ int swz(int r) {
    if constexpr (kChunks == 16) return (((r ^ ((r >> 1) & 4)) & 7) << 1) | ((r >> 3) & 1);
    return r & (kChunks - 1);
  }
};

// Item of block bid in a dK/dV grid of nblk blocks over pairs x T key blocks
// (items pair-major, pair = (sequence, KV head)).  The work of key block kt
// falls with kt (later keys are seen by fewer query rows).  XCD x (= bid mod
// 8) runs a contiguous item range; its blocks fill its 32 CUs one round at
// a time, so local blocks i, i + 32, ... share a CU while they are resident
// together.  A pair whose first item opens an odd round of its XCD takes its
// key blocks in descending order, which pairs the heavy blocks of one round
// with the light ones of the next on each CU (at 1596 x 471, b = 8: 12%
// less time than ascending order everywhere).  The order is reversed within
// whole pairs, so every item is still run exactly once.
constexpr int kCusPerXcd = 32;
constexpr int kCus = 8 * kCusPerXcd;
__device__ __forceinline__ void dkdv_item(int bid, int nblk, int T, int& pair, int& kt) {
  const int xcd = bid & 7, per = nblk >> 3, rem = nblk & 7;
  const int item = xcd * per + min(xcd, rem) + (bid >> 3);
  pair = item / T;
  const int kt0 = item - pair * T;
  // the XCD range holding the pair's first item, and that item's place in it
  const int first = pair * T;
  const int x = first < rem * (per + 1) ? first / (per + 1) : rem + (first - rem * (per + 1)) / max(per, 1);
  const int local = first - (x * per + min(x, rem));
  kt = ((local / kCusPerXcd) & 1) ? T - 1 - kt0 : kt0;
}

// Heaviest-first order: block bid takes key block bid / pairs of pair bid %
// pairs, so the first key blocks (which most query rows see) of every pair
// start first and the lightest last, and when the pairs split evenly over the
// eight XCDs every key block of a pair runs on the same one.
__device__ __forceinline__ void dkdv_item_heaviest_first(int bid, int pairs, int& pair, int& kt) {
  kt = bid / pairs;
  pair = bid - kt * pairs;
}

// -------------------------------------------- dK / dV, fp32, 16 keys a block
//
// A block owns 16 keys of one (sequence, KV head); its kWaves waves deal the
// (query head, 16-row query tile) steps that see them round, each wave with
// two tile buffers of its own (Q and dO rows, LSE, Delta) filled by untracked
// direct loads one step ahead: no barrier until the waves' sums are added, in
// a fixed order, through LDS at the end.  Per step a wave computes on the
// 16x16x4 fp32 MFMA
//   S = Q K^T - LSE/scale,  dP = dO V^T - Delta     (rows x keys)
//   P = exp2(scale log2e S),  dZ = P dP     (masked)
//   dV^T += dO^T P,  dK^T += Q^T dZ          (d x keys, 16-row blocks of d)
// The k index of a product is free as long as both operands agree on it: S
// and dP take elements 16c + 4g + t from lane group g for MFMA t, so a row's
// operands are 16-byte reads, and the C layout (rows 4g + i in group g) makes
// P and dZ their own B operands with row 4g + t for MFMA t.
//
// Bound by the fp32 MFMA once the chip is full; few sequences leave it idle,
// and then what counts is the longest chain of steps of a wave.  Blocks of
// 128 keys, 32 a wave, ran every step of a key in one wave: at 632 x 182 (b =
// 4, 8/4 heads of 64) 32 blocks took 193 us, and 128-wide heads spilled.
template <int D>
struct KvBwdShapeF32 {
  static constexpr int kWaves = D == 128 ? 4 : 8;  // two 8 KB (16 KB) tile pairs a wave in 160 KB
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kKeys = 16;
};

// the swizzle of the fp32 tiles' 16-byte chunks: a permutation of 16 rows
// (row-wise reads of 16 rows at one chunk hit distinct banks) that puts rows
// 4g + t of the four lane groups in distinct quarters (the transposed reads
// of 4 rows x 16 columns hit 64 distinct banks)
__device__ __forceinline__ int swz_f32(int r) { return r & 15; }

template <int D, bool kRuns>
__global__ __launch_bounds__(KvBwdShapeF32<D>::kThreads, KvBwdShapeF32<D>::kWaves / 4) void prefill_bwd_dkdv_f32_kernel(
    PrefillBwdArgs a) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  constexpr int kWaves = KvBwdShapeF32<D>::kWaves;
  constexpr int kQ = 16;                        // query rows per step
  constexpr int kDB = D / 16;                   // 16-element blocks of d
  constexpr int kChunks = D / 4;                // 16-byte chunks per row
  constexpr int kRowsPerLoad = 64 / kChunks;    // rows one wave-wide direct load fills
  constexpr int kLoads = kQ / kRowsPerLoad;     // direct loads per matrix and step
  constexpr int kVm = 2 * kLoads + 1;           // (+1: LSE and Delta)

  struct __attribute__((aligned(256))) Buf {
    float q[kQ * D];
    float g[kQ * D];
    float l[64];  // LSE of the rows at 0.., Delta at 32..
  };
  __shared__ Buf s_buf[kWaves][2];

  const int heads = a.pv.kv_heads;
  int pair, kt;
  dkdv_item_heaviest_first(blockIdx.x, gridDim.x / a.num_key_tiles, pair, kt);
  const int g = pair % heads;
  const int b = pair / heads;

  const auto sp = span_view<kRuns>(a, b, a.w_eff);
  const int rows = min(sp.rows(), a.q_len);
  const int clen = min(min(sp.clen(), a.pv.max_pages << a.pv.page_shift), a.hat_cap);
  const int kb0 = kt * kQ;
  if (kb0 >= clen || rows == 0) return;  // block-uniform

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int gq = lane >> 4, j = lane & 15;  // lane group, column of the 16x16 C layout
  const int hq = a.num_q_heads;
  const int group = hq / heads;
  const int gshift = __builtin_ctz(group);  // (a power of two)
  const int key = kb0 + j;
  const int tau = key < clen ? sp.visible_from(key, a.mask_mode) : INT_MAX;
  // the first row that sees a key of the block, and the row from which on all
  // its keys are visible
  const int q_first = sp.visible_from(kb0, a.mask_mode);
  const int q_all = sp.visible_from(min(kb0 + 15, clen - 1), a.mask_mode);

  // K and V of this lane's key, elements 16c + 4gq .. +3 (a key past the
  // cache or without a page is zero)
  f32x4 kf[kDB], vf[kDB];
  {
    const int shift = a.pv.page_shift;
    const int32_t e = a.table[(int64_t)b * a.pv.max_pages + min(key >> shift, a.pv.max_pages - 1)];
    const bool ok = key < clen && e >= 0 && e < a.pv.num_pages;
    const int64_t off = page_row<D>(ok ? e : 0, g, key & ((1 << shift) - 1), a.pv) + 4 * gq;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < kDB; ++c) {
      const f32x4 k = *reinterpret_cast<const f32x4*>(static_cast<const float*>(a.k_pages) + off + 16 * c);
      const f32x4 v = *reinterpret_cast<const f32x4*>(static_cast<const float*>(a.v_pages) + off + 16 * c);
      kf[c] = ok ? k : zero;
      vf[c] = ok ? v : zero;
    }
  }

  // steps: (query head, 16-row tile) pairs, last rows first, so that the
  // blocks of a (sequence, KV head) read the same tiles at the same time
  const int t0 = q_first / kQ, t1 = (rows + kQ - 1) / kQ;
  const int n_steps = max(t1 - t0, 0) << gshift;
  const int rlast = rows - 1;
  const int lrow = lane / kChunks, lpos = lane % kChunks;
  const uint64_t row_bytes = (uint64_t)hq * D * sizeof(float);
  auto load_step = [&](int n, Buf& bf) __attribute__((always_inline)) {
    const int h = g * group + (n & (group - 1));
    const int q0 = (t1 - 1 - (n >> gshift)) * kQ;
    const uint64_t base_off = (((uint64_t)b * a.q_len + q0) * hq + h) * D * sizeof(float);
    const char* qb = static_cast<const char*>(a.q) + base_off;
    const char* gb = static_cast<const char*>(a.dout) + base_off;
#pragma unroll
    for (int l = 0; l < kLoads; ++l) {
      const int r = l * kRowsPerLoad + lrow;  // (rows past the end read the last row: finite, and masked)
      const uint32_t off = (uint32_t)((uint64_t)(min(q0 + r, rlast) - q0) * row_bytes) + ((lpos ^ swz_f32(r)) << 4);
      lds_dma16(qb, off, lds_addr(bf.q + l * kRowsPerLoad * D));
      lds_dma16(gb, off, lds_addr(bf.g + l * kRowsPerLoad * D));
    }
    const float* src = lane < 32 ? a.lse : a.delta;
    const int64_t stat = ((int64_t)b * hq + h) * a.q_len + min(q0 + j, rlast);
    lds_dma4(src + stat, lds_addr(bf.l));
  };

  f32x4 dk[kDB], dv[kDB];
#pragma unroll
  for (int db = 0; db < kDB; ++db)
#pragma unroll
    for (int i = 0; i < 4; ++i) dk[db][i] = dv[db][i] = 0.f;
  const float neg_inv_scale = -1.f / a.scale;

  auto compute = [&](int n, const Buf& bf) __attribute__((always_inline)) {
    const int q0 = (t1 - 1 - (n >> gshift)) * kQ;
    // S and dP accumulators start from -LSE/scale and -Delta of their rows
    const f32x4 lv = *reinterpret_cast<const f32x4*>(bf.l + 4 * gq);
    const f32x4 dl = *reinterpret_cast<const f32x4*>(bf.l + 32 + 4 * gq);
    f32x4 s, dp;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[i] = lv[i] * neg_inv_scale;
      dp[i] = -dl[i];
    }
#pragma unroll
    for (int c = 0; c < kDB; ++c) {
      const int at = j * D + (((4 * c + gq) ^ swz_f32(j)) << 2);
      const f32x4 qa = *reinterpret_cast<const f32x4*>(bf.q + at);
      const f32x4 ga = *reinterpret_cast<const f32x4*>(bf.g + at);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        s = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[t], kf[c][t], s, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_16x16x4f32(ga[t], vf[c][t], dp, 0, 0, 0);
      }
    }
    float pv[4], zv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) pv[i] = fast_exp2(s[i] * a.scale_log2);
    if (q0 < q_all || q0 + kQ > rows) {  // uniform: some row or key masked
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = q0 + 4 * gq + i;
        const bool vis = r >= tau && r < rows;
        pv[i] = vis ? pv[i] : 0.f;
        dp[i] = vis ? dp[i] : 0.f;
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) zv[i] = pv[i] * dp[i];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int r = 4 * gq + t;
#pragma unroll
      for (int db = 0; db < kDB; ++db) {
        const int at = r * D + (((4 * db + (j >> 2)) ^ swz_f32(r)) << 2) + (j & 3);
        dv[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(bf.g[at], pv[t], dv[db], 0, 0, 0);
        dk[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(bf.q[at], zv[t], dk[db], 0, 0, 0);
      }
    }
  };

  // wave w takes steps w, w + kWaves, ...; its own loads only, so a count of
  // them is all it waits for (the first wait covers the K/V loads too)
  Buf& b0 = s_buf[wave][0];
  Buf& b1 = s_buf[wave][1];
  // The steps of the last query tile, where it is ragged: there the dO rows past
  // the end, copies of the last one, are cleared (an infinite one would meet its
  // zero weights in dV as 0 * infinity).  Out of line, the check costs 0% at d =
  // 64 and 1% at d = 128; as a first step before the loop, whose code short
  // chains fetch once more, up to 8%.
  const int clear_steps = rows % kQ ? group : 0;
  auto step = [&](int n, Buf& cur, Buf& nxt) __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(63));  // the last step's LDS reads are done before nxt is refilled
    asm volatile("" ::: "memory");
    if (n + kWaves < n_steps) {
      load_step(n + kWaves, nxt);
      __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(kVm));
    } else {
      __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(0));
    }
    asm volatile("" ::: "memory");
    if (__builtin_expect(n < clear_steps, false)) {
      for (int i = (rows - (t1 - 1) * kQ) * kChunks + lane; i < kQ * kChunks; i += 64)
        *reinterpret_cast<f32x4*>(cur.g + 4 * i) = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __builtin_amdgcn_sched_barrier(0);
    compute(n, cur);
  };
  if (wave < n_steps) load_step(wave, b0);
  for (int n = wave; n < n_steps; n += 2 * kWaves) {
    step(n, b0, b1);
    if (n + kWaves < n_steps) step(n + kWaves, b1, b0);
  }

  // the waves' sums through their own (idle) buffers: plane (dK or dV, 16-row
  // block of d) of 64 lanes x 4 values, each plane added up by one wave
  constexpr int kPlanes = 2 * kDB;
  static_assert(kPlanes * 256 * sizeof(float) <= 2 * sizeof(Buf), "a wave's sums fit its buffers");
  asm volatile("" ::: "memory");
  {
    f32x4* mine = reinterpret_cast<f32x4*>(&s_buf[wave][0]);
#pragma unroll
    for (int db = 0; db < kDB; ++db) {
      mine[(2 * db) * 64 + lane] = dk[db];
      mine[(2 * db + 1) * 64 + lane] = dv[db];
    }
  }
  __syncthreads();
  if (key >= clen) return;
  const int64_t row = (((int64_t)b * a.hat_cap + key) * heads + g) * D + 4 * gq;
#pragma unroll
  for (int k = 0; k < kPlanes / kWaves; ++k) {
    const int plane = wave + k * kWaves;  // 2 db + (0: dK, 1: dV)
    f32x4 sum = reinterpret_cast<const f32x4*>(&s_buf[0][0])[plane * 64 + lane];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) sum += reinterpret_cast<const f32x4*>(&s_buf[w][0])[plane * 64 + lane];
    const bool is_v = plane & 1;
    const float sc = is_v ? 1.f : a.scale;
    *reinterpret_cast<float4*>((is_v ? a.dv_hat : a.dk_hat) + row + 16 * (plane >> 1)) =
        make_float4(sum[0] * sc, sum[1] * sc, sum[2] * sc, sum[3] * sc);
  }
}

// ---------------------------------------------------- dQ, bf16, 16 rows a wave
//
// The bf16 dQ kernel on the 16x16x32 MFMA.  A wave owns 16 query rows of one
// query head and keeps their Q and dO operands in registers; a block of
// kWaves waves owns 16 * kWaves / G rows of one (sequence, KV head) for all G
// heads and streams the 32-key tiles they see through LDS (three buffers,
// untracked direct loads two tiles ahead, as in the forward).  Per tile a
// wave computes, keys as rows of the 16x16 blocks (so that P and dZ0 are
// their own B operands, as in the dK/dV kernel):
//   S^T = K Q^T,  dP^T = V dO^T       (two 16-key blocks)
//   P = exp2(scale log2e S - log2e LSE),  dZ0 = P (dP - Delta0)
//   dQ^T += K^T dZ0^T,  Kbar^T += K^T P^T    (16-row blocks of d)
// with Delta0 = dO . O (the stored output) and the exact Delta = sum P dP
// beside it; at the end dQ = scale (dZ0 K + (Delta0 - Delta) Kbar).
template <int G>
struct DqShape16 {
  static constexpr int kRowBlocks = G >= 4 ? 1 : 4 / G;
  static constexpr int kWaves = G * kRowBlocks;
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kRows = 16 * kRowBlocks;
};

template <int D, int G, bool kRuns>
__global__ __launch_bounds__(DqShape16<G>::kThreads, 3) void prefill_bwd_dq16_kernel(PrefillBwdArgs a) {
  typedef bf16_bits T;
  typedef QTile<D> Q;  // the K and V tiles: 32 rows, chunks swizzled per row
  typedef bf16x8_t Frag;
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  constexpr int kWaves = DqShape16<G>::kWaves;
  constexpr int kRows = DqShape16<G>::kRows;
  constexpr int kKeys = 32;
  constexpr int kDC = D / 32;  // K-dim chunks of S^T and dP^T
  constexpr int kDB = D / 16;  // 16-row blocks of dQ^T and Kbar^T
  constexpr int kLoadsPerWave = Q::kLoads >= kWaves ? Q::kLoads / kWaves : 1;
  static_assert(Q::kLoads % kWaves == 0 || kWaves % Q::kLoads == 0, "loads split evenly over waves");
  constexpr int kVm = 2 * kLoadsPerWave;

  __shared__ __attribute__((aligned(256))) T s_k0[Q::kElems];
  __shared__ __attribute__((aligned(256))) T s_k1[Q::kElems];
  __shared__ __attribute__((aligned(256))) T s_k2[Q::kElems];
  __shared__ __attribute__((aligned(256))) T s_v0[Q::kElems];
  __shared__ __attribute__((aligned(256))) T s_v1[Q::kElems];
  __shared__ __attribute__((aligned(256))) T s_v2[Q::kElems];

  // XCD-aware, heaviest-first item order (as in the forward)
  int pair, tile;
  query_tile_item(blockIdx.x, gridDim.x, a.num_q_tiles, pair, tile);
  const int heads = a.pv.kv_heads;
  const int g = pair % heads;
  const int b = pair / heads;
  const int p0 = tile * kRows;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int gq = lane >> 4, j = lane & 15;
  const int h = g * G + wave % G;
  const int wrow0 = p0 + (wave / G) * 16;  // first row of this wave
  const int q = wrow0 + j;                 // this lane's row (column of the C layout)
  const int hq = a.num_q_heads;

  // this lane's row of Q, dO and O (elements 32c + 8gq .. +7, the B operand
  // layout of S^T = K Q^T) and its LSE: the rows do not depend on the span
  // lengths, so with one run they are requested first and are in flight
  // during the span and block-table round trips (a row past the tensor reads
  // its last row: in range, never stored); a segment table's scan comes
  // first (its tracked loads' waits would take these along)
  Frag qf[kDC], gf[kDC], of[kDC];
  float lse = 0.f;
  auto load_rows = [&]() __attribute__((always_inline)) {
    const int qr = min(q, a.q_len - 1);
    const int64_t row = ((int64_t)b * a.q_len + qr) * hq + h;
    const T* qp = static_cast<const T*>(a.q) + row * D + 8 * gq;
    const T* gp = static_cast<const T*>(a.dout) + row * D + 8 * gq;
    const T* op = static_cast<const T*>(a.out) + row * D + 8 * gq;
    static_for<kDC>([&](auto c) {
      constexpr int kC = decltype(c)::value;
      untracked_load16<kC * 64>(qf[kC], qp);
      untracked_load16<kC * 64>(gf[kC], gp);
      untracked_load16<kC * 64>(of[kC], op);
    });
    const float* lp = a.lse + ((int64_t)b * hq + h) * a.q_len + qr;
    asm volatile("global_load_dword %0, %1, off" : "=v"(lse) : "v"(lp) : "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  if constexpr (!kRuns) load_rows();

  const auto sp = span_view<kRuns>(a, b, a.w_eff);
  const int rows = min(sp.rows(), a.q_len);
  const int clen = min(sp.clen(), a.pv.max_pages << a.pv.page_shift);
  if (p0 >= rows) {
    // the row loads land before the wave ends (with one run they were
    // issued above; an asm statement ahead of a segment scan would turn its
    // scalar loads into vector loads)
    if constexpr (!kRuns) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    return;
  }
  const int kmax = min(sp.visible(min(p0 + kRows, rows) - 1, a.mask_mode), clen);
  const int kclamp = max(kmax - 1, 0);  // last visible key: the row loaded for keys past kmax

  const bool qvalid = q < rows;
  const int nvis = qvalid ? min(sp.visible(q, a.mask_mode), clen) : 0;
  const int nvis_lo = wrow0 < rows ? min(sp.visible(wrow0, a.mask_mode), clen) : 0;
  const int shift = a.pv.page_shift, slot_mask = (1 << shift) - 1;
  const int32_t* table_row = a.table + (int64_t)b * a.pv.max_pages;
  const int ntiles = (kmax + kKeys - 1) / kKeys;
  const bool loads = Q::kLoads >= kWaves || wave < Q::kLoads;
  auto load_row0 = [&](int i) { return (Q::kLoads >= kWaves ? wave * kLoadsPerWave + i : wave) * Q::kRowsPerLoad; };
  const int lrow = lane / Q::kChunks, lpos = lane % Q::kChunks;
  if constexpr (kRuns) load_rows();  // after every segment scan

  // block-table entries: one per wave and tile (the forward's scheme)
  constexpr int kWaveRows = kLoadsPerWave * Q::kRowsPerLoad;
  static_assert(kWaveRows <= 8, "one page holds a wave's rows of a tile");
  const int wrow_load = loads ? load_row0(0) : 0;
  typedef __attribute__((address_space(4))) const int32_t* const_ptr;
  auto table_load = [&](int kt) __attribute__((always_inline)) {
    const int row0 = min(kt * kKeys + wrow_load, kclamp);
    return ((const_ptr)table_row)[min(row0 >> shift, a.pv.max_pages - 1)];
  };
  const uint64_t head_bytes = (uint64_t)D * sizeof(T) << shift;
  const uint64_t page_bytes = head_bytes * heads;
  const uintptr_t kpool_g = (uintptr_t)a.k_pages + (uint64_t)g * head_bytes;
  const uintptr_t v_minus_k = (uintptr_t)a.v_pages - (uintptr_t)a.k_pages;
  const uint32_t npages = (uint32_t)a.pv.num_pages;
  auto tile_load = [&](int kt, int e, T* sk, T* sv) __attribute__((always_inline)) {
    if (!loads) return;
    const uint32_t page = (uint32_t)e < npages ? (uint32_t)e : 0u;  // a bad entry reads an in-range page
    const uintptr_t kbase = kpool_g + (uint64_t)page * page_bytes;
    const uintptr_t vbase = kbase + v_minus_k;
#pragma unroll
    for (int i = 0; i < kLoadsPerWave; ++i) {
      const int r = load_row0(i) + lrow;
      const int key = min(kt * kKeys + r, kclamp);
      const uint32_t off = (uint32_t)((key & slot_mask) * D * 2) + ((lpos ^ Q::swz(r)) << 4);
      lds_dma16((const void*)kbase, off, lds_addr(sk + load_row0(i) * D));
      lds_dma16((const void*)vbase, off, lds_addr(sv + load_row0(i) * D));
    }
  };

  f32x4 dq[kDB], kbar[kDB];
#pragma unroll
  for (int db = 0; db < kDB; ++db)
#pragma unroll
    for (int i = 0; i < 4; ++i) dq[db][i] = kbar[db][i] = 0.f;
  float dsum = 0.f;  // this lane's share of Delta = sum over keys of P dP

  // prologue: the row operands (issued above), tiles 0 and 1; wait for the
  // operands and tile 0
  int pg[3] = {table_load(0), table_load(1), table_load(2)};
  tile_load(0, pg[0], s_k0, s_v0);
  if (ntiles > 1 && loads) {
    tile_load(1, pg[1], s_k1, s_v1);
    bare_barrier<kVm>();
  } else {
    // (a wave that loads no tile rows has only its row operands in flight:
    // it waits for all of them)
    bare_barrier<0>();
  }
  // Delta0 = dO . O over the row: the lane's 32 products, then the four lane
  // groups that share the row
  float delta0 = 0.f;
#pragma unroll
  for (int c = 0; c < kDC; ++c) delta0 += frag_dot(gf[c], of[c]);
  delta0 += __shfl_xor(delta0, 16, 64);
  delta0 += __shfl_xor(delta0, 32, 64);
  const float lse2 = lse * kLog2eF;

  // fragment addresses (bytes), one register per tile and pattern (patterns as
  // in the dK/dV kernel): row-wise operands of S^T / dP^T at ar ^ 64c (+16 rows for
  // the second key block), transposed K^T operands at at ^ 32db (+16 rows)
  const int rr = 4 * gq + (j >> 2);
  const uint32_t ar_off = (uint32_t)(j * D * 2 + ((gq ^ Q::swz(j)) << 4));
  const uint32_t at_off = (uint32_t)(rr * D * 2 + ((((j & 3) >> 1) ^ Q::swz(rr)) << 4) + ((j & 1) << 3));
  typedef __attribute__((address_space(3))) const u16x8_t* lds_frag_ptr;

  auto attend = [&](int kt, const T* sk, const T* sv) __attribute__((always_inline)) {
    uint32_t ar_k = lds_addr(sk) + ar_off, ar_v = lds_addr(sv) + ar_off, at_k = lds_addr(sk) + at_off;
    asm volatile("" : "+v"(ar_k), "+v"(ar_v), "+v"(at_k));
    auto arow = [&](uint32_t base, int blk, int c) __attribute__((always_inline)) {
      return __builtin_bit_cast(Frag, *(lds_frag_ptr)(uintptr_t)((base ^ (uint32_t)(64 * c)) + (uint32_t)(blk * 16 * D * 2)));
    };
    auto atr = [&](int db) __attribute__((always_inline)) {
      const uint32_t al = at_k ^ (uint32_t)(32 * db);
      const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)al);
      const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)(al + 16 * D * 2));
      const u16x8_t v = {(unsigned short)lo[0], (unsigned short)lo[1], (unsigned short)lo[2], (unsigned short)lo[3],
                         (unsigned short)hi[0], (unsigned short)hi[1], (unsigned short)hi[2], (unsigned short)hi[3]};
      return __builtin_bit_cast(Frag, v);
    };
    // S^T and dP^T: rows = keys 16 blk + 4 gq + i of the tile, column = row q
    f32x4 s[2], dp[2];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
      for (int i = 0; i < 4; ++i) s[blk][i] = dp[blk][i] = 0.f;
    constexpr int kNS = 4 * kDC;  // (c, blk, S or dP)
    auto aop = [&](int idx) __attribute__((always_inline)) {
      const int c = idx / 4, blk = (idx / 2) % 2, t = idx % 2;
      return arow(t ? ar_v : ar_k, blk, c);
    };
    constexpr int kAheadS = 3;
    Frag sb[kAheadS];
#pragma unroll
    for (int i = 0; i < kAheadS; ++i) sb[i] = aop(i);
#pragma unroll
    for (int idx = 0; idx < kNS; ++idx) {
      const Frag cur = sb[idx % kAheadS];
      if (idx + kAheadS < kNS) sb[idx % kAheadS] = aop(idx + kAheadS);
      const int c = idx / 4, blk = (idx / 2) % 2;
      if (idx % 2 == 0) s[blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur, qf[c], s[blk], 0, 0, 0);
      else dp[blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur, gf[c], dp[blk], 0, 0, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x100, kAheadS, 0);
#pragma unroll
    for (int idx = 0; idx + kAheadS < kNS; ++idx) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, kAheadS, 0);

    constexpr int kAheadT = 2;
    Frag tb[kAheadT];
#pragma unroll
    for (int i = 0; i < kAheadT; ++i) tb[i] = atr(i);
    __builtin_amdgcn_sched_barrier(0);

    // P and dZ0 in the order of the B operand (element t: key 4gq + t, t < 4,
    // or 16 + 4gq + t - 4); keys past the row's bound get weight 0
    float pv[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) pv[t] = fast_exp2(__builtin_fmaf(s[t / 4][t % 4], a.scale_log2, -lse2));
    const int kb = kt * kKeys;
    if (kb + kKeys > nvis_lo) {  // uniform: the tile straddles some row's bound
      const int lim = nvis - kb - 4 * gq;  // element t is visible iff 16 (t/4) + t%4 < lim
#pragma unroll
      for (int t = 0; t < 8; ++t) pv[t] = 16 * (t / 4) + t % 4 < lim ? pv[t] : 0.f;
    }
    Frag pf, zf;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const float d = dp[t / 4][t % 4];
      dsum = __builtin_fmaf(pv[t], d, dsum);
      pf[t] = (__bf16)pv[t];
      zf[t] = (__bf16)(pv[t] * (d - delta0));
    }
    // dQ^T += K^T dZ0^T and Kbar^T += K^T P^T, one transposed K operand each
#pragma unroll
    for (int db = 0; db < kDB; ++db) {
      const Frag cur = tb[db % kAheadT];
      if (db + kAheadT < kDB) tb[db % kAheadT] = atr(db + kAheadT);
      dq[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur, zf, dq[db], 0, 0, 0);
      kbar[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur, pf, kbar[db], 0, 0, 0);
    }
#pragma unroll
    for (int db = 0; db + kAheadT < kDB; ++db) {
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 1);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 1);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 2 * kAheadT, 1);
  };

  auto tile_step = [&](int kt, auto par) {
    constexpr int kPar = decltype(par)::value;
    constexpr int kNext2 = (kPar + 2) % 3;
    T* const sk = kPar == 0 ? s_k0 : kPar == 1 ? s_k1 : s_k2;
    T* const sv = kPar == 0 ? s_v0 : kPar == 1 ? s_v1 : s_v2;
    const bool more = kt + 2 < ntiles;  // uniform
    if (more) {
      tile_load(kt + 2, pg[kNext2], kNext2 == 0 ? s_k0 : kNext2 == 1 ? s_k1 : s_k2,
                kNext2 == 0 ? s_v0 : kNext2 == 1 ? s_v1 : s_v2);
      if (kt + 3 < ntiles) pg[kPar] = table_load(kt + 3);
    }
    attend(kt, sk, sv);
    if (more) bare_barrier<kVm>();
    else bare_barrier<0>();
  };
  for (int kt = 0; kt < ntiles; kt += 3) {
    tile_step(kt, std::integral_constant<int, 0>());
    if (kt + 1 >= ntiles) break;
    tile_step(kt + 1, std::integral_constant<int, 1>());
    if (kt + 2 >= ntiles) break;
    tile_step(kt + 2, std::integral_constant<int, 2>());
  }

  // Delta over the whole row, then dQ = scale (dZ0 K + (Delta0 - Delta) Kbar)
  float delta = dsum;
  delta += __shfl_xor(delta, 16, 64);
  delta += __shfl_xor(delta, 32, 64);
  const int64_t stat = ((int64_t)b * hq + h) * a.q_len + q;
  if (gq == 0 && qvalid) a.delta[stat] = delta;
  const float sc = a.scale, fix = delta0 - delta;
  // rows leave through LDS (the idle tile buffers, 4 KB per wave: row j,
  // 16-byte chunks swizzled as in the tiles) as 16-byte row stores
  static_assert(kWaves <= 8, "a 16-row half of one tile buffer per wave");
  T* const so = (wave / 2 == 0 ? s_k0 : wave / 2 == 1 ? s_k1 : wave / 2 == 2 ? s_k2 : s_v0) + (wave % 2) * 16 * D;
#pragma unroll
  for (int db = 0; db < kDB; ++db) {
    const int e = 16 * db + 4 * gq;  // first of the lane's four elements
    Mfma<T>::store4(so + j * D + ((((e >> 3) ^ Q::swz(j)) << 3) | (e & 7)),
                    sc * __builtin_fmaf(fix, kbar[db][0], dq[db][0]), sc * __builtin_fmaf(fix, kbar[db][1], dq[db][1]),
                    sc * __builtin_fmaf(fix, kbar[db][2], dq[db][2]), sc * __builtin_fmaf(fix, kbar[db][3], dq[db][3]));
  }
  __syncthreads();
  T* const dqp = static_cast<T*>(a.dq);
#pragma unroll
  for (int r0 = 0; r0 < 16; r0 += Q::kRowsPerLoad) {
    const int r = r0 + lrow, row = wrow0 + r;
    if (row < rows) {
      const uint4 v = *reinterpret_cast<const uint4*>(so + r * D + ((lpos ^ Q::swz(r)) << 3));
      // non-temporal: nothing later in the backward reads dQ (-1%)
      typedef unsigned int nt_u32x4 __attribute__((ext_vector_type(4)));
      __builtin_nontemporal_store(nt_u32x4{v.x, v.y, v.z, v.w},
                                  reinterpret_cast<nt_u32x4*>(dqp + (((int64_t)b * a.q_len + row) * hq + h) * D + lpos * 8));
    }
  }
}

// ----------------------------------------------- dK / dV, bf16, 16 keys a wave
//
// The bf16 dK/dV kernel on the 16x16x32 MFMA: a wave owns 16 keys, so its K
// and V operands (16 VGPRs each at d = 128) and its dK^T and dV^T
// accumulators (32 each) leave room for three waves per SIMD (160 registers, no
// scratch).  kWaves waves form
// a step group with 16 kWaves keys of one (sequence, KV head), and the SG groups
// of a block own the same keys and deal the (query head, 32-row query tile) steps
// that see them round, so a block's chain of steps is 1 / SG of its keys'
// steps; at the end the groups' sums are added through LDS in a fixed order.
// Each step's Q, dO, LSE and Delta are staged once in LDS for its group by
// untracked direct loads, kBufs - 1 steps ahead, as in the forward, and each
// wave reads its MFMA operands four ahead of the products.
// (1596 x 471, b = 8: 77.6 us; 107 with one group.  Timed when SG = 3 took 89, with
// bank conflicts and scratch: read eight ahead at two waves per SIMD and SG = 2
// 91 us; 32 keys a wave on the 32x32x16 MFMA, which halves the LDS reads, spills
// at two waves per SIMD, 105 us.)  Per step a wave computes
//   S  = Q K^T  - LSE/scale    (two 16 x 16 blocks: query rows 0-15, 16-31)
//   dP = dO V^T - Delta
//   P = exp2(scale log2e S),  dZ = P dP     (masked)
//   dV^T += dO^T P,  dK^T += Q^T dZ          (d x keys, 16-row blocks of d)
// The C layout of the 16x16 MFMA gives lane (g, j) (g = lane / 16) rows 4g +
// i (i < 4) and column j; the P.V-type products take their K index (query
// rows) in the order k = 8g + t <-> row 4g + t (t < 4), 16 + 4g + t - 4
// (t >= 4), so P and dZ are their own B operands and dO^T / Q^T come from two
// transposed LDS reads (rows 4g.., 16 + 4g..) per head-dim block.
template <int D, bool kRuns, int kWaves, int SG, int kBufs>
__global__ __launch_bounds__(64 * kWaves * SG, SG == 1 ? 3 : kWaves * SG / 4) void prefill_bwd_dkdv16_kernel(PrefillBwdArgs a) {
  typedef bf16_bits T;
  typedef QTile<D> Q;
  typedef bf16x8_t Frag;
  constexpr int kBlockKeys = 16 * kWaves;
  constexpr int kQ = 32;           // query rows per step
  constexpr int kDC = D / 32;      // K-dim chunks of the S and dP products
  constexpr int kDB = D / 16;      // 16-row blocks of dK^T and dV^T
  constexpr int kLoadsPerWave = 2 * Q::kLoads / kWaves;  // Q and dO direct loads per step
  static_assert((2 * Q::kLoads) % kWaves == 0, "loads split evenly over waves");
  constexpr int kVm = kLoadsPerWave;                     // (+1 for the wave that loads LSE / Delta)

  struct __attribute__((aligned(256))) Buf {
    T q[Q::kElems];
    T g[Q::kElems];
    float l[2 * kQ];  // LSE, Delta
  };
  __shared__ Buf s_buf[SG][kBufs];  // per step group

  int pair, kt;
  if constexpr (SG == 1) dkdv_item(blockIdx.x, gridDim.x, a.num_key_tiles, pair, kt);
  else dkdv_item_heaviest_first(blockIdx.x, gridDim.x / a.num_key_tiles, pair, kt);
  const int heads = a.pv.kv_heads;
  const int g = pair % heads;
  const int b = pair / heads;

  const auto sp = span_view<kRuns>(a, b, a.w_eff);
  const int rows = min(sp.rows(), a.q_len);
  const int clen = min(min(sp.clen(), a.pv.max_pages << a.pv.page_shift), a.hat_cap);
  const int kb0 = kt * kBlockKeys;
  if (kb0 >= clen || rows == 0) return;  // block-uniform

  const int tid = threadIdx.x, lane = tid & 63, bwave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave = bwave % kWaves, sg = bwave / kWaves;  // place in the step group, step group
  const int gq = lane >> 4, j = lane & 15;  // lane group, column of the 16x16 C layout
  const int hq = a.num_q_heads;
  const int group = hq / heads;
  const int gshift = __builtin_ctz(group);  // (a power of two)
  const int kw = kb0 + 16 * wave;   // this wave's first key
  const int key = kw + j;           // this lane's key
  const int tau = key < clen ? sp.visible_from(key, a.mask_mode) : INT_MAX;
  // first row that sees a key of this wave, and from which row on every
  // valid key of the wave is visible
  const int wave_from = kw < clen ? sp.visible_from(kw, a.mask_mode) : INT_MAX;
  const int wave_all = kw < clen ? sp.visible_from(min(kw + 15, clen - 1), a.mask_mode) : INT_MAX;

  // steps: (query head, 32-row tile) pairs from the first tile a key of the
  // block is visible in
  const int q_first = sp.visible_from(kb0, a.mask_mode);
  const int t0 = q_first / kQ, t1 = (rows + kQ - 1) / kQ;
  const int all_steps = max(t1 - t0, 0) << gshift;
  // the group's steps sg, sg + SG, ...; every group takes part in the barriers
  // of the longest (group 0)
  const int n_steps = (all_steps - sg + SG - 1) / SG;
  const int max_steps = (all_steps + SG - 1) / SG;

  // Step n's Q and dO rows (rows past the end read the last row: finite, and
  // masked), 16-byte chunks swizzled per row (QTile), plus LSE (lanes 0-31)
  // and Delta (32-63) of its rows by the last wave.  The row base is uniform.
  const int lrow = lane / Q::kChunks, lpos = lane % Q::kChunks;
  const int rlast = rows - 1;
  auto load_step = [&](int n, Buf& bf) __attribute__((always_inline)) {
    const int m = n * SG + sg;
    const int h = g * group + (m & (group - 1));
    const int q0 = (t1 - 1 - (m >> gshift)) * kQ;
    const int rbase = min(q0, rlast);
    const uint64_t row_bytes = (uint64_t)hq * D * sizeof(T);
    const uint64_t base_off = (((uint64_t)b * a.q_len + rbase) * hq + h) * D * sizeof(T);
    const char* qb = static_cast<const char*>(a.q) + base_off;
    const char* gb = static_cast<const char*>(a.dout) + base_off;
#pragma unroll
    for (int i = 0; i < kLoadsPerWave; ++i) {
      const int l = wave * kLoadsPerWave + i;           // 0 .. 2 kLoads - 1: Q loads, then dO loads
      const bool is_g = l >= Q::kLoads;                 // uniform
      const int lq = is_g ? l - Q::kLoads : l;
      const int r = lq * Q::kRowsPerLoad + lrow;        // row within the tile
      const uint32_t off = (uint32_t)((uint64_t)(min(q0 + r, rlast) - rbase) * row_bytes) +
                           ((lpos ^ Q::swz(r)) << 4);
      lds_dma16(is_g ? gb : qb, off, lds_addr((is_g ? bf.g : bf.q) + lq * Q::kRowsPerLoad * D));
    }
    if (wave == kWaves - 1) {
      const float* src = lane < 32 ? a.lse : a.delta;
      const int64_t stat = ((int64_t)b * hq + h) * a.q_len + min(q0 + (lane & 31), rlast);
      lds_dma4(src + stat, lds_addr(bf.l));
    }
  };

  // K and V operands of this lane's key: elements 32c + 8 gq .. +7 (B operand
  // layout of S = Q K^T and dP = dO V^T); a key past the cache or without a
  // page reads a row of page 0 (its column of every product is never stored)
  Frag kf[kDC], vf[kDC];
  auto load_kv = [&]() __attribute__((always_inline)) {
    const int shift = a.pv.page_shift;
    const int32_t e = a.table[(int64_t)b * a.pv.max_pages + min(key >> shift, a.pv.max_pages - 1)];
    const bool ok = key < clen && e >= 0 && e < a.pv.num_pages;
    const int64_t off = page_row<D>(ok ? e : 0, g, key & ((1 << shift) - 1), a.pv) + 8 * gq;
    const T* kp = static_cast<const T*>(a.k_pages) + off;
    const T* vp = static_cast<const T*>(a.v_pages) + off;
#pragma unroll
    for (int c = 0; c < kDC; ++c) {
      kf[c] = Mfma<T>::load(kp + 32 * c);
      vf[c] = Mfma<T>::load(vp + 32 * c);
    }
  };
  // prologue: the first kBufs - 1 steps and the K and V operands, in flight
  // together and waited for together (the K/V loads are the compiler's: it may
  // move or spill their registers).  The operands first, but for d = 64 with
  // more than a block a CU (us of the attention backward, operands behind /
  // before the steps: d = 128, 92 x 47, b = 64 39.7 / 38.9, 407 x 126, b = 64,
  // 32/8 heads 331 / 313; d = 64, 92 x 47, b = 1 13.8 / 13.6 and b = 16 15.4 /
  // 15.0, but 92 x 62, b = 64 26.5 / 26.7, 782 x 220, b = 32 97 / 99).
  const int my_vm = kVm + (wave == kWaves - 1 ? 1 : 0);
  const bool kv_first = D == 128 || gridDim.x <= kCus;
  if (kv_first) load_kv();
  if (n_steps > 0) load_step(0, s_buf[sg][0]);
  if (kBufs > 2 && n_steps > 1) load_step(1, s_buf[sg][1]);
  if (!kv_first) load_kv();
  bare_barrier<0>();

  typedef float f32x4 __attribute__((ext_vector_type(4)));
  f32x4 dk[kDB], dv[kDB];
#pragma unroll
  for (int db = 0; db < kDB; ++db)
#pragma unroll
    for (int i = 0; i < 4; ++i) dk[db][i] = dv[db][i] = 0.f;

  // Fragment addresses (bytes) in the Q tile of the group's first buffer, one
  // register per pattern; the other buffers, and the dO tiles, are a multiple of
  // 256 bytes further, in the reads' immediate offsets (that leaves the bits
  // of the XORs alone).  With a register per pattern, tile and buffer the third
  // buffer's spilled, and reloading them waited for the direct loads in flight.
  //  - row-wise A operand of S / dP: lane (gq, j) reads row 16blk + j, chunk
  //    (4c + gq) ^ swz(row) = 4c ^ x with x = gq ^ swz(j) (swz(16blk + j) =
  //    swz(j)): address ar0 ^ 64c, plus 16 rows for blk = 1;
  //  - transposed A operand of dV^T / dK^T (ds_read_b64_tr_b16): lane j of
  //    group gq points at row 4gq + j/4 (and 16 + 4gq + j/4), elements 16db +
  //    4(j%4) .. +3, i.e. chunk 2db + e (e = (j%4)/2) at position 2db ^ (e ^
  //    swz(row)), swz(row) the same for both rows: address at0 ^ 32db.
  const int rr = 4 * gq + (j >> 2);
  const uint32_t tile0 = lds_addr(s_buf[sg][0].q);
  const uint32_t ar0 = tile0 + (uint32_t)(j * D * 2 + ((gq ^ Q::swz(j)) << 4));
  const uint32_t at0 = tile0 + (uint32_t)(rr * D * 2 + ((((j & 3) >> 1) ^ Q::swz(rr)) << 4) + ((j & 1) << 3));
  const float neg_inv_scale = -1.f / a.scale;
  typedef __attribute__((address_space(3))) const u16x8_t* lds_frag_ptr;

  // step n from buffer par; the loads of the next kBufs - 1 steps may be in flight
  auto compute = [&](int n, auto par) __attribute__((always_inline)) {
    const Buf& bf = s_buf[sg][decltype(par)::value];
    constexpr uint32_t kTileQ = decltype(par)::value * sizeof(Buf), kTileG = kTileQ + Q::kElems * sizeof(T);
    static_assert(sizeof(Buf) % 256 == 0 && Q::kElems * sizeof(T) % 256 == 0, "tiles on 256-byte boundaries");
    const int q0 = (t1 - 1 - ((n * SG + sg) >> gshift)) * kQ;
    if (q0 + kQ <= wave_from) return;  // no row of the tile sees a key of this wave
    uint32_t ar = ar0, at = at0;
    asm volatile("" : "+v"(ar), "+v"(at));  // (keeps the XORed addresses from being held across steps)
    auto arow = [&](uint32_t tile, int blk, int c) __attribute__((always_inline)) {
      return __builtin_bit_cast(Frag, *(lds_frag_ptr)(uintptr_t)((ar ^ (uint32_t)(64 * c)) + (tile + (uint32_t)(blk * 16 * D * 2))));
    };
    auto atr = [&](uint32_t tile, int db) __attribute__((always_inline)) {
      const uint32_t al = (at ^ (uint32_t)(32 * db)) + tile;
      const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)al);
      const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(uintptr_t)(al + 16 * D * 2));
      const u16x8_t v = {(unsigned short)lo[0], (unsigned short)lo[1], (unsigned short)lo[2], (unsigned short)lo[3],
                         (unsigned short)hi[0], (unsigned short)hi[1], (unsigned short)hi[2], (unsigned short)hi[3]};
      return __builtin_bit_cast(Frag, v);
    };
    // S and dP accumulators start from -LSE/scale and -Delta of their rows
    f32x4 s[2], dp[2];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
      const float4 lv = *reinterpret_cast<const float4*>(bf.l + 16 * blk + 4 * gq);
      const float4 dl = *reinterpret_cast<const float4*>(bf.l + kQ + 16 * blk + 4 * gq);
      s[blk][0] = lv.x * neg_inv_scale; s[blk][1] = lv.y * neg_inv_scale;
      s[blk][2] = lv.z * neg_inv_scale; s[blk][3] = lv.w * neg_inv_scale;
      dp[blk][0] = -dl.x; dp[blk][1] = -dl.y; dp[blk][2] = -dl.z; dp[blk][3] = -dl.w;
    }
    __builtin_amdgcn_sched_barrier(0);  // (these reads first)
    // S / dP: 4 kDC MFMAs over 2 kDC row-wise operands of each tile, read
    // kAheadS ahead of the chain
    constexpr int kNS = 4 * kDC;  // (c, blk, S or dP)
    auto aop = [&](int idx) __attribute__((always_inline)) {
      const int c = idx / 4, blk = (idx / 2) % 2, t = idx % 2;
      return arow(t ? kTileG : kTileQ, blk, c);
    };
    constexpr int kAheadS = 4;
    Frag sb[kAheadS];
#pragma unroll
    for (int i = 0; i < kAheadS; ++i) sb[i] = aop(i);
#pragma unroll
    for (int idx = 0; idx < kNS; ++idx) {
      const Frag cur = sb[idx % kAheadS];
      if (idx + kAheadS < kNS) sb[idx % kAheadS] = aop(idx + kAheadS);
      const int c = idx / 4, blk = (idx / 2) % 2;
      if (idx % 2 == 0) s[blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur, kf[c], s[blk], 0, 0, 0);
      else dp[blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur, vf[c], dp[blk], 0, 0, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x100, kAheadS, 0);  // DS reads
#pragma unroll
    for (int idx = 0; idx + kAheadS < kNS; ++idx) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // MFMA
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, kAheadS, 0);

    // the first transposed operands of dV / dK, read during the softmax
    constexpr int kNT = 2 * kDB;  // (db, dV or dK)
    auto top = [&](int idx) __attribute__((always_inline)) { return atr(idx % 2 ? kTileQ : kTileG, idx / 2); };
    constexpr int kAheadT = 4;
    Frag tb[kAheadT];
#pragma unroll
    for (int i = 0; i < kAheadT; ++i) tb[i] = top(i);
    __builtin_amdgcn_sched_barrier(0);

    // P and dZ in the B-operand order of the dV / dK products: element t of
    // a lane is row 4gq + t (t < 4) or 16 + 4gq + t - 4
    Frag pf, zf;
    float pv[8];
#pragma unroll
    for (int blk = 0; blk < 2; ++blk)
#pragma unroll
      for (int i = 0; i < 4; ++i) pv[4 * blk + i] = fast_exp2(s[blk][i] * a.scale_log2);
    if (q0 < wave_all || q0 + kQ > rows) {  // uniform: some row or key masked
      // row 16 blk + 4 gq + i of the tile is visible to this lane's key iff
      // it lies in [tau, rows): 16 blk + i in [lo, hi)
      const int lo = tau - q0 - 4 * gq, hi = rows - q0 - 4 * gq;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int r = 16 * (t / 4) + t % 4;
        pv[t] = r >= lo && r < hi ? pv[t] : 0.f;
      }
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      pf[t] = (__bf16)pv[t];
      zf[t] = (__bf16)(pv[t] * dp[t / 4][t % 4]);
    }
#pragma unroll
    for (int idx = 0; idx < kNT; ++idx) {
      const Frag cur = tb[idx % kAheadT];
      if (idx + kAheadT < kNT) tb[idx % kAheadT] = top(idx + kAheadT);
      const int db = idx / 2;
      if (idx % 2 == 0) dv[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur, pf, dv[db], 0, 0, 0);
      else dk[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cur, zf, dk[db], 0, 0, 0);
    }
#pragma unroll
    for (int idx = 0; idx + kAheadT < kNT; ++idx) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 1);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 1);  // (two transposed reads)
    }
    __builtin_amdgcn_sched_group_barrier(0x008, kAheadT, 1);
  };

  auto barrier_after = [&](int n) __attribute__((always_inline)) {
    // step n+1's loads landed once only step n+2's are in flight (with two
    // buffers, none)
    if (kBufs > 2 && n + 2 < n_steps) {
      if (my_vm == kVm) bare_barrier<kVm>();
      else bare_barrier<kVm + 1>();
    } else {
      bare_barrier<0>();
    }
  };
  auto step = [&](int n, auto par) __attribute__((always_inline)) {
    constexpr int kPar = decltype(par)::value;
    // (into the buffer step n-1 used)
    if (n + kBufs - 1 < n_steps) load_step(n + kBufs - 1, s_buf[sg][(kPar + kBufs - 1) % kBufs]);
    if (SG == 1 || n < n_steps) compute(n, par);
    barrier_after(n);
  };
  for (int n = 0; n < max_steps; n += kBufs) {
    step(n, std::integral_constant<int, 0>());
    if (n + 1 >= max_steps) break;
    step(n + 1, std::integral_constant<int, 1>());
    if constexpr (kBufs > 2) {
      if (n + 2 >= max_steps) break;
      step(n + 2, std::integral_constant<int, 2>());
    }
  }

  // The step groups' sums through the idle tile buffers, in a fixed order:
  // group 0 finishes dK (adding the others' to its own), group 1 dV.
  if constexpr (SG > 1) {
    constexpr int kPlane = kWaves * 64;  // f32x4 per 16-row block of d
    static_assert(2 * (SG - 1) * kDB * kPlane * 16 <= (int)sizeof(s_buf), "the sums fit the buffers");
    f32x4* const parts = reinterpret_cast<f32x4*>(&s_buf[0][0]);
    const int at = wave * 64 + lane;
    if (sg != 0) {
#pragma unroll
      for (int db = 0; db < kDB; ++db) parts[((sg - 1) * kDB + db) * kPlane + at] = dk[db];
    }
    if (sg != 1) {
      const int slot = SG - 1 + (sg == 0 ? 0 : sg - 1);
#pragma unroll
      for (int db = 0; db < kDB; ++db) parts[(slot * kDB + db) * kPlane + at] = dv[db];
    }
    __syncthreads();
    if (sg > 1) return;
#pragma unroll
    for (int o = 0; o < SG - 1; ++o)
#pragma unroll
      for (int db = 0; db < kDB; ++db) {
        if (sg == 0) dk[db] += parts[(o * kDB + db) * kPlane + at];
        else dv[db] += parts[((SG - 1 + o) * kDB + db) * kPlane + at];
      }
  }

  // lane (gq, j) holds d = 16db + 4gq + i (i < 4) of its key
  if (key >= clen) return;
  float* dkrow = a.dk_hat + (((int64_t)b * a.hat_cap + key) * heads + g) * D + 4 * gq;
  float* dvrow = a.dv_hat + (((int64_t)b * a.hat_cap + key) * heads + g) * D + 4 * gq;
  const float sc = a.scale;
#pragma unroll
  for (int db = 0; db < kDB; ++db) {
    if (SG == 1 || sg == 0)
      *reinterpret_cast<float4*>(dkrow + 16 * db) = make_float4(dk[db][0] * sc, dk[db][1] * sc, dk[db][2] * sc, dk[db][3] * sc);
    if (SG == 1 || sg == 1)
      *reinterpret_cast<float4*>(dvrow + 16 * db) = make_float4(dv[db][0], dv[db][1], dv[db][2], dv[db][3]);
  }
}

template <typename T, int D, bool kRuns>
hipError_t launch_dkdv(const PrefillBwdArgs& a, int batch, hipStream_t s) {
  auto run = [&](auto kernel, int keys, int threads) {
    PrefillBwdArgs c = a;
    c.num_key_tiles = (a.max_keys + keys - 1) / keys;
    return launch_struct(kernel, dim3((unsigned)(batch * a.pv.kv_heads * c.num_key_tiles)), dim3(threads), s, c);
  };
  if constexpr (sizeof(T) == 4) {
    return run(prefill_bwd_dkdv_f32_kernel<D, kRuns>, KvBwdShapeF32<D>::kKeys, KvBwdShapeF32<D>::kThreads);
  } else {
    // The longest chain of steps, and the blocks, of a 64-key split.  Up to
    // three blocks a CU all blocks of one step group are resident from the
    // start and the longest chain sets the time, so the steps are dealt out to
    // more groups: up to a block a CU to eight (d = 64) or four groups of two
    // waves and 32 keys (us, one group of four waves / three / groups of two: 112
    // blocks of <= 196 steps 160 / 102 / 71, 160 of 24 27 / 22 / 17, 160 of 92 at d
    // = 64 61 / 37 / 23, 256 of 100 89 / 61 / 55, 256 of 18 22 / 21 / 25, 44 of 6
    // 10.8 / 12.6 / 10.0), up to three to three groups of four waves and 64 keys
    // (392 of 98 112 / 82 / 97, 512 of 100 106 / 90 / 109, 640 of 102 124 / 110 /
    // 134).  The larger blocks pay their prologue and sums in the open, so more
    // blocks, or short chains, keep one group (1024 of 100 195 / 175, where three
    // would still pay, 2048 of 100 306 / 365, 448 of 24 31 / 36, 512 of 18 28 / 37).
    // Both counts come from the caller's bounds: max_keys is the smaller of
    // max_total_len and hat_capacity, so gradients allocated for more keys than
    // the cache holds take the shape of that many (1596 x 471, b = 8, at a
    // capacity of 1596: the backward 185 us, at 471 134).
    const int64_t chain = (int64_t)(a.num_q_heads / a.pv.kv_heads) * ((a.q_rows + 31) / 32);
    const int64_t blocks = (int64_t)batch * a.pv.kv_heads * ((a.max_keys + 63) / 64);
    if (blocks <= kCus && chain > 12)
      return run(prefill_bwd_dkdv16_kernel<D, kRuns, 2, D == 64 ? 8 : 4, 2>, 32, D == 64 ? 1024 : 512);
    if (blocks <= 3 * kCus && chain > 50)
      return run(prefill_bwd_dkdv16_kernel<D, kRuns, 4, 3, 3>, 64, 768);
    return run(prefill_bwd_dkdv16_kernel<D, kRuns, 4, 1, 3>, 64, 256);
  }
}

template <int D, bool kRuns>
hipError_t launch_dq16(const PrefillBwdArgs& a, int group, int batch, hipStream_t s) {
  const dim3 grid((unsigned)(batch * a.pv.kv_heads * a.num_q_tiles));
  switch (group) {
    case 1: return launch_struct(prefill_bwd_dq16_kernel<D, 1, kRuns>, grid, dim3(DqShape16<1>::kThreads), s, a);
    case 2: return launch_struct(prefill_bwd_dq16_kernel<D, 2, kRuns>, grid, dim3(DqShape16<2>::kThreads), s, a);
    case 4: return launch_struct(prefill_bwd_dq16_kernel<D, 4, kRuns>, grid, dim3(DqShape16<4>::kThreads), s, a);
    default: return launch_struct(prefill_bwd_dq16_kernel<D, 8, kRuns>, grid, dim3(DqShape16<8>::kThreads), s, a);
  }
}

template <typename T, int D>
hipError_t launch_bwd_d(const PrefillBwdArgs& a, int group, int batch, hipStream_t s) {
  const bool runs = a.segs.seg_start != nullptr;
  hipError_t e;
  if constexpr (sizeof(T) == 4) e = launch_prefill_bwd_dq_f32(a, D, group, batch, s);
  else e = runs ? launch_dq16<D, true>(a, group, batch, s) : launch_dq16<D, false>(a, group, batch, s);
  if (e != hipSuccess) return e;
  return runs ? launch_dkdv<T, D, true>(a, batch, s) : launch_dkdv<T, D, false>(a, batch, s);
}

}  // namespace

int prefill_bwd_rows_per_tile(int dtype, int group) {
  if (dtype == 0) return kF32Rows;
  switch (group) {
    case 1: return DqShape16<1>::kRows;
    case 2: return DqShape16<2>::kRows;
    case 4: return DqShape16<4>::kRows;
    default: return DqShape16<8>::kRows;
  }
}

hipError_t launch_prefill_bwd(const PrefillBwdArgs& a, int dtype, int head_dim, int group,
                              int batch, hipStream_t s) {
  if (dtype == 1) {
    if (head_dim == 128) return launch_bwd_d<bf16_bits, 128>(a, group, batch, s);
    return launch_bwd_d<bf16_bits, 64>(a, group, batch, s);
  }
  if (head_dim == 128) return launch_bwd_d<float, 128>(a, group, batch, s);
  return launch_bwd_d<float, 64>(a, group, batch, s);
}

}  // namespace skv

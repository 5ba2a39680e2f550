// fp32 attention over the compressed cache and its dQ (arXiv 2607.06827, Sec.
// III-B, Eq. 5 under the causal mask over compressed positions; formulas and
// mask as in prefill_attn.hip and prefill_bwd.hip).
//
// A block owns 16 query rows of one query head; its kWaves waves deal the
// 16-key tiles that the rows see round, each wave with a K/V tile buffer of its
// own filled by untracked direct loads, so no wave waits for another until the
// waves' partial results are merged through LDS in a fixed order.  Per tile a
// wave computes on the 16x16x4 fp32 MFMA, keys as rows,
//   S^T = K Q^T                               (keys x queries)
//   O^T += V^T P^T                            (16-row blocks of d)
// and for dQ also dP^T = V dO^T, dQ^T += K^T dZ0^T, Kbar^T += K^T P^T.  The k
// index of a product is free as long as both operands agree on it: lane group
// g takes elements 16c + 4g + t of a row for MFMA t (16-byte reads), and the C
// layout (keys 4g + i, query column j) makes P and dZ0 their own B operands.
//
// Bound by the fp32 MFMA where the batch fills the chip and by the chain of
// tiles of a wave where it does not; the latency of a tile's loads is hidden by
// the other waves (two or more a SIMD), not by a second buffer, which would
// halve them.  dQ at 632 x 182, b = 4, 8/4 heads of 64: 41 -> 27 us; at 1532 x
// 407, b = 16, 16/8 heads of 128: 1322 -> 1077 us, against 32-row waves that
// shared register-staged tiles; the forward: see launch_prefill.
#include "attn_mfma.hpp"
#include "kernels.hpp"
#include "kernels_bwd.hpp"

namespace skv {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 4;
constexpr int kRows = kF32Rows;  // query rows of a block
constexpr int kKeys = 16;  // keys per tile
// running maxima may lag by up to 2^kSlack before the accumulators are rescaled
constexpr float kSlack = 8.f;

// A wave's K and V tiles: 16 unpadded rows, 16-byte chunk c of row r at c ^ r
// (16 rows at one chunk, and 4 rows 4g + t at 16 columns, hit 64 distinct banks).
template <int D>
struct KvTile {
  float k[kKeys * D];
  float v[kKeys * D];
};

// One 16-byte operand of row r of a tile: elements 4c .. 4c+3.
template <int D>
__device__ __forceinline__ f32x4 row_read(const float* t, int r, int c) {
  return *reinterpret_cast<const f32x4*>(t + r * D + ((c ^ r) << 2));
}
// Element e of row r.
template <int D>
__device__ __forceinline__ float elem(const float* t, int r, int e) {
  return t[r * D + (((e >> 2) ^ r) << 2) + (e & 3)];
}

// Where a block's work lies; false when its rows are past the sequence.
struct Place {
  int b, g, h, q, row0, rows, kmax, nvis, nvis_lo;
  bool qvalid;
};

template <bool kRuns, typename A>
__device__ __forceinline__ bool place(const A& a, int tiles, int j, Place& w) {
  const int heads = a.pv.kv_heads;
  const int group = a.num_q_heads / heads;
  const int gshift = __builtin_ctz(group);  // (a power of two)
  int pair, item;
  query_tile_item(blockIdx.x, gridDim.x, tiles << gshift, pair, item);  // heaviest rows first
  w.g = pair % heads;
  w.b = pair / heads;
  w.h = w.g * group + (item & (group - 1));
  w.row0 = (item >> gshift) * kRows;
  const auto sp = span_view<kRuns>(a, w.b, a.w_eff);
  w.rows = min(sp.rows(), a.q_len);
  if (w.row0 >= w.rows) return false;
  const int clen = min(sp.clen(), a.pv.max_pages << a.pv.page_shift);
  w.q = w.row0 + j;
  w.qvalid = w.q < w.rows;
  w.kmax = min(sp.visible(min(w.row0 + kRows, w.rows) - 1, a.mask_mode), clen);
  w.nvis = w.qvalid ? min(sp.visible(w.q, a.mask_mode), clen) : 0;
  w.nvis_lo = min(sp.visible(w.row0, a.mask_mode), clen);  // keys every row of the block sees
  return true;
}

// Tile kt of (sequence, KV head) into the wave's buffer: two halves of eight
// keys, each in one page (pages hold at least eight; a key past kmax loads
// the last visible one), rows of a bad table entry zero.
template <int D, typename A>
__device__ __forceinline__ void load_tile(const A& a, const Place& w, int kt, KvTile<D>& buf, int lane) {
  constexpr int kChunks = D / 4;              // 16-byte chunks per row
  constexpr int kRowsPerLoad = 64 / kChunks;  // rows one wave-wide direct load fills
  constexpr int kLoads = 8 / kRowsPerLoad;    // direct loads per half and matrix
  const int shift = a.pv.page_shift, slot_mask = (1 << shift) - 1;
  typedef __attribute__((address_space(4))) const int32_t* const_ptr;
  const const_ptr table = (const_ptr)(a.table + (int64_t)w.b * a.pv.max_pages);
  const uint64_t head_bytes = (uint64_t)D * sizeof(float) << shift;
  const int kclamp = w.kmax - 1;
  const int lrow = lane / kChunks, lpos = lane % kChunks;
  int e[2];
#pragma unroll
  for (int half = 0; half < 2; ++half)
    e[half] = table[min(min(kt * kKeys + 8 * half, kclamp) >> shift, a.pv.max_pages - 1)];
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const uint64_t at = ((uint64_t)(uint32_t)e[half] * a.pv.kv_heads + w.g) * head_bytes;
    const bool ok = e[half] >= 0 && e[half] < a.pv.num_pages;  // uniform
#pragma unroll
    for (int l = 0; l < kLoads; ++l) {
      const int r0 = 8 * half + l * kRowsPerLoad, r = r0 + lrow;
      const int key = min(kt * kKeys + r, kclamp);
      const uint32_t off = (uint32_t)((key & slot_mask) * D * 4) + ((lpos ^ r) << 4);
      if (ok) {
        lds_dma16(static_cast<const char*>(a.k_pages) + at, off, lds_addr(buf.k + r0 * D));
        lds_dma16(static_cast<const char*>(a.v_pages) + at, off, lds_addr(buf.v + r0 * D));
      } else {
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        *reinterpret_cast<f32x4*>(buf.k + r0 * D + 4 * lane) = zero;
        *reinterpret_cast<f32x4*>(buf.v + r0 * D + 4 * lane) = zero;
      }
    }
  }
}

// Every load of the wave has landed and its LDS accesses are done.
__device__ __forceinline__ void wait_all() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(wait_vm_lgkm0(0));
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

template <int D>
constexpr int waves_per_simd() {
  return D == 128 ? 2 : 4;  // the tiles of eight (16) waves a CU fit its 160 KB
}

// ------------------------------------------------------------------ forward

template <int D, bool kRuns>
__global__ __launch_bounds__(64 * kWaves, waves_per_simd<D>()) void prefill_f32_kernel(PrefillArgs a) {
  constexpr int kDB = D / 16;
  constexpr float kLn2 = 0.6931471805599453f;
  __shared__ __attribute__((aligned(256))) KvTile<D> s_tile[kWaves];
  __shared__ float s_m[kWaves][kRows], s_l[kWaves][kRows];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int gq = lane >> 4, j = lane & 15;  // lane group, column of the 16x16 C layout
  Place w;
  if (!place<kRuns>(a, a.num_tiles, j, w)) return;
  const int hq = a.num_q_heads;
  const int ntiles = (w.kmax + kKeys - 1) / kKeys;

  // this lane's query row, elements 16c + 4gq .. +3 (rows past the end read
  // row 0 of the sequence: never stored)
  f32x4 qf[kDB];
  const float* qrow = static_cast<const float*>(a.q) + (((int64_t)w.b * a.q_len + (w.qvalid ? w.q : 0)) * hq + w.h) * D + 4 * gq;
#pragma unroll
  for (int c = 0; c < kDB; ++c) qf[c] = *reinterpret_cast<const f32x4*>(qrow + 16 * c);

  f32x4 o[kDB];
#pragma unroll
  for (int db = 0; db < kDB; ++db)
#pragma unroll
    for (int i = 0; i < 4; ++i) o[db][i] = 0.f;
  float m_run = neg_inf(), l_run = 0.f;  // of row q; l_run this lane's share

  KvTile<D>& t = s_tile[wave];
  for (int kt = wave; kt < ntiles; kt += kWaves) {
    wait_all();  // the last tile's reads
    load_tile<D>(a, w, kt, t, lane);
    wait_all();
    // values of keys past the visible range (copies of the last one's) are
    // zero: an infinite one would meet its zero weight as 0 * infinity
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    if (kt == ntiles - 1) {
      for (int i = (w.kmax - kt * kKeys) * (D / 4) + lane; i < kKeys * (D / 4); i += 64)
        *reinterpret_cast<f32x4*>(t.v + 4 * i) = zero;
    }
    f32x4 s = zero;
#pragma unroll
    for (int c = 0; c < kDB; ++c) {
      const f32x4 ka = row_read<D>(t.k, j, 4 * c + gq);
#pragma unroll
      for (int i = 0; i < 4; ++i) s = __builtin_amdgcn_mfma_f32_16x16x4f32(ka[i], qf[c][i], s, 0, 0, 0);
    }
    const int kb = kt * kKeys;
    if (kb + kKeys > w.nvis_lo) {  // uniform: the tile straddles some row's bound
#pragma unroll
      for (int i = 0; i < 4; ++i) s[i] = kb + 4 * gq + i < w.nvis ? s[i] : neg_inf();
    }
    float mt = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
    mt = fmaxf(mt, xor_shuffle(mt, 16));
    mt = fmaxf(mt, xor_shuffle(mt, 32)) * a.scale_log2;  // the scale is > 0
    const bool grown = mt > m_run + kSlack;
    if (__any(grown)) {  // uniform: a factor of 1 for the rows that stay
      const float m_new = grown ? mt : m_run;
      const float corr = grown ? fast_exp2(m_run - m_new) : 1.f;
      l_run *= corr;
#pragma unroll
      for (int db = 0; db < kDB; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i) o[db][i] *= corr;
      m_run = m_new;
    }
    const float m_use = m_run == neg_inf() ? 0.f : m_run;  // nothing visible yet: weights exp2(-inf) = 0
    float p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      p[i] = fast_exp2(__builtin_fmaf(s[i], a.scale_log2, -m_use));
      l_run += p[i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int db = 0; db < kDB; ++db)
        o[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(elem<D>(t.v, 4 * gq + i, 16 * db + j), p[i], o[db], 0, 0, 0);
  }

  // merge the waves: row maxima and sums, then the planes (16-row blocks of d,
  // 64 lanes x 4 values) in the waves' own tile buffers, each plane by one wave
  l_run += xor_shuffle(l_run, 16);
  l_run += xor_shuffle(l_run, 32);
  wait_all();
  f32x4* const mine = reinterpret_cast<f32x4*>(&s_tile[wave]);
#pragma unroll
  for (int db = 0; db < kDB; ++db) mine[db * 64 + lane] = o[db];
  if (gq == 0) {
    s_m[wave][j] = m_run;
    s_l[wave][j] = l_run;
  }
  __syncthreads();
  float m = s_m[0][j];
#pragma unroll
  for (int v = 1; v < kWaves; ++v) m = fmaxf(m, s_m[v][j]);
  const float m_use = m == neg_inf() ? 0.f : m;
  float f[kWaves], l = 0.f;
#pragma unroll
  for (int v = 0; v < kWaves; ++v) {
    f[v] = fast_exp2(s_m[v][j] - m_use);
    l = __builtin_fmaf(f[v], s_l[v][j], l);
  }
  if (!w.qvalid) return;
  const float inv = l > 0.f ? 1.f / l : 0.f;
  if (wave == 0 && gq == 0 && a.lse)
    a.lse[((int64_t)w.b * hq + w.h) * a.q_len + w.q] = l > 0.f ? (m + __log2f(l)) * kLn2 : neg_inf();
  float* const orow = static_cast<float*>(a.out) + (((int64_t)w.b * a.q_len + w.q) * hq + w.h) * D + 4 * gq;
#pragma unroll
  for (int n = 0; n < kDB / kWaves; ++n) {
    const int db = wave + n * kWaves;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int v = 0; v < kWaves; ++v) {
      const f32x4 x = reinterpret_cast<const f32x4*>(&s_tile[v])[db * 64 + lane];
#pragma unroll
      for (int i = 0; i < 4; ++i) sum[i] = __builtin_fmaf(f[v], x[i], sum[i]);
    }
    *reinterpret_cast<float4*>(orow + 16 * db) = make_float4(sum[0] * inv, sum[1] * inv, sum[2] * inv, sum[3] * inv);
  }
}

// ----------------------------------------------------------------------- dQ

template <int D, bool kRuns>
__global__ __launch_bounds__(64 * kWaves, waves_per_simd<D>()) void prefill_bwd_dq_f32_kernel(PrefillBwdArgs a) {
  constexpr int kDB = D / 16;
  constexpr float kLog2e = 1.4426950408889634f;
  __shared__ __attribute__((aligned(256))) KvTile<D> s_tile[kWaves];
  __shared__ float s_d[kWaves][kRows];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int gq = lane >> 4, j = lane & 15;
  Place w;
  if (!place<kRuns>(a, a.num_q_tiles, j, w)) return;
  const int hq = a.num_q_heads;
  const int ntiles = (w.kmax + kKeys - 1) / kKeys;

  // this lane's row of Q and dO, elements 16c + 4gq .. +3, and Delta0 = dO . O
  // from the stored output (rows past the end read row 0: never stored)
  f32x4 qf[kDB], gf[kDB];
  const int64_t off = (((int64_t)w.b * a.q_len + (w.qvalid ? w.q : 0)) * hq + w.h) * D + 4 * gq;
  float delta0 = 0.f;
#pragma unroll
  for (int c = 0; c < kDB; ++c) {
    qf[c] = *reinterpret_cast<const f32x4*>(static_cast<const float*>(a.q) + off + 16 * c);
    gf[c] = *reinterpret_cast<const f32x4*>(static_cast<const float*>(a.dout) + off + 16 * c);
    const f32x4 of = *reinterpret_cast<const f32x4*>(static_cast<const float*>(a.out) + off + 16 * c);
#pragma unroll
    for (int i = 0; i < 4; ++i) delta0 = __builtin_fmaf(gf[c][i], of[i], delta0);
  }
  const int64_t stat = ((int64_t)w.b * hq + w.h) * a.q_len + (w.qvalid ? w.q : 0);
  const float lse2 = a.lse[stat] * kLog2e;
  delta0 += xor_shuffle(delta0, 16);
  delta0 += xor_shuffle(delta0, 32);

  f32x4 dq[kDB], kbar[kDB];
#pragma unroll
  for (int db = 0; db < kDB; ++db)
#pragma unroll
    for (int i = 0; i < 4; ++i) dq[db][i] = kbar[db][i] = 0.f;
  float dsum = 0.f;  // this lane's share of Delta = sum over keys of P dP

  KvTile<D>& t = s_tile[wave];
  for (int kt = wave; kt < ntiles; kt += kWaves) {
    wait_all();
    load_tile<D>(a, w, kt, t, lane);
    wait_all();
    f32x4 s = {0.f, 0.f, 0.f, 0.f}, dp = s;
#pragma unroll
    for (int c = 0; c < kDB; ++c) {
      const f32x4 ka = row_read<D>(t.k, j, 4 * c + gq);
      const f32x4 va = row_read<D>(t.v, j, 4 * c + gq);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s = __builtin_amdgcn_mfma_f32_16x16x4f32(ka[i], qf[c][i], s, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_16x16x4f32(va[i], gf[c][i], dp, 0, 0, 0);
      }
    }
    float p[4], z[4];
    const int lim = w.nvis - kt * kKeys - 4 * gq;  // key i is visible iff i < lim
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float e = fast_exp2(__builtin_fmaf(s[i], a.scale_log2, -lse2));
      p[i] = i < lim ? e : 0.f;
      z[i] = p[i] * (dp[i] - delta0);
      dsum = __builtin_fmaf(p[i], dp[i], dsum);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int db = 0; db < kDB; ++db) {
        const float ke = elem<D>(t.k, 4 * gq + i, 16 * db + j);
        dq[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(ke, z[i], dq[db], 0, 0, 0);
        kbar[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(ke, p[i], kbar[db], 0, 0, 0);
      }
  }

  // merge the waves: Delta, then dQ = scale (dZ0 K + (Delta0 - Delta) Kbar)
  dsum += xor_shuffle(dsum, 16);
  dsum += xor_shuffle(dsum, 32);
  wait_all();
  f32x4* const mine = reinterpret_cast<f32x4*>(&s_tile[wave]);
#pragma unroll
  for (int db = 0; db < kDB; ++db) {
    mine[(2 * db) * 64 + lane] = dq[db];
    mine[(2 * db + 1) * 64 + lane] = kbar[db];
  }
  if (gq == 0) s_d[wave][j] = dsum;
  __syncthreads();
  if (!w.qvalid) return;
  float delta = s_d[0][j];
#pragma unroll
  for (int v = 1; v < kWaves; ++v) delta += s_d[v][j];
  if (wave == 0 && gq == 0) a.delta[stat] = delta;
  const float sc = a.scale, fix = delta0 - delta;
  float* const drow = static_cast<float*>(a.dq) + off;
#pragma unroll
  for (int n = 0; n < kDB / kWaves; ++n) {
    const int db = wave + n * kWaves;
    f32x4 x = reinterpret_cast<const f32x4*>(&s_tile[0])[(2 * db) * 64 + lane];
    f32x4 y = reinterpret_cast<const f32x4*>(&s_tile[0])[(2 * db + 1) * 64 + lane];
#pragma unroll
    for (int v = 1; v < kWaves; ++v) {
      x += reinterpret_cast<const f32x4*>(&s_tile[v])[(2 * db) * 64 + lane];
      y += reinterpret_cast<const f32x4*>(&s_tile[v])[(2 * db + 1) * 64 + lane];
    }
    *reinterpret_cast<float4*>(drow + 16 * db) =
        make_float4(sc * __builtin_fmaf(fix, y[0], x[0]), sc * __builtin_fmaf(fix, y[1], x[1]),
                    sc * __builtin_fmaf(fix, y[2], x[2]), sc * __builtin_fmaf(fix, y[3], x[3]));
  }
}

}  // namespace

hipError_t launch_prefill_f32(const PrefillArgs& a, int head_dim, int group, int batch, hipStream_t s) {
  const dim3 grid((unsigned)(batch * a.pv.kv_heads * a.num_tiles * group)), block(64 * kWaves);
  const bool runs = a.segs.seg_start != nullptr;
  if (head_dim == 128)
    return runs ? launch_struct(prefill_f32_kernel<128, true>, grid, block, s, a)
                : launch_struct(prefill_f32_kernel<128, false>, grid, block, s, a);
  return runs ? launch_struct(prefill_f32_kernel<64, true>, grid, block, s, a)
              : launch_struct(prefill_f32_kernel<64, false>, grid, block, s, a);
}

hipError_t launch_prefill_bwd_dq_f32(const PrefillBwdArgs& a, int head_dim, int group, int batch, hipStream_t s) {
  const dim3 grid((unsigned)(batch * a.pv.kv_heads * a.num_q_tiles * group)), block(64 * kWaves);
  const bool runs = a.segs.seg_start != nullptr;
  if (head_dim == 128)
    return runs ? launch_struct(prefill_bwd_dq_f32_kernel<128, true>, grid, block, s, a)
                : launch_struct(prefill_bwd_dq_f32_kernel<128, false>, grid, block, s, a);
  return runs ? launch_struct(prefill_bwd_dq_f32_kernel<64, true>, grid, block, s, a)
              : launch_struct(prefill_bwd_dq_f32_kernel<64, false>, grid, block, s, a);
}

}  // namespace skv

// Block-sparse softmax attention for gfx950: 64 x 64 score blocks on the
// flat block butterfly mask, head dim 64, bf16 I/O, fp32 softmax/accumulate.
//
// Workgroup = groups of 2 waves; a group owns one 64-row block (of queries
// for the forward and dQ, of keys for dK/dV), each wave 32 rows of it.
// Everything is computed in transposed form so that each lane owns ONE row
// (its softmax statistics are per-lane scalars) and the probability tile
// feeds the next MFMA straight from registers (32x32x16 MFMA):
//   forward : S^T = K_j Q_w^T, online softmax per query, O^T += V_j^T P^T.
//   dQ      : recompute S^T, P^T; dP^T = V_j dO_w^T; dS^T = P^T o (dP^T -
//             delta); dQ^T += K_j^T dS^T.
//   dK, dV  : S = Q_i K_w^T, P, dP = dO_i V_w^T, dS; dV^T += dO_i^T P,
//             dK^T += Q_i^T dS.
// An accumulator of a 32 x 32 tile holds, in lane l, rows 8 (e / 4) + 4
// (l / 32) + e % 4 of column l % 32; its registers 8 j .. 8 j + 7 are used as
// the K-operand of 16 rows in that order, and the matching operand is read
// from LDS with the transpose read in the same order.
//
// The tiles of a kept block go global -> LDS directly.  A wave reads whole
// tiles from LDS whatever its row count, so 32 rows per wave halve the LDS
// bytes per score of the 16-row waves these kernels had before, and the
// swizzled tiles have no bank conflicts.  Counters at 8 x 12 x 4096 x 64,
// 7 blocks per row: forward VALU 53 % (exponentials three tenths of it), MFMA
// 31 %, LDS 15 % of cycles; dQ 43 / 32 / 16 %, dK/dV 39 / 37 / 28 %: the
// serial S -> softmax -> product chain of few waves per SIMD bounds them, so
// forward and dQ keep one stage per operand (16 KiB per workgroup, four
// waves per SIMD; two stages and 2.5 waves: 79 against 66 us, 111 against
// 101 us) and refill each operand as soon as its last read is done; dK/dV,
// whose accumulators leave two waves per SIMD, keeps two stages (one stage
// and three waves: 123 -> 131 us).  16-row waves -> this: forward 85 -> 66,
// dQ 113 -> 101, dK/dV 152 -> 122 us.  Measured and not kept: wave priority
// around the MFMA phases, the softmax of one half of the keys under the MFMAs
// of the other, maxima replaced by a check of the sums (all within 3 %).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "pf_dma.h"
#include "pf_launch.h"

namespace pf {
namespace {

constexpr int D = 64;                    // head dim
constexpr int BQ = 64;                   // block size
constexpr int TILE = BQ * D * 2;         // bytes of a 64 x 64 bf16 tile
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// 2^x on the hardware exponential unit (v_exp_f32): results below 2^-126
// flush toward zero, which a softmax probability can afford; saves the
// range-reduction sequence the library exp2f adds for denormal outputs.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// x combined with the value of lane l ^ 32 by max or +: the swap exchanges
// the halves inside the VALU, where a lane shuffle would make a round trip
// through the LDS.
__device__ __forceinline__ float max_xor32(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float add_xor32(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)lo) |
         ((uint32_t)__builtin_bit_cast(uint16_t, (__bf16)hi) << 16);
}

// LDS tile: 64 rows of 128 bytes, the 16-byte chunk c of row r at position
// c ^ chunk_swz(r).  Row pairs (256 bytes, all 64 banks) get the eight
// values of the bit-reversed pair index: 16 rows at one chunk (fragment
// read) and 4 rows x 4 chunks (transpose read) both fall in distinct banks.
__device__ __forceinline__ int chunk_swz(int r) {
  return ((r & 2) << 1) | ((r & 4) >> 1) | ((r & 8) >> 3);
}

// Copies of one tile by the 2 waves of a group: wave w fills the 1 KiB
// windows (8 rows) 4 w .. 4 w + 3.
struct TileCopy {
  uint32_t voff[2];  // lane part, even / odd windows
  int w4;            // first window of this wave
  __device__ __forceinline__ void init(int lane, int w) {
    const int x = (((lane >> 4) & 1) << 2) | (((lane >> 5) & 1) << 1);
#pragma unroll
    for (int o = 0; o < 2; ++o)
      voff[o] = (uint32_t)((lane >> 3) * 128 + (((lane & 7) ^ x ^ o) << 4));
    w4 = w * 4;
  }
  // live false: the copies read nothing and leave zeros (an empty range), so
  // that the loop has no branch around them and the waits stay counted.
  __device__ __forceinline__ void issue(const bf16_t *g, uint8_t *tile, bool live) const {
    const rsrc_t r = make_rsrc(g, live ? TILE : 0);
    sfor<4>([&](auto i) __attribute__((always_inline)) {
      dma16(r, tile + (w4 + i) * 1024, voff[i & 1], (uint32_t)((w4 + i) * 1024));
    });
  }
};

// Operand of a 32x32x16 MFMA from a tile: row r0 + l % 32, k = ks * 16 +
// (l / 32) * 8 + 0..7.
__device__ __forceinline__ bf16x8 frag_r(const uint8_t *tile, int r0, int ks, int lane) {
  const int r = r0 + (lane & 31), c = ks * 2 + (lane >> 5);
  return *(const bf16x8 *)(tile + r * 128 + ((c ^ chunk_swz(r)) << 4));
}
// Same from global memory (64-column rows).
__device__ __forceinline__ bf16x8 frag_g(const bf16_t *p, int r0, int ks, int lane) {
  return *(const bf16x8 *)(p + (int64_t)(r0 + (lane & 31)) * D + ks * 16 + (lane >> 5) * 8);
}
// Operand A[m][k] = tile[k][m], m = m0 + l % 32, k in the accumulator's row
// order: kb + 4 (l / 32) + 0..3, then kb + 8 + 4 (l / 32) + 0..3.
__device__ __forceinline__ bf16x8 frag_t(const uint8_t *tile, int kb, int m0, int lane) {
  const int g = lane >> 4, i = lane & 15;
  const int c = (m0 >> 3) + (g & 1) * 2 + ((i & 3) >> 1), half = (i & 1) << 3;
  const int k = kb + (g >> 1) * 4 + (i >> 2);
  const int lo_off = k * 128 + ((c ^ chunk_swz(k)) << 4) + half;
  const int hi_off = (k + 8) * 128 + ((c ^ chunk_swz(k + 8)) << 4) + half;
  const s16x4 lo = tr16(tile + lo_off), hi = tr16(tile + hi_off);
  const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8, v);
}
// Registers 8 j .. 8 j + 7 of an accumulator as a bf16 K-operand.
__device__ __forceinline__ bf16x8 pack_k(const f32x16 &s, int j) {
  bf16x8 v;
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (__bf16)s[8 * j + e];
  return v;
}

#define MFMA32(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16((a), (b), (c), 0, 0, 0)

// Row (query or key) l % 32's 64 columns held as two transposed accumulators,
// times `scale`, to 128 contiguous bytes at dst: the halves swap registers
// so that each lane stores 16 bytes at a time.
__device__ __forceinline__ void store_row(bf16_t *dst, const f32x16 (&o)[2], float scale, int lane) {
#pragma unroll
  for (int dt = 0; dt < 2; ++dt)
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int e = 8 * p;
      const uint32_t x0 = pack2(o[dt][e] * scale, o[dt][e + 1] * scale);
      const uint32_t x1 = pack2(o[dt][e + 2] * scale, o[dt][e + 3] * scale);
      const uint32_t y0 = pack2(o[dt][e + 4] * scale, o[dt][e + 5] * scale);
      const uint32_t y1 = pack2(o[dt][e + 6] * scale, o[dt][e + 7] * scale);
      const auto s0 = __builtin_amdgcn_permlane32_swap(x0, y0, false, false);
      const auto s1 = __builtin_amdgcn_permlane32_swap(x1, y1, false, false);
      *(u32x4 *)(dst + dt * 32 + p * 16 + (lane >> 5) * 8) = u32x4{s0[0], s1[0], s0[1], s1[1]};
    }
}

// Merge area of group g, float slot v (0..15) of this wave's lane in stage
// object `obj` (one 8 KiB tile per group: 16 floats x 64 lanes x 2 waves).
__device__ __forceinline__ float *merge_at(uint8_t *obj, int g, int w, int lane) {
  return (float *)(obj + g * TILE) + w * (16 * 64) + lane;
}

// Work order: (head, block) of logical id L.  Block rows (or, for dK/dV,
// block columns) below nlong are the global stripes of the mask, which keep
// every block of the other side: they go first, over all heads, so that the
// long workgroups do not trail the launch; the rest follow head by head.
__device__ __forceinline__ void attn_order(int L, int BH, int nb, int nlong, int &bh, int &blk) {
  if (L < nlong * BH) {
    blk = L / BH;
    bh = L % BH;
  } else {
    const int r = L - nlong * BH, m = nb - nlong;
    bh = r / m;
    blk = nlong + r % m;
  }
}

// ---------------------------------------------------------------------------
// Forward
// ---------------------------------------------------------------------------
// NG groups share one 64-query block: group g takes the row's kept blocks g,
// g + NG, ... (each group has its own double-buffered K/V tiles; all groups
// run the same number of iterations so every barrier is reached by the whole
// workgroup) and the groups' softmax states (reference, sum, unnormalised O)
// are merged through LDS in group order at the end.
template <int NG, int ST>
__global__ __launch_bounds__(128 * NG, ST == 1 ? 4 : 1) void attn_fwd_kernel(AttnArgs a) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & 1);
  const int grp = NG > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 7) : 0;
  uint8_t *const kst = stage_buf<0, NG * TILE>(), *const vst = stage_buf<1, NG * TILE>();
  __shared__ float ml[NG > 1 ? NG : 1][256];  // merge: reference and sum per lane
  uint8_t *const k0s = kst + grp * TILE, *const v0s = vst + grp * TILE;

  const int bid = xcd_remap(blockIdx.x, gridDim.x) + a.first;
  int bh, qb;
  attn_order(bid, a.BH, a.nbq, a.nlong, bh, qb);
  const int64_t head = (int64_t)bh * a.S * D;
  const bf16_t *Q = (const bf16_t *)a.Q + head;
  const bf16_t *K = (const bf16_t *)a.K + head;
  const bf16_t *V = (const bf16_t *)a.V + head;
  const int q0 = qb * BQ + w * 32;
  const float c = a.scale * kLog2e;

  // Rows are never empty; indices past a row's end are clamped into it and
  // their copies switched off.
  const int p0 = ld_meta(a.row_ptr + qb), p1 = ld_meta(a.row_ptr + qb + 1);
  const int iters = (p1 - p0 + NG - 1) / NG;
  TileCopy cp;
  cp.init(lane, w);
  int ccur = ld_meta(a.col_idx + min(p0 + grp, p1 - 1));
  cp.issue(K + (int64_t)ccur * BQ * D, k0s, p0 + grp < p1);
  if constexpr (ST == 2) cp.issue(V + (int64_t)ccur * BQ * D, v0s, p0 + grp < p1);
  bf16x8 qf[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) qf[ks] = frag_g(Q, q0, ks, lane);
  // Block column of this group's next tile, loaded one iteration ahead so
  // that the copies do not wait on it.
  int cn = ld_meta(a.col_idx + min(p0 + grp + NG, p1 - 1));

  float m_run = -INFINITY, l_run = 0.f;  // l_run: this lane's keys only
  f32x16 o[2];
#pragma unroll
  for (int e = 0; e < 16; ++e) o[0][e] = o[1][e] = 0.f;

  f32x16 s[2];
  // S^T[key][query] for 64 keys x this wave's 32 queries.
  auto scores = [&](const uint8_t *kc) __attribute__((always_inline)) {
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
#pragma unroll
      for (int e = 0; e < 16; ++e) s[kt][e] = 0.f;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) s[kt] = MFMA32(frag_r(kc, kt * 32, ks, lane), qf[ks], s[kt]);
    }
  };
  auto softmax = [&]() __attribute__((always_inline)) {
    float bmax = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int e = 0; e < 16; ++e) bmax = fmaxf(bmax, s[kt][e]);
    // The softmax reference m_run (the same in both lanes of a query) moves
    // only when some lane's maximum grew by more than 8 (log2 units): until
    // then the probabilities stay below 2^8 and the rescale of O and l, a
    // wave-uniform branch, is skipped.
    if (__builtin_amdgcn_ballot_w64(fmaxf(m_run, bmax * c) > m_run + 8.0f)) {
      const float m_cand = fmaxf(m_run, max_xor32(bmax) * c);
      const float alpha = fast_exp2(m_run - m_cand);
      m_run = m_cand;
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[dt][e] *= alpha;
    }
    float rs = 0.f;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float x = fast_exp2(s[kt][e] * c - m_run);
        s[kt][e] = x;
        rs += x;
      }
    l_run += rs;
  };
  // O^T[dim][query] += V^T[dim][key] P^T[key][query]
  auto product = [&](const uint8_t *vc) __attribute__((always_inline)) {
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const bf16x8 pb = pack_k(s[kt], j);
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
          o[dt] = MFMA32(frag_t(vc, kt * 32 + j * 16, dt * 32, lane), pb, o[dt]);
      }
  };
  if constexpr (ST == 1) {
    static_assert(NG == 1 || ST == 2, "groups are double-buffered");
    for (int p = p0; p < p1; ++p) {
      wait_vm<0>();  // this wave's K copies have landed,
      barrier();     // every wave's have, and the last block's V is read
      cp.issue(V + (int64_t)ccur * BQ * D, v0s, true);
      scores(k0s);
      wait_vm<4>();  // (no wait: the four V copies may be in flight)
      barrier();     // every wave has read K
      cp.issue(K + (int64_t)cn * BQ * D, k0s, p + 1 < p1);
      ccur = cn;
      cn = ld_meta(a.col_idx + min(p + 2, p1 - 1));
      softmax();
      wait_vm<4>();  // V has landed; the next K copies stay in flight
      barrier();
      product(v0s);
    }
  } else {
    uint8_t *const k1s = stage_buf<2, NG * TILE>() + grp * TILE;
    uint8_t *const v1s = stage_buf<3, NG * TILE>() + grp * TILE;
    auto step = [&](int it, uint8_t *kc, uint8_t *vc, uint8_t *kn, uint8_t *vn)
        __attribute__((always_inline)) {
      const int p = p0 + it * NG + grp;
      wait_vm<0>();  // this wave's copies of the block have landed,
      barrier();     // every wave's have, and nobody reads the other stage
      if (p + NG < p1) {
        cp.issue(K + (int64_t)cn * BQ * D, kn, true);
        cp.issue(V + (int64_t)cn * BQ * D, vn, true);
      }
      cn = ld_meta(a.col_idx + min(p + 2 * NG, p1 - 1));
      if (NG > 1 && p >= p1) return;
      scores(kc);
      softmax();
      product(vc);
    };
    for (int it = 0; it < iters; it += 2) {
      step(it, k0s, v0s, k1s, v1s);
      if (it + 1 < iters) step(it + 1, k1s, v1s, k0s, v0s);
    }
  }
  wait_vm<0>();  // no copy outlives the workgroup

  if constexpr (NG > 1) {
    // Merge: groups 1.. leave (o, m, l) per lane in their tiles, group 0
    // combines them relative to the largest reference.  A group without
    // blocks has m = -inf and contributes 0.
    barrier();
    if (grp > 0) {
      float *m0 = merge_at(kst, grp, w, lane), *m1 = merge_at(vst, grp, w, lane);
      float *m2 = &ml[grp][w * 128 + lane];
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        m0[e * 64] = o[0][e];
        m1[e * 64] = o[1][e];
      }
      m2[0] = m_run;
      m2[64] = l_run;
    }
    __syncthreads();
    if (grp > 0) return;
    float m = m_run;
#pragma unroll
    for (int g = 1; g < NG; ++g) m = fmaxf(m, ml[g][w * 128 + lane]);
    const float s0 = fast_exp2(m_run - m);
    l_run *= s0;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      o[0][e] *= s0;
      o[1][e] *= s0;
    }
#pragma unroll
    for (int g = 1; g < NG; ++g) {
      const float *m0 = merge_at(kst, g, w, lane), *m1 = merge_at(vst, g, w, lane);
      const float *m2 = &ml[g][w * 128 + lane];
      const float sg = m2[0] == -INFINITY ? 0.f : fast_exp2(m2[0] - m);
      l_run += m2[64] * sg;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        o[0][e] += m0[e * 64] * sg;
        o[1][e] += m1[e * 64] * sg;
      }
    }
    m_run = m;
  }

  l_run = add_xor32(l_run);
  const int q = q0 + (lane & 31);
  store_row((bf16_t *)a.Oout + head + (int64_t)q * D, o, 1.f / l_run, lane);
  if (lane < 32) a.lse[(int64_t)bh * a.S + q] = (m_run + __log2f(l_run)) * kLn2;
}

// ---------------------------------------------------------------------------
// Backward, pass 1: delta and dQ (a group per query block)
// ---------------------------------------------------------------------------
// NG groups split the row's kept blocks as in the forward; their dQ partial
// sums are added through LDS in group order.
template <int NG, int ST>
__global__ __launch_bounds__(128 * NG, ST == 1 ? 4 : 1) void attn_bwd_dq_kernel(AttnArgs a) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & 1);
  const int grp = NG > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 7) : 0;
  uint8_t *const kst = stage_buf<0, NG * TILE>(), *const vst = stage_buf<1, NG * TILE>();
  uint8_t *const k0s = kst + grp * TILE, *const v0s = vst + grp * TILE;

  const int bid = xcd_remap(blockIdx.x, gridDim.x) + a.first;
  int bh, qb;
  attn_order(bid, a.BH, a.nbq, a.nlong, bh, qb);
  const int64_t head = (int64_t)bh * a.S * D;
  const bf16_t *Q = (const bf16_t *)a.Q + head;
  const bf16_t *K = (const bf16_t *)a.K + head;
  const bf16_t *V = (const bf16_t *)a.V + head;
  const bf16_t *O = (const bf16_t *)a.O + head;
  const bf16_t *dO = (const bf16_t *)a.dO + head;
  const int q0 = qb * BQ + w * 32;
  const int q = q0 + (lane & 31);
  const float c = a.scale * kLog2e;

  const int p0 = ld_meta(a.row_ptr + qb), p1 = ld_meta(a.row_ptr + qb + 1);
  const int iters = (p1 - p0 + NG - 1) / NG;
  TileCopy cp;
  cp.init(lane, w);
  const int c0 = ld_meta(a.col_idx + min(p0 + grp, p1 - 1));
  cp.issue(V + (int64_t)c0 * BQ * D, v0s, p0 + grp < p1);
  cp.issue(K + (int64_t)c0 * BQ * D, k0s, p0 + grp < p1);
  bf16x8 qf[4], dof[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    qf[ks] = frag_g(Q, q0, ks, lane);
    dof[ks] = frag_g(dO, q0, ks, lane);
  }
  // delta = rowsum(dO o O): the two lanes of a query hold half its columns
  // each in the fragment layout.
  float delta = 0.f;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const bf16x8 of = frag_g(O, q0, ks, lane);
#pragma unroll
    for (int e = 0; e < 8; ++e) delta += (float)of[e] * (float)dof[ks][e];
  }
  delta = add_xor32(delta);
  if (lane < 32 && grp == 0) a.delta[(int64_t)bh * a.S + q] = delta;
  const float lse2 = a.lse_in[(int64_t)bh * a.S + q] * kLog2e;
  // Next block column one iteration ahead, as in the forward.
  int cn = ld_meta(a.col_idx + min(p0 + grp + NG, p1 - 1));

  f32x16 dq[2];
#pragma unroll
  for (int e = 0; e < 16; ++e) dq[0][e] = dq[1][e] = 0.f;

  // S^T and dP^T of 32 keys, dS^T from them, and its product with K.
  f32x16 s, dp;
  auto scores = [&](const uint8_t *kc, const uint8_t *vc, int kt) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] = dp[e] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      s = MFMA32(frag_r(kc, kt * 32, ks, lane), qf[ks], s);
      dp = MFMA32(frag_r(vc, kt * 32, ks, lane), dof[ks], dp);
    }
  };
  auto grads = [&](const uint8_t *kc, int kt) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float pr = fast_exp2(s[e] * c - lse2);
      s[e] = pr * (dp[e] - delta);  // dS^T
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const bf16x8 d = pack_k(s, j);
#pragma unroll
      for (int dt = 0; dt < 2; ++dt)
        dq[dt] = MFMA32(frag_t(kc, kt * 32 + j * 16, dt * 32, lane), d, dq[dt]);
    }
  };
  if constexpr (ST == 1) {
    static_assert(NG == 1 || ST == 2, "groups are double-buffered");
    for (int p = p0; p < p1; ++p) {
      wait_vm<0>();  // this wave's copies of the block have landed,
      barrier();     // every wave's have
      const int cc = cn;
      cn = ld_meta(a.col_idx + min(p + 2, p1 - 1));
      scores(k0s, v0s, 0);
      grads(k0s, 0);
      scores(k0s, v0s, 1);
      wait_vm<0>();
      barrier();  // every wave has read V
      cp.issue(V + (int64_t)cc * BQ * D, v0s, p + 1 < p1);
      grads(k0s, 1);
      wait_vm<4>();
      barrier();  // every wave has read K
      cp.issue(K + (int64_t)cc * BQ * D, k0s, p + 1 < p1);
    }
  } else {
    uint8_t *const k1s = stage_buf<2, NG * TILE>() + grp * TILE;
    uint8_t *const v1s = stage_buf<3, NG * TILE>() + grp * TILE;
    auto step = [&](int it, uint8_t *kc, uint8_t *vc, uint8_t *kn, uint8_t *vn)
        __attribute__((always_inline)) {
      const int p = p0 + it * NG + grp;
      wait_vm<0>();
      barrier();
      if (p + NG < p1) {
        cp.issue(K + (int64_t)cn * BQ * D, kn, true);
        cp.issue(V + (int64_t)cn * BQ * D, vn, true);
      }
      cn = ld_meta(a.col_idx + min(p + 2 * NG, p1 - 1));
      if (NG > 1 && p >= p1) return;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        scores(kc, vc, kt);
        grads(kc, kt);
      }
    };
    for (int it = 0; it < iters; it += 2) {
      step(it, k0s, v0s, k1s, v1s);
      if (it + 1 < iters) step(it + 1, k1s, v1s, k0s, v0s);
    }
  }
  wait_vm<0>();  // no copy outlives the workgroup

  if constexpr (NG > 1) {
    // Groups 1.. leave their 32 partial sums per lane in their tiles; group
    // 0 adds them in group order.
    barrier();
    if (grp > 0) {
      float *m0 = merge_at(kst, grp, w, lane), *m1 = merge_at(vst, grp, w, lane);
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        m0[e * 64] = dq[0][e];
        m1[e * 64] = dq[1][e];
      }
    }
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int g = 1; g < NG; ++g) {
      const float *m0 = merge_at(kst, g, w, lane), *m1 = merge_at(vst, g, w, lane);
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        dq[0][e] += m0[e * 64];
        dq[1][e] += m1[e * 64];
      }
    }
  }
  store_row((bf16_t *)a.dQ + head + (int64_t)q * D, dq, a.scale, lane);
}

// ---------------------------------------------------------------------------
// Backward, pass 2: dK and dV (a group per key block)
// ---------------------------------------------------------------------------
// NG groups split the column's kept blocks as in the forward; their dK and
// dV partial sums are added through LDS in group order.
template <int NG>
__global__ __launch_bounds__(128 * NG) void attn_bwd_dkv_kernel(AttnArgs a) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & 1);
  const int grp = NG > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 7) : 0;
  uint8_t *const qs0 = stage_buf<0, NG * TILE>(), *const ds0 = stage_buf<1, NG * TILE>();
  uint8_t *const qs1 = stage_buf<2, NG * TILE>(), *const ds1 = stage_buf<3, NG * TILE>();
  // Row terms of the 64 queries: lse (log2 units), then -delta.
  __shared__ __attribute__((aligned(16))) float rt0[NG][2 * BQ], rt1[NG][2 * BQ];

  const int bid = xcd_remap(blockIdx.x, gridDim.x) + a.first;
  int bh, kb;
  attn_order(bid, a.BH, a.nbq, a.nlong, bh, kb);
  const int64_t head = (int64_t)bh * a.S * D;
  const bf16_t *Q = (const bf16_t *)a.Q + head;
  const bf16_t *K = (const bf16_t *)a.K + head;
  const bf16_t *V = (const bf16_t *)a.V + head;
  const bf16_t *dO = (const bf16_t *)a.dO + head;
  // Wave 0 of a group carries the lse values, wave 1 the delta values.
  const float *rt_g = (w == 0 ? a.lse_in : a.delta) + (int64_t)bh * a.S;
  const float rt_scale = w == 0 ? kLog2e : -1.f;
  const int k0 = kb * BQ + w * 32;
  const float c = a.scale * kLog2e;

  const int p0 = ld_meta(a.col_ptr + kb), p1 = ld_meta(a.col_ptr + kb + 1);
  f32x16 dk[2], dv[2];
#pragma unroll
  for (int e = 0; e < 16; ++e) dk[0][e] = dk[1][e] = dv[0][e] = dv[1][e] = 0.f;

  if (p0 < p1) {  // a key block no query attends keeps zero gradients
    const int iters = (p1 - p0 + NG - 1) / NG;
    TileCopy cp;
    cp.init(lane, w);
    float rt = 0.f;  // raw row term of the block in flight
    auto issue = [&](int row, uint8_t *qt, uint8_t *dt) __attribute__((always_inline)) {
      cp.issue(Q + (int64_t)row * BQ * D, qt + grp * TILE, true);
      cp.issue(dO + (int64_t)row * BQ * D, dt + grp * TILE, true);
      rt = rt_g[row * BQ + lane];
    };
    if (p0 + grp < p1) issue(ld_meta(a.row_idx + p0 + grp), qs0, ds0);
    bf16x8 kf[4], vf[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      kf[ks] = frag_g(K, k0, ks, lane);
      vf[ks] = frag_g(V, k0, ks, lane);
    }
    int rn = ld_meta(a.row_idx + min(p0 + grp + NG, p1 - 1));

    auto step = [&](int it, uint8_t *qc, uint8_t *dc, float (&rc)[NG][2 * BQ], uint8_t *qn,
                    uint8_t *dn) __attribute__((always_inline)) {
      const int p = p0 + it * NG + grp;
      wait_vm<0>();
      // The stage's row terms were last read two blocks ago, before the
      // previous barrier.
      rc[grp][w * BQ + lane] = rt * rt_scale;
      wait_vm<0>();
      barrier();
      if (p + NG < p1) issue(rn, qn, dn);
      rn = ld_meta(a.row_idx + min(p + 2 * NG, p1 - 1));
      if (p >= p1) return;
      qc += grp * TILE;
      dc += grp * TILE;
      const float *lsep = &rc[grp][(lane >> 5) * 4], *delp = lsep + BQ;
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
        // S[query][key], dP[query][key] for 32 queries x this wave's 32 keys.
        // The accumulators of dP start at -delta.
        f32x16 s = {}, dp;
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
          const f32x4 de = *(const f32x4 *)(delp + qt * 32 + e4 * 8);
#pragma unroll
          for (int j = 0; j < 4; ++j) dp[e4 * 4 + j] = de[j];
        }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          s = MFMA32(frag_r(qc, qt * 32, ks, lane), kf[ks], s);
          dp = MFMA32(frag_r(dc, qt * 32, ks, lane), vf[ks], dp);
        }
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
          const f32x4 ls = *(const f32x4 *)(lsep + qt * 32 + e4 * 8);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int e = e4 * 4 + j;
            const float pr = fast_exp2(s[e] * c - ls[j]);
            s[e] = pr;
            dp[e] = pr * dp[e];  // dS
          }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const bf16x8 pb = pack_k(s, j), sb = pack_k(dp, j);
#pragma unroll
          for (int dt = 0; dt < 2; ++dt) {
            dv[dt] = MFMA32(frag_t(dc, qt * 32 + j * 16, dt * 32, lane), pb, dv[dt]);
            dk[dt] = MFMA32(frag_t(qc, qt * 32 + j * 16, dt * 32, lane), sb, dk[dt]);
          }
        }
      }
    };
    for (int it = 0; it < iters; it += 2) {
      step(it, qs0, ds0, rt0, qs1, ds1);
      if (it + 1 < iters) step(it + 1, qs1, ds1, rt1, qs0, ds0);
    }
  }

  if constexpr (NG > 1) {
    // Groups 1.. leave their 64 partial sums per lane in their tiles; group
    // 0 adds them in group order.  (The key block's kept-block count is
    // workgroup-uniform, so every thread reaches these barriers.)
    wait_vm<0>();
    barrier();
    if (grp > 0) {
      float *m0 = merge_at(qs0, grp, w, lane), *m1 = merge_at(ds0, grp, w, lane);
      float *m2 = merge_at(qs1, grp, w, lane), *m3 = merge_at(ds1, grp, w, lane);
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        m0[e * 64] = dk[0][e];
        m1[e * 64] = dk[1][e];
        m2[e * 64] = dv[0][e];
        m3[e * 64] = dv[1][e];
      }
    }
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int g = 1; g < NG; ++g) {
      const float *m0 = merge_at(qs0, g, w, lane), *m1 = merge_at(ds0, g, w, lane);
      const float *m2 = merge_at(qs1, g, w, lane), *m3 = merge_at(ds1, g, w, lane);
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        dk[0][e] += m0[e * 64];
        dk[1][e] += m1[e * 64];
        dv[0][e] += m2[e * 64];
        dv[1][e] += m3[e * 64];
      }
    }
  }

  const int64_t key = k0 + (lane & 31);
  store_row((bf16_t *)a.dK + head + key * D, dk, a.scale, lane);
  store_row((bf16_t *)a.dV + head + key * D, dv, 1.f, lane);
}

}  // namespace

// Launchers.  part 0: every block row (column) with the plain kernel;
// part 1: the nlong global rows (columns) of every head with the grouped
// kernel; part 2: the remaining rows with the plain kernel.
//
// `few` (two groups per block row, two stages per operand) is the plain kernel
// of launches of at most two workgroups per CU: nothing else runs on the CU
// then, and a row's serial chain of blocks is the time.  It takes rows of two
// blocks and more on average while no CU has a second workgroup, of three and a
// half and more up to two.  One group, one stage / two groups, two stages, forward and
// dQ (us): 144 workgroups, 2 blocks per row 4.3 + 5.9 / 4.3 + 5.5, 3 blocks 4.7 +
// 6.6 / 4.7 + 6.0; 384 workgroups, 2 blocks 5.0 + 7.2 / 5.4 + 7.6, 3 blocks 6.4 + 8.8 / 6.4 +
// 8.7, 3.7 blocks 6.7 + 9.8 / 6.6 + 8.9; 768 workgroups, 5 blocks 9.6 + 13.5 / 11.6 + 15.1.
// The average is of the launch's own rows: a stripe's long rows, in a launch of
// their own, say nothing about the others.
//
// The grouped kernels take four groups in two stages.  Eight groups in one
// stage, as many waves and bytes of LDS per block in flight, pay for a longer
// merge and a wait per operand.  12 heads x 384 / 1024 / 4096, one stripe, forward
// + dQ of both launches, us, with 16-row waves in four groups / eight groups / four
// groups: 30.7 / 35.7 / 30.2, 39.1 / 43.4 / 36.6, 85.4 / 78.0 / 69.5; 96 heads 33.3 /
// 38.9 / 33.0, 59.0 / 58.7 / 51.0, 181 / 166 / 155.
namespace {
constexpr int64_t kAttnFewWG = 512;
template <typename F1, typename FG>
hipError_t attn_launch(F1 plain, F1 few, int nfew, FG grouped, int ng, AttnArgs a, int part,
                       hipStream_t s) {
  // Block rows of the launch and their kept blocks (a long row keeps all).
  int64_t grid, rows = a.nbq, nnzb = a.nnzb;
  if (part == 2) {
    rows -= a.nlong;
    nnzb -= (int64_t)a.nlong * a.nbq;
  }
  if (part == 1) {
    grid = (int64_t)a.BH * a.nlong;
    a.first = 0;
  } else if (part == 2) {
    grid = (int64_t)a.BH * (a.nbq - a.nlong);
    a.first = a.BH * a.nlong;
  } else {
    grid = (int64_t)a.BH * a.nbq;
    a.first = 0;
  }
  if (grid <= 0 || grid > 0x7fffffff) return hipErrorInvalidValue;
  if (part == 1)
    launch_kernel(grouped, dim3((unsigned)grid), dim3(128 * ng), s, a);
  else if (grid <= kAttnFewWG && 2 * nnzb >= (grid <= kAttnFewWG / 2 ? 4 : 7) * rows)
    launch_kernel(few, dim3((unsigned)grid), dim3(128 * nfew), s, a);
  else
    launch_kernel(plain, dim3((unsigned)grid), dim3(128), s, a);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_attn_fwd(const AttnArgs &a, int part, hipStream_t s) {
  return attn_launch(attn_fwd_kernel<1, 1>, attn_fwd_kernel<2, 2>, 2, attn_fwd_kernel<4, 2>, 4, a,
                     part, s);
}

hipError_t launch_attn_bwd_dq(const AttnArgs &a, int part, hipStream_t s) {
  return attn_launch(attn_bwd_dq_kernel<1, 1>, attn_bwd_dq_kernel<2, 2>, 2,
                     attn_bwd_dq_kernel<4, 2>, 4, a, part, s);
}

hipError_t launch_attn_bwd_dkv(const AttnArgs &a, int part, hipStream_t s) {
  return attn_launch(attn_bwd_dkv_kernel<1>, attn_bwd_dkv_kernel<1>, 1, attn_bwd_dkv_kernel<4>, 4,
                     a, part, s);
}

// Scratch of the allocation-free attention backward: the row terms delta,
// one float per query row of the call (kAttnScratchRows at most).  Each GPU
// the library runs on holds its own copy until the process ends.  In host
// code `scratch` names a host-side stand-in, not device memory: only the
// address attn_scratch returns may reach a kernel.
static __device__ __align__(256) float scratch[kAttnScratchRows];

hipError_t attn_scratch(float **ptr) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void *addr[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(mu);
  if (!addr[dev]) {
    // Once per device, with that device current: its copy of the array.
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *ptr = (float *)addr[dev];
  return hipSuccess;
}

}  // namespace pf

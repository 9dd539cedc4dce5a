// Rank-r products of the low-rank term (bf16), Section 3.3's U (V^T x)
// evaluated for a batch of tokens:
//
//   T_lr = X V^T   V is r x K row-major: B read as [n][k]   (BKN = false)
//   S    = dY U    U is N x r row-major: B read as [k][n]   (BKN = true)
//
// C[M x r] = A[M x K] . op(B) with r small (a multiple of the block size).
// The block-sparse tile kernels would need a split of K with fp32 partials
// and a second pass to keep the chip busy at this width.  Here one workgroup
// owns a small TM x TN tile and its NW waves split the K range among
// themselves (wave w takes the 64-wide K steps w, w + NW, ...), each
// accumulating the whole tile; the NW tiles are summed through LDS in wave
// order (deterministic) and stored once.
//
// The product is bound by the operand bytes each compute unit reads,
// (TM + TN) K 2 per workgroup, and by how many of them are in flight.  Every
// wave copies its own steps global -> LDS directly (whole 128-byte row
// segments, NS steps in flight, no barrier in the loop) into a private
// region, chunks XOR-swizzled so that the MFMA operand reads and the
// transpose reads of a [k][n] B (U) have no bank conflicts.  Reading the
// operands from global memory in MFMA layout instead (16 rows of 32 bytes
// per request; before / now, the kernel in a loop over one call): T_lr of 4096 x
// 768 to r = 96 6.6 / 5.7 us, 4096 x 3072 19.7 / 8.7, 1024 x 8192 to r = 256 48.6 / 13.7,
// 2509 x 4096 to r = 256 52.2 / 13.9; S of 4096 x 3072 to r = 96 12.8 / 10.9, 512 x 4096
// to r = 64 14.8 / 7.5.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "pf_dma.h"
#include "pf_launch.h"

namespace pf {
namespace {

constexpr int SK_BK = 64;  // K per step

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)lo) |
         ((uint32_t)__builtin_bit_cast(uint16_t, (__bf16)hi) << 16);
}

template <bool BKN, int TM, int TN, int NW, int NS>
__global__ __launch_bounds__(64 * NW) void skinny_kernel(SkinnyArgs a) {
  constexpr int A_BYTES = TM * 128, B_BYTES = TN * 128;  // one step of one wave
  constexpr int ROWB = BKN ? TN * 2 : 128;               // B row of the LDS tile
  constexpr int NWA = A_BYTES / 1024, NWB = B_BYTES / 1024, DPS = NWA + NWB;
  constexpr int MT = TM / 32, NT = TN / 32;
  static_assert(NS >= 2 && NS <= 4 && DPS * (NS - 1) < 64, "copies in flight");

  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ncol_tiles = (a.ncols + TN - 1) / TN;
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const int tt = bid / ncol_tiles, ct = bid % ncol_tiles;  // column tiles of a token tile adjacent
  const int64_t t0 = (int64_t)tt * TM;
  const int n0 = ct * TN;
  const int ksteps = (a.K + SK_BK - 1) / SK_BK;

  // Stages: a separate LDS object per stage and operand (see pf_dma.h).
  auto stage_a = [&](auto j) __attribute__((always_inline)) -> uint8_t * {
    return stage_buf<decltype(j)::value, NW * A_BYTES>() + w * A_BYTES;
  };
  auto stage_b = [&](auto j) __attribute__((always_inline)) -> uint8_t * {
    return stage_buf<8 + decltype(j)::value, NW * B_BYTES>() + w * B_BYTES;
  };

  // Rows past M (and, for [n][k], past r) read as zero by the buffer range;
  // chunks past K, and columns of U past r, are pointed out of range (the
  // host keeps every operand below that offset).
  constexpr uint32_t OUT = 0x7ffffff0u;
  const int64_t a_rows = a.M - t0 < TM ? a.M - t0 : TM;
  const bf16_t *const abase = (const bf16_t *)a.A + t0 * a.lda;
  const int64_t abytes = a_rows * a.lda * 2;
  const bf16_t *const bbase = (const bf16_t *)a.B + (BKN ? 0 : (int64_t)n0 * a.ldb);
  const int64_t bbytes = BKN ? (int64_t)a.K * a.ldb * 2 : (int64_t)(a.ncols - n0) * a.ldb * 2;
  const rsrc_t rA = make_rsrc(abase, abytes), rB = make_rsrc(bbase, bbytes);
  // Lane part of a copy: row lane / 8 of the window, source chunk of the
  // swizzled position (even / odd windows of 8 rows).
  int chunk[2];
  chunk[0] = (lane & 7) ^ (lane >> 4);
  chunk[1] = chunk[0] ^ 4;
  const uint32_t arow = (uint32_t)((lane >> 3) * a.lda * 2);
  constexpr int LPR = ROWB / 16;  // lanes per [k][n] row
  uint32_t bvoff = 0;             // [k][n]: row and column of this lane's chunk
  if constexpr (BKN) {
    const int row = lane / LPR, c = (lane % LPR) ^ (LPR == 8 ? ((lane >> 4) & 1) << 2 : 0);
    bvoff = n0 + c * 8 < a.ncols ? (uint32_t)(row * a.ldb * 2 + (n0 + c * 8) * 2) : OUT;
  }
  const uint32_t brow = (uint32_t)((lane >> 3) * a.ldb * 2);

  // Steps in an order rotated per token tile, so that the workgroups do not
  // all read the same columns of rows a power of two apart at a time.
  const int rot = (tt * NW) % ksteps;
  auto issue = [&](int i, uint8_t *da, uint8_t *db) __attribute__((always_inline)) {
    int s = w + i * NW;
    const bool live = s < ksteps;
    s += rot;
    if (s >= ksteps) s -= ksteps;
    s = __builtin_amdgcn_readfirstlane(live ? s : 0);
    uint32_t vk[2];  // K offset of the lane's chunk within a row
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      const int k = s * SK_BK + chunk[o] * 8;
      vk[o] = live && k < a.K ? (uint32_t)(k * 2) : OUT;
    }
    sfor<NWA>([&](auto i) __attribute__((always_inline)) {
      const uint32_t v = vk[i & 1] == OUT ? OUT : arow + vk[i & 1];
      dma16(rA, da + i * 1024, v, (uint32_t)(i * 8 * a.lda * 2));
    });
    if constexpr (!BKN) {
      sfor<NWB>([&](auto i) __attribute__((always_inline)) {
        const uint32_t v = vk[i & 1] == OUT ? OUT : brow + vk[i & 1];
        dma16(rB, db + i * 1024, v, (uint32_t)(i * 8 * a.ldb * 2));
      });
    } else {
      // The step's rows go into the lane part, which the range check covers:
      // rows past K fall outside the buffer.
      sfor<NWB>([&](auto i) __attribute__((always_inline)) {
        const uint32_t rows = (uint32_t)((s * SK_BK + i * (64 / LPR)) * a.ldb * 2);
        dma16(rB, db + i * 1024, live && bvoff != OUT ? bvoff + rows : OUT, 0);
      });
    }
  };

  f32x16 acc[NT][MT];
  sfor<NT>([&](auto j) __attribute__((always_inline)) {
    sfor<MT>([&](auto m) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[j][m][e] = 0.f;
    });
  });
  auto compute = [&](const uint8_t *da, const uint8_t *db) __attribute__((always_inline)) {
    sfor<4>([&](auto ks) __attribute__((always_inline)) {
      bf16x8 xf[MT];
      sfor<MT>([&](auto m) __attribute__((always_inline)) {
        xf[m] = frag_rows<128>(da, m * 32, ks, lane);
      });
      sfor<NT>([&](auto j) __attribute__((always_inline)) {
        bf16x8 wf;
        if constexpr (BKN) wf = frag_kn<ROWB>(db, j * 32, ks, lane);
        else wf = frag_rows<128>(db, j * 32, ks, lane);
        // D rows = output columns, D columns = tokens: lane l ends with token
        // l % 32 and columns (e / 4) * 8 + (l / 32) * 4 + e % 4 of tile j.
        sfor<MT>([&](auto m) __attribute__((always_inline)) {
          acc[j][m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, xf[m], acc[j][m], 0, 0, 0);
        });
      });
    });
  };

  // Each wave on its own: NS steps in flight, a stage refilled as soon as
  // its reads have returned.  Whole rounds of NS steps; steps past the end
  // copy nothing and add zeros, so the waits stay counted.
  const int n = (ksteps + NW - 1) / NW;
  sfor<NS>([&](auto j) __attribute__((always_inline)) { issue(j, stage_a(j), stage_b(j)); });
  for (int i = 0; i < n; i += NS) {
    sfor<NS>([&](auto j) __attribute__((always_inline)) {
      wait_vm<DPS *(NS - 1)>();
      compute(stage_a(j), stage_b(j));
      wait_vm<DPS *(NS - 1)>();  // (LDS reads returned)
      issue(i + NS + j, stage_a(j), stage_b(j));
    });
  }

  // Sum the waves' tiles in wave order through LDS: every wave leaves its
  // 32 x 32 blocks (4 KiB fp32, lane-major: float index e * 64 + lane) in its
  // own part of stage 0, the first MT in A's and the rest in B's.
  wait_vm<0>();
  __syncthreads();
  auto red = [&](int ww, int blk) __attribute__((always_inline)) -> float * {
    return (float *)(blk < MT ? stage_buf<0, NW * A_BYTES>() + ww * A_BYTES + blk * 4096
                              : stage_buf<8, NW * B_BYTES>() + ww * B_BYTES + (blk - MT) * 4096);
  };
  static_assert(MT * NT <= MT + NT, "reduction room");
  sfor<NT>([&](auto j) __attribute__((always_inline)) {
    sfor<MT>([&](auto m) __attribute__((always_inline)) {
      float *const r = red(w, j * MT + m);
#pragma unroll
      for (int e = 0; e < 16; ++e) r[e * 64 + lane] = acc[j][m][e];
    });
  });
  __syncthreads();
  // Items: 4 consecutive output columns of one token row each.
  for (int item = threadIdx.x; item < NT * MT * 4 * 64; item += 64 * NW) {
    const int l = item & 63, g = (item >> 6) & 3, blk = item >> 8;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) {
      const float *const r = red(ww, blk) + g * 256 + l;
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] += r[q * 64];
    }
    const int64_t t = t0 + (blk % MT) * 32 + (l & 31);
    const int col = n0 + (blk / MT) * 32 + g * 8 + (l >> 5) * 4;
    if (t < a.M && col < a.ncols) {
      bf16_t *dst = (bf16_t *)a.C + t * a.ldc + col;
      *(u32x2 *)dst = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
    }
  }
}

template <bool BKN, int TM, int TN, int NW, int NS>
hipError_t skinny_go(const SkinnyArgs &a, hipStream_t s) {
  const int64_t tiles = ((a.M + TM - 1) / TM) * ((a.ncols + TN - 1) / TN);
  if (tiles <= 0 || tiles > 0x7fffffff) return hipErrorInvalidValue;
  launch_kernel(skinny_kernel<BKN, TM, TN, NW, NS>, dim3((unsigned)tiles), dim3(64 * NW), s, a);
  return hipGetLastError();
}

template <bool BKN>
hipError_t skinny_pick(const SkinnyArgs &a, hipStream_t s) {
  // Long K: as many waves as the LDS holds (S of 2100 x 4096 to r = 128:
  // 13.1 us with six waves, 15.6 with four); short K: four, whose few steps
  // each need no third stage.
  const bool deep = a.K >= 48 * SK_BK;
  const SkinnyTile t = skinny_tile(BKN, a.M, a.ncols);
  if (t.m == 64 && t.n == 64) return skinny_go<BKN, 64, 64, 4, 2>(a, s);
  if (t.m == 64) return skinny_go<BKN, 64, 32, 4, 2>(a, s);
  if (t.n == 64)
    return deep ? skinny_go<BKN, 32, 64, 6, 2>(a, s) : skinny_go<BKN, 32, 64, 4, 2>(a, s);
  return deep ? skinny_go<BKN, 32, 32, 8, 2>(a, s) : skinny_go<BKN, 32, 32, 4, 2>(a, s);
}

}  // namespace

hipError_t launch_skinny(bool b_kn, const SkinnyArgs &a, hipStream_t s) {
  return b_kn ? skinny_pick<true>(a, s) : skinny_pick<false>(a, s);
}

}  // namespace pf

// NT products of few output tiles (bf16 and fp32): the block-sparse forward
// and backward-data of small token counts, and the fp32 rank-r products.
//
//   C[M x n] = A[M x k] . B^T over a tile's virtual K list (its kept blocks,
//   then the low-rank blocks), as the NT kernels of gemm_dma.hip.
//
// With few token rows the 128-row tiles of those kernels leave most of the
// chip idle, and each workgroup walks its K list alone: the time is the
// launch plus a serial chain of loads.  Here a workgroup owns 32 token rows x
// 32 output columns (a 32-column slice of one output block) and its NW waves
// split the K list among themselves, 128 bytes of every row per step (wave w
// takes steps w, w + NW, ...).  Each wave copies its steps global -> LDS
// directly into a private double-buffered region (no barrier in the loop, both
// stages in flight before the first wait); the waves' 32 x 32 sums are added
// through LDS in wave order (deterministic), and the epilogue (GELU, GELU',
// mixing weight) is applied once.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "pf_dma.h"
#include "pf_gelu.h"
#include "pf_launch.h"

namespace pf {
namespace {

// Vector of 4 outputs to memory.
__device__ __forceinline__ void put4(bf16_t *p, const float (&v)[4]) {
  auto h = [](float x) { return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)x); };
  *(u32x2 *)p = u32x2{h(v[0]) | (h(v[1]) << 16), h(v[2]) | (h(v[3]) << 16)};
}
__device__ __forceinline__ void put4(float *p, const float (&v)[4]) {
  *(f32x4 *)p = f32x4{v[0], v[1], v[2], v[3]};
}
__device__ __forceinline__ f32x4 get4(const bf16_t *p) {
  const u32x2 x = *(const u32x2 *)p;
  return f32x4{__uint_as_float(x[0] << 16), __uint_as_float(x[0] & 0xffff0000u),
               __uint_as_float(x[1] << 16), __uint_as_float(x[1] & 0xffff0000u)};
}
__device__ __forceinline__ f32x4 get4(const float *p) { return *(const f32x4 *)p; }

// fp32 outputs keep the library erff (as in the NT kernels they replace).
template <typename T>
__device__ __forceinline__ float gelu_s(float x) {
  if constexpr (sizeof(T) == 2) return gelu_fast(x);
  else return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f));
}
template <typename T>
__device__ __forceinline__ float gelu_grad_s(float x) {
  if constexpr (sizeof(T) == 2) return gelu_grad_fast(x);
  else {
    const float cdf = 0.5f * (1.0f + erff(x * 0.70710678118654752f));
    return cdf + x * (0.39894228040143268f * __expf(-0.5f * x * x));
  }
}

// T: bf16 or float storage.  NH: sub-blocks per step (2 for bf16 blocks of 32,
// half a 128-byte step each).  BKN: B read as [k][n].  EPI: 0 none, 1 GELU
// forward, 2 GELU backward.
template <typename T, int NH, bool BKN, bool DENSE, int EPI, int NW>
__global__ __launch_bounds__(64 * NW) void small_kernel(SmallArgs a) {
  constexpr int ES = sizeof(T), KW = 128 / NH / ES;  // K width of a sub-block
  constexpr int RBA = KW * ES;                       // its bytes per row: 128 or 64
  constexpr int RBB = BKN ? 32 * ES : RBA;
  constexpr int SUB = 4096 / NH;                     // bytes of an A or B sub-block
  constexpr int WPS = SUB / 1024;                    // 1 KiB copies per sub-block
  constexpr int DPS = 2 * NH * WPS;                  // copies per wave and step (8)
  const NTArgs &n = a.nt;

  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const int mtiles = (int)((n.M + 31) / 32);
  const int mt = bid % mtiles, cs = bid / mtiles;  // token tiles of a slice adjacent
  const int64_t m0 = (int64_t)mt * 32;
  const int lb = a.log2_blk, blk = 1 << lb, sl = blk >> 5;

  // The 32-column slice: output block ob, columns c0 .. c0 + 31 of it.
  int nsteps, kcol_off = 0, blk_off = 0, g = 0, ob, c0;
  if constexpr (DENSE) {
    nsteps = n.dense_nsteps;
    ob = cs / sl;
    c0 = cs % sl * 32;
  } else {
    const int o = cs / sl;
    const NTTile *tile = n.tiles + o / a.G;
    g = o % a.G;
    c0 = cs % sl * 32;
    if (g >= ld_meta(&tile->g)) return;
    nsteps = ld_meta(&tile->nsteps);
    kcol_off = ld_meta(&tile->kcol_off);
    blk_off = ld_meta(&tile->blk_off);
    ob = ld_meta(&tile->out_blk[g]);
  }
  const int64_t col0 = (int64_t)ob * blk + c0;
  const int vblocks = nsteps + n.nlr;
  const int total = ((vblocks << lb) + KW * NH - 1) / (KW * NH);

  auto stage_a = [&](auto j) __attribute__((always_inline)) -> uint8_t * {
    return stage_buf<decltype(j)::value, NW * 4096>() + w * 4096;
  };
  auto stage_b = [&](auto j) __attribute__((always_inline)) -> uint8_t * {
    return stage_buf<8 + decltype(j)::value, NW * 4096>() + w * 4096;
  };

  // Epilogue item of this thread (the first 256 threads): 4 consecutive
  // columns of one token row.  Its pre-activations are loaded up front.
  const int il = threadIdx.x & 63, ig = threadIdx.x >> 6;
  const int64_t et = m0 + (il & 31);
  const int64_t eoff = et * n.ldc + col0 + ig * 8 + (il >> 5) * 4;
  const bool elive = threadIdx.x < 256 && et < n.M;
  f32x4 aux = {0.f, 0.f, 0.f, 0.f};
  if constexpr (EPI == 2)
    if (elive) aux = get4((const T *)n.aux + eoff);

  // Lane part of the copies.  Rows of 8 chunks are swizzled by row pair (two
  // variants: even / odd windows), rows of 4 by groups of 4 rows; a [k][n]
  // tile lies unswizzled (64-byte rows: conflict-free transpose reads).
  constexpr int CPRA = RBA / 16, CPRB = RBB / 16;
  constexpr uint32_t OUT = 0x7ffffff0u;
  uint32_t a_chunk[2], b_chunk[2];
  a_chunk[0] = (uint32_t)(((lane % CPRA) ^ ((lane >> 4) & 3)) << 4);
  a_chunk[1] = CPRA == 8 ? a_chunk[0] ^ 64u : a_chunk[0];
  if constexpr (BKN) b_chunk[0] = b_chunk[1] = (uint32_t)((lane % CPRB) << 4);
  else {
    b_chunk[0] = a_chunk[0];
    b_chunk[1] = a_chunk[1];
  }
  const uint32_t a_row = (uint32_t)(lane / CPRA), b_row = (uint32_t)(lane / CPRB);

  auto issue = [&](int i, uint8_t *da, uint8_t *db) __attribute__((always_inline)) {
    const int s = w + i * NW;
    sfor<NH>([&](auto h) __attribute__((always_inline)) {
      const int k0 = __builtin_amdgcn_readfirstlane((s * NH + h) * KW);
      const int c = k0 >> lb, kk = k0 & (blk - 1);
      const bool sp = c < nsteps, live = c < vblocks;
      const int cc = min(c, nsteps - 1), cr = min(c, vblocks - 1) - nsteps;
      const T *ab, *bb;
      int64_t lda, ldb, acol;
      if constexpr (DENSE) {
        const int kl = live ? k0 : 0;
        ab = (const T *)n.A + m0 * n.lda;
        lda = n.lda;
        acol = kl;
        ldb = n.ldb;
        bb = (const T *)n.B + (BKN ? (int64_t)kl * ldb + col0 : col0 * ldb + kl);
      } else {
        const int kcol = ld_meta(&n.kcols[kcol_off + max(cc, 0)]);
        const int64_t pb = ld_meta(&n.blks[blk_off + max(cc, 0) * a.G + g]);
        const T *spb = (const T *)n.B + (pb << (2 * lb)) + (BKN ? kk * blk + c0 : c0 * blk + kk);
        const int64_t kr = (int64_t)max(cr, 0) * blk + kk;
        const T *lrb = (const T *)n.R + (BKN ? kr * n.ldr + col0 : col0 * n.ldr + kr);
        ab = sp ? (const T *)n.A + m0 * n.lda : (const T *)n.L + m0 * n.ldl;
        lda = sp ? n.lda : n.ldl;
        acol = ((int64_t)(sp ? kcol : max(cr, 0)) << lb) + kk;
        bb = sp ? spb : lrb;
        ldb = sp ? blk : n.ldr;
      }
      // Rows past M fall outside A's range, which covers this tile's rows only:
      // OUT, where a dead sub-block is pointed, then lies outside it however
      // large the operand (the host keeps 512 rows below 2^31 bytes).  B's rows
      // all exist.
      const rsrc_t rA = make_rsrc(ab, min<int64_t>(32, n.M - m0) * lda * ES);
      const rsrc_t rB = make_rsrc(bb, 0x7ffffff0);
      const uint32_t av = a_row * (uint32_t)(lda * ES) + (uint32_t)(acol * ES);
      const uint32_t bv = b_row * (uint32_t)(ldb * ES);
      sfor<WPS>([&](auto i) __attribute__((always_inline)) {
        dma16(rA, da + h * SUB + i * 1024, live ? av + a_chunk[i & 1] : OUT,
              (uint32_t)(i * (1024 / RBA) * lda * ES));
      });
      sfor<WPS>([&](auto i) __attribute__((always_inline)) {
        dma16(rB, db + h * SUB + i * 1024, live ? bv + b_chunk[i & 1] : OUT,
              (uint32_t)(i * (1024 / RBB) * ldb * ES));
      });
    });
  };

  // fp32: two accumulators, the even and the odd steps of the wave, so that no
  // chain of sums is longer than the tile kernel's K split leaves it (128 terms below
  // 1024 deep): T_lr of 512 x 896 to r = 64 is 2.1e-7 off by that split, 2.7e-7 with one
  // accumulator, 2.0e-7 so (0.2 us a launch).
  constexpr int NACC = ES == 4 ? 2 : 1;
  f32x16 acc[NACC];
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[0][e] = acc[NACC - 1][e] = 0.f;
  // Mixing weight: this wave's kept-block sums are scaled once, before its
  // first low-rank K slice or after its last step.
  bool scale = n.mix != 0;
  auto rescale = [&]() __attribute__((always_inline)) {
    sfor<NACC>([&](auto q) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[q][e] *= n.mix_ratio;
    });
    scale = false;
  };
  const int kswitch = nsteps << lb;
  // D rows = output columns, D columns = tokens: lane l ends with token l % 32
  // and columns (e / 4) * 8 + (l / 32) * 4 + e % 4.
  auto compute = [&](int i, auto j, const uint8_t *da, const uint8_t *db) __attribute__((always_inline)) {
    f32x16 &sum = acc[decltype(j)::value % NACC];
    const int s = w + i * NW;
    sfor<NH>([&](auto h) __attribute__((always_inline)) {
      if (scale && (s * NH + h) * KW >= kswitch) rescale();
      if constexpr (ES == 2) {
        sfor<KW / 16>([&](auto kq) __attribute__((always_inline)) {
          const bf16x8 xf = frag_rows<RBA>(da + h * SUB, 0, kq, lane);
          bf16x8 wf;
          if constexpr (BKN) wf = frag_kn<RBB>(db + h * SUB, 0, kq, lane);
          else wf = frag_rows<RBB>(db + h * SUB, 0, kq, lane);
          sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, xf, sum, 0, 0, 0);
        });
      } else {
        // Lane half h takes the K chunks 2 c + h (4 values): the MFMAs of c
        // visit k = 8 c + 4 h + 0..3.
        const int r = lane & 31, hf = lane >> 5, sw = swz_row<8>(r);
        sfor<4>([&](auto c) __attribute__((always_inline)) {
          const f32x4 x = *(const f32x4 *)(da + r * 128 + (((2 * c + hf) ^ sw) << 4));
          f32x4 b;
          if constexpr (BKN) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
              b[q] = *(const float *)(db + (8 * c + 4 * hf + q) * 128 + r * 4);
          } else {
            b = *(const f32x4 *)(db + r * 128 + (((2 * c + hf) ^ sw) << 4));
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) sum = __builtin_amdgcn_mfma_f32_32x32x2f32(b[q], x[q], sum, 0, 0, 0);
        });
      }
    });
  };

  // Each wave on its own: two steps in flight, a stage refilled as soon as
  // its reads have returned.  Steps past the end copy nothing and add zeros.
  const int steps = (total + NW - 1) / NW;
  sfor<2>([&](auto j) __attribute__((always_inline)) { issue(j, stage_a(j), stage_b(j)); });
  for (int i = 0; i < steps; i += 2) {
    sfor<2>([&](auto j) __attribute__((always_inline)) {
      wait_vm<DPS>();
      compute(i + j, j, stage_a(j), stage_b(j));
      wait_vm<DPS>();  // (LDS reads returned)
      issue(i + 2 + j, stage_a(j), stage_b(j));
    });
  }
  if (scale) rescale();

  // Sum the waves' tiles in wave order (fp32, lane-major: float index e * 64 +
  // lane of wave w's stage 0).
  wait_vm<0>();
  __syncthreads();
  float *const red = (float *)stage_buf<0, NW * 4096>();
#pragma unroll
  for (int e = 0; e < 16; ++e)
    red[w * 1024 + e * 64 + lane] = NACC == 2 ? acc[0][e] + acc[NACC - 1][e] : acc[0][e];
  __syncthreads();
  if (!elive) return;
  float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ww = 0; ww < NW; ++ww)
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] += red[ww * 1024 + (ig * 4 + q) * 64 + il];
  if (n.mix) {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] *= n.mix_out;
  }
  if constexpr (EPI == 1) {
    put4((T *)n.C2 + eoff, v);
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = gelu_s<T>(v[q]);
  } else if constexpr (EPI == 2) {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] *= gelu_grad_s<T>(aux[q]);
  }
  put4((T *)n.C + eoff, v);
}

template <typename T, int NH, bool BKN, bool DENSE, int EPI>
hipError_t small_go(const SmallArgs &a, int64_t grid, bool deep, hipStream_t s) {
  if (deep)
    launch_kernel(small_kernel<T, NH, BKN, DENSE, EPI, 8>, dim3((unsigned)grid), dim3(512), s, a);
  else
    launch_kernel(small_kernel<T, NH, BKN, DENSE, EPI, 4>, dim3((unsigned)grid), dim3(256), s, a);
  return hipGetLastError();
}

template <typename T, int NH, bool BKN>
hipError_t small_epi(const SmallArgs &a, int64_t grid, bool deep, hipStream_t s) {
  if (a.nt.epi == 1) return small_go<T, NH, BKN, false, BKN ? 2 : 1>(a, grid, deep, s);
  return small_go<T, NH, BKN, false, 0>(a, grid, deep, s);
}

}  // namespace

hipError_t launch_small(int dtype, int blk, int G, bool b_kn, int kmax, const NTArgs &nt,
                        hipStream_t s) {
  SmallArgs a{nt, G, 0};
  while ((1 << a.log2_blk) < blk) ++a.log2_blk;
  if (blk < 32 || (1 << a.log2_blk) != blk) return hipErrorInvalidValue;
  const int64_t slices = nt.dense ? (int64_t)nt.dense_nblk * (blk / 32) : (int64_t)nt.ntiles * G * (blk / 32);
  const int64_t grid = ((nt.M + 31) / 32) * slices;
  if (grid <= 0 || grid > 0x7fffffff) return hipErrorInvalidValue;
  // Eight waves once four would have eight or more steps each.
  const bool deep = (int64_t)kmax * blk * (dtype == 0 ? 2 : 4) >= 32 * 128;
  if (nt.dense) {
    if (dtype == 0) return hipErrorInvalidValue;
    return b_kn ? small_go<float, 1, true, true, 0>(a, grid, deep, s)
                : small_go<float, 1, false, true, 0>(a, grid, deep, s);
  }
  if (dtype != 0)
    return b_kn ? small_epi<float, 1, true>(a, grid, deep, s) : small_epi<float, 1, false>(a, grid, deep, s);
  if (blk == 32)
    return b_kn ? small_epi<bf16_t, 2, true>(a, grid, deep, s) : small_epi<bf16_t, 2, false>(a, grid, deep, s);
  return b_kn ? small_epi<bf16_t, 1, true>(a, grid, deep, s) : small_epi<bf16_t, 1, false>(a, grid, deep, s);
}

}  // namespace pf

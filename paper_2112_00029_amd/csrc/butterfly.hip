// Product form of the block butterfly (Section 3.2: a product of factors,
// each a matrix on the support of I + B_k; appendix on benchmarking the
// butterfly multiply), applied to a batch of token rows in one launch.
//
// The product of the factors with strides 2 .. k is block-diagonal in groups
// of k blocks, so a workgroup owns TM token rows x NB = 2 NW blocks (one
// group, or several whole groups of a small k): it loads that activation
// tile into LDS once, applies the L = log2 k factors one after another, and
// writes the result.  A factor of stride 2^(f+1) maps each block pair (p, p + h),
// h = 2^f, onto itself:
//     forward        y_p = x_p W(p,p)^T + x_q W(p,q)^T,  q = p + h (and y_q alike)
//     backward-data  g'_p = g_p F(p,p) + g_q F(q,p)              (and g'_q alike)
// so every wave takes one pair, reads both input blocks from one LDS tile,
// runs the 32 x 32 block products on MFMA and writes both output blocks to
// the other tile; one barrier separates factors.  Optionally the input of
// every factor (forward) or the gradient at every factor's output (backward)
// is written out, token-major as [T][L][n], for the weight gradient, by the
// phase that reads the tile.
//
// What bounds it is the weights a compute unit reads, one whole group's per
// factor (2048 x 1024, five factors: 128 KiB per factor and workgroup, about
// 1 us at 64 bytes per clock; all bytes of the pass together take 6 us of
// memory time).  Hence 16 tokens per workgroup (16x16x32 MFMA: one block's
// whole K per instruction, 128 workgroups at that size), a wave per pair, and
// weights loaded one factor ahead as whole contiguous KiB, staged in a
// private LDS region of the wave (the forward reads its rows, the backward
// its columns with the transpose read).  Forward / backward pass with saved
// activations: 40 / 40 us with 32 tokens, 4 waves walking the pairs and the
// tile updated in place; 17.1 / 19.6 us so but with weights loaded in operand
// order (16 rows of 64 bytes apart per request); 15.4 / 15.0 us now.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pf_launch.h"

namespace pf {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef uint16_t bf16_t;

constexpr int BB = kBflyBlock;  // block size (32)
constexpr int TM = 16;          // token rows per workgroup
constexpr int BLK_BYTES = BB * BB * 2;

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)lo) |
         ((uint32_t)__builtin_bit_cast(uint16_t, (__bf16)hi) << 16);
}

__device__ __forceinline__ s16x4 tr16(const uint8_t *p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(p));
}

// Workgroup barrier for LDS alone: this wave's LDS accesses are done
// (lgkmcnt 0); the factor's saved rows and the next factor's weights stay in
// flight, which __syncthreads would wait for.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// One pair's four weight blocks in registers: chunk j holds 16-row half j % 2
// of block j / 2 of [W(p,p) W(p,q) W(q,p) W(q,q)], lane l 16 bytes at 16 l
// (row l / 4, columns 8 (l % 4) .. + 7).
struct WReg {
  u32x4 r[8];
};

template <bool BWD, int NW>
__global__ __launch_bounds__(64 * NW) void bfly_kernel(BflyArgs a) {
  constexpr int NB = 2 * NW;            // blocks per workgroup
  constexpr int CPR = NB * BB * 2 / 16;  // 16-byte chunks per activation row
  static_assert(CPR >= 16, "swizzle");
  __shared__ __attribute__((aligned(16))) uint8_t act_s[2][TM * CPR * 16];
  __shared__ __attribute__((aligned(16))) uint8_t wst_s[NW * 2 * BLK_BYTES];

  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, q4 = lane >> 4;
  const int nsets = (a.nb + NB - 1) / NB;
  const int tt = blockIdx.x / nsets, set = blockIdx.x % nsets;
  const int64_t t0 = (int64_t)tt * TM;
  const int b0 = set * NB;                     // first block of this workgroup
  const int nblk = min(NB, a.nb - b0);         // whole groups of k blocks
  const int64_t col0 = (int64_t)b0 * BB;
  const int rows = (int)min<int64_t>(TM, a.T - t0);
  const int cpv = nblk * (BB * 2 / 16);        // chunks per row in use

  // Activation tile: row m (token t0 + m), chunk c at position c XOR m, so
  // that the 16 rows a fragment read touches fall in distinct banks.
  auto act = [&](int buf, int m, int c) __attribute__((always_inline)) -> uint8_t * {
    return act_s[buf] + m * (CPR * 16) + ((c ^ m) << 4);
  };
  const bf16_t *F = (const bf16_t *)a.F;
  const bool live = 2 * w < nblk;
  // Block row p of pair w of factor f (p & h == 0).
  auto pair_row = [&](int f) __attribute__((always_inline)) -> int {
    return ((w >> f) << (f + 1)) | (w & ((1 << f) - 1));
  };
  auto wload = [&](int f, WReg &W) __attribute__((always_inline)) {
    if (!live) return;
    const int h = 1 << f;
    const int64_t P = (int64_t)b0 + pair_row(f);
    // The two kept blocks of a block row are contiguous (ascending column).
    const bf16_t *rp = F + ((int64_t)f * a.nb + P) * 2 * BB * BB;
    const bf16_t *rq = F + ((int64_t)f * a.nb + P + h) * 2 * BB * BB;
#pragma unroll
    for (int j = 0; j < 8; ++j)
      W.r[j] = *(const u32x4 *)((j < 4 ? rp : rq) + (j & 3) * (16 * BB) + lane * 8);
  };

  const int L = a.nfac;
  WReg WA, WB;
  wload(BWD ? L - 1 : 0, WA);
  const bf16_t *in = (const bf16_t *)a.in;
  for (int idx = threadIdx.x; idx < TM * CPR; idx += 64 * NW) {
    const int m = idx / CPR, c = idx % CPR;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (m < rows && c < cpv) v = *(const u32x4 *)(in + (t0 + m) * a.n + col0 + c * 8);
    *(u32x4 *)act(0, m, c) = v;
  }
  lds_barrier();

  // Copy of tile `buf` to dst (row stride ld elements, column offset off).
  auto copy_out = [&](int buf, bf16_t *dst, int64_t ld, int64_t off) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < TM * CPR / (64 * NW); ++i) {
      const int idx = threadIdx.x + i * 64 * NW, m = idx / CPR, c = idx % CPR;
      if (m < rows && c < cpv)
        *(u32x4 *)(dst + (t0 + m) * ld + off + col0 + c * 8) = *(const u32x4 *)act(buf, m, c);
    }
  };
  static_assert(TM * CPR % (64 * NW) == 0, "copy");

  // Two of the pair's blocks at a time in this wave's staging region, 32 rows
  // of 64 bytes.  Chunk c of a row sits at c ^ swz(row): the forward reads 16
  // rows at one chunk, the backward 4 rows of 4 row groups at a 32-byte half
  // (transpose read); both then fall in distinct banks.  A wave's LDS
  // accesses complete in order.
  uint8_t *const wst = wst_s + w * 2 * BLK_BYTES;
  auto swz = [](int row) __attribute__((always_inline)) -> int {
    return BWD ? ((row >> 3) & 1) << 1 : (row >> 2) & 3;
  };
  auto stage = [&](const WReg &W, int i) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = (j & 1) * 16 + (lane >> 2);
      *(u32x4 *)(wst + (j >> 1) * BLK_BYTES + row * 64 + (((lane & 3) ^ swz(row)) << 4)) =
          W.r[4 * i + j];
    }
  };
  // A[m][k] = block[16 half + m][k], k = 8 (l / 16) + 0..7.
  auto frag_row = [&](int blk, int half) __attribute__((always_inline)) -> bf16x8 {
    const int row = half * 16 + r16;
    return *(const bf16x8 *)(wst + blk * BLK_BYTES + row * 64 + ((q4 ^ swz(row)) << 4));
  };
  // A[m][k] = block[k][16 half + m], k = 8 (l / 16) + 0..7.
  auto frag_tr = [&](int blk, int half) __attribute__((always_inline)) -> bf16x8 {
    const int k = q4 * 8 + (r16 >> 2);
    const uint8_t *p = wst + blk * BLK_BYTES + k * 64 + ((half ^ (q4 & 1)) << 5) + (r16 & 3) * 8;
    const s16x4 lo = tr16(p), hi = tr16(p + 4 * 64);
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  };

  auto process = [&](int f, int src, const WReg &W) __attribute__((always_inline)) {
    if (!live) return;
    const int p = pair_row(f), q = p + (1 << f);
    // Token operand of a block: token l % 16, features 8 (l / 16) .. + 7.
    const bf16x8 x[2] = {*(const bf16x8 *)act(src, r16, p * 4 + q4),
                         *(const bf16x8 *)act(src, r16, q * 4 + q4)};
    f32x4 acc[2][2];  // [output block][16-feature half]
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) acc[o][hf] = f32x4{0.f, 0.f, 0.f, 0.f};
    // Forward: output o from input i uses W(o, i); staged pair s holds output
    // s's blocks.  Backward: F(i, o); staged pair s holds input s's blocks.
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      stage(W, s);
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
          const int o = BWD ? b : s, i = BWD ? s : b;
          acc[o][hf] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              BWD ? frag_tr(b, hf) : frag_row(b, hf), x[i], acc[o][hf], 0, 0, 0);
        }
    }
    // Lane l: token l % 16, features 16 hf + 4 (l / 16) .. + 3, as bf16.
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
      for (int hf = 0; hf < 2; ++hf) {
        const u32x2 v = {pack_bf16x2(acc[o][hf][0], acc[o][hf][1]),
                         pack_bf16x2(acc[o][hf][2], acc[o][hf][3])};
        *(u32x2 *)(act(src ^ 1, r16, (o ? q : p) * 4 + hf * 2 + (q4 >> 1)) + (q4 & 1) * 8) = v;
      }
  };

  bf16_t *save = (bf16_t *)a.save;
  const int64_t sld = (int64_t)L * a.n;
  // Factor fi of the order reads tile fi % 2: its weights are in Wc, the
  // next factor's go to Wn.
  auto phase = [&](int fi, int src, const WReg &Wc, WReg &Wn) __attribute__((always_inline)) {
    const int f = BWD ? L - 1 - fi : fi;
    if (fi + 1 < L) wload(BWD ? f - 1 : f + 1, Wn);
    process(f, src, Wc);
    if (save) copy_out(src, save, sld, (int64_t)f * a.n);
    lds_barrier();
  };
  int fi = 0;
  for (; fi + 1 < L; fi += 2) {
    phase(fi, 0, WA, WB);
    phase(fi + 1, 1, WB, WA);
  }
  if (fi < L) phase(fi, 0, WA, WB);
  copy_out(L & 1, (bf16_t *)a.out, a.n, 0);
}

template <int NW>
hipError_t bfly_go(bool bwd, const BflyArgs &a, hipStream_t s) {
  const int64_t grid = ((a.T + TM - 1) / TM) * ((a.nb + 2 * NW - 1) / (2 * NW));
  if (grid <= 0 || grid > 0x7fffffff) return hipErrorInvalidValue;
  if (bwd)
    launch_kernel(bfly_kernel<true, NW>, dim3((unsigned)grid), dim3(64 * NW), s, a);
  else
    launch_kernel(bfly_kernel<false, NW>, dim3((unsigned)grid), dim3(64 * NW), s, a);
  return hipGetLastError();
}

}  // namespace

// Blocks per workgroup: one group from k = 8 on, so that the most workgroups
// run; the smaller groups are taken 8 blocks at a time (four waves).
hipError_t launch_bfly(bool bwd, const BflyArgs &a, hipStream_t s) {
  if (a.k < 2 || a.k * BB > kBflyMaxGroupCols || a.nb % a.k || a.T < 1) return hipErrorInvalidValue;
  if (a.k <= 8) return bfly_go<4>(bwd, a, s);
  if (a.k == 16) return bfly_go<8>(bwd, a, s);
  return bfly_go<16>(bwd, a, s);
}

}  // namespace pf

// Weight-gradient product on 128 x 128 tiles, bf16 (any block size):
//   dW = dY^T X on the kept blocks, dU = dY^T T_lr, dV = S^T X
// reduced over the tokens, or over one of several token splits whose fp32
// partials tn_reduce_kernel (gemm_kernels.hip) adds in split order.
//
// Operands go global -> LDS directly in 32-token steps, four stages (three
// steps in flight), each stage a separate LDS object, and the loop has no
// branch around a copy or a wait (as the 256 x 256 kernel of gemm_tnw.hip);
// 64 KiB of stages leave room for two workgroups per CU.  The loop is bound by
// the operand lines (64 flop per staged byte), so it is the copies in flight
// that count: through registers (four stages of 64 tokens, one LDS write and
// a barrier per step) the same tiles took 64 and 60 us where this takes 50
// and 50 (8192 tokens, 4096 x 1024 and 1024 x 4096, b = 64), 21.9 where this
// takes 18.9 (4096 tokens, 3072 x 768, b = 32).
//
// Orientation as in gemm_tnw.hip: the MFMA takes the X-side fragment first,
// so a lane holds 4 consecutive columns of one row of dW (dU, dV).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "pf_dma.h"
#include "pf_launch.h"

namespace pf {
namespace {

constexpr int kDT = 128;         // tile side
constexpr int kDK = 32;          // tokens per step
constexpr int kDNS = 4;          // pipeline stages
constexpr int kDOp = kDK * 256;  // bytes of one operand in a stage
constexpr int kDDma = 2 * (kDOp / 1024) / 4;  // copies per wave and step

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  return (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)lo) |
         ((uint32_t)__builtin_bit_cast(uint16_t, (__bf16)hi) << 16);
}
__device__ __forceinline__ float bf(uint32_t bits) { return __uint_as_float(bits << 16); }

template <int BLK>
__global__ __launch_bounds__(256, 2) void tnd_kernel(TNArgs a_arg) {
  const TNArgs a = a_arg;
  constexpr int GT = kDT / BLK, CPB = BLK / 8;  // blocks per side, 16-byte chunks per block row
  constexpr int TM = 2, TN = 2;                 // 4 waves as 2 x 2, 64 x 64 each
  static_assert(GT <= kTNMax, "item width");
  uint8_t *const lds0 = stage_buf<0, 2 * kDOp>(), *const lds1 = stage_buf<1, 2 * kDOp>();
  uint8_t *const lds2 = stage_buf<2, 2 * kDOp>(), *const lds3 = stage_buf<3, 2 * kDOp>();
  auto stage = [&](auto j) __attribute__((always_inline)) -> uint8_t * {
    constexpr int J = decltype(j)::value % kDNS;
    if constexpr (J == 0) return lds0;
    else if constexpr (J == 1) return lds1;
    else if constexpr (J == 2) return lds2;
    else return lds3;
  };

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w >> 1, wn = w & 1;
  // Work item: a kept-block item, or a tile of a dense region (dU, dV).
  const int nb0 = a.n_dense > 0 ? (a.dr[0].nb_blk + GT - 1) / GT : 0;
  const int n0 = a.n_dense > 0 ? (a.dr[0].na_blk + GT - 1) / GT * nb0 : 0;
  const int nb1 = a.n_dense > 1 ? (a.dr[1].nb_blk + GT - 1) / GT : 0;
  const int n1 = a.n_dense > 1 ? (a.dr[1].na_blk + GT - 1) / GT * nb1 : 0;
  const int items_total = a.n_items + n0 + n1;
  const int bid = xcd_remap(blockIdx.x, gridDim.x);
  const int split = bid / items_total, pos = bid % items_total;
  const int item = a.n_order > 0 ? (int)a_arg.order[pos] : pos;
  const bool sparse = item < a.n_items;
  const TNItem *const it = sparse ? a.items + item : nullptr;
  const bool r1 = item >= a.n_items + n0;
  const int dq = sparse ? 0 : item - a.n_items - (r1 ? n0 : 0), nbd = max(r1 ? nb1 : nb0, 1);
  const TNDense &d = a.dr[r1 ? 1 : 0];
  const int ag = dq / nbd, bg = dq % nbd;
  const int na = sparse ? 0 : min(GT, d.na_blk - ag * GT), nb = sparse ? 0 : min(GT, d.nb_blk - bg * GT);
  auto acol = [&](int g) __attribute__((always_inline)) -> int {
    return sparse ? ld_meta(&it->a_col[g]) : ag * GT + min(g, na - 1);
  };
  auto bcol = [&](int g) __attribute__((always_inline)) -> int {
    return sparse ? ld_meta(&it->b_col[g]) : bg * GT + min(g, nb - 1);
  };
  auto oblk = [&](int ga, int gb) __attribute__((always_inline)) -> int {
    return sparse ? ld_meta(&it->out_blk[ga * kTNMax + gb]) : (ga < na && gb < nb ? 0 : -1);
  };
  const int64_t lda = sparse ? a.lda : d.lda, ldb = sparse ? a.ldb : d.ldb;
  const int64_t t0 = (int64_t)split * a.chunk, t1 = min<int64_t>(a.T, t0 + a.chunk);
  const int n = t1 > t0 ? (int)((t1 - t0 + kDK - 1) / kDK) : 0;

  // Token rows past t1 read as zeros (buffer range).  Lane part of the copies:
  // row lane / 16 of a 4-row window, chunk position lane % 16, which holds the
  // global chunk XOR-swizzled by the row (see frag_kn).
  const uint32_t lda_b = (uint32_t)(lda * 2), ldb_b = (uint32_t)(ldb * 2);
  const rsrc_t rA = make_rsrc((const bf16_t *)(sparse ? a.A : d.A) + t0 * lda, (t1 - t0) * (int64_t)lda_b);
  const rsrc_t rB = make_rsrc((const bf16_t *)(sparse ? a.B : d.B) + t0 * ldb, (t1 - t0) * (int64_t)ldb_b);
  const int rr = lane >> 4, cg = (lane & 15) ^ (rr << 2);
  // (Per-lane block index: the item lists are read with vector loads here.)
  const int ga_l = cg / CPB;
  const int ca = sparse ? it->a_col[ga_l] : ag * GT + min(ga_l, na - 1);
  const int cb = sparse ? it->b_col[ga_l] : bg * GT + min(ga_l, nb - 1);
  const uint32_t inb = (uint32_t)((cg % CPB) * 16);
  const uint32_t voA = rr * lda_b + (uint32_t)(ca * BLK * 2) + inb;
  const uint32_t voB = rr * ldb_b + (uint32_t)(cb * BLK * 2) + inb;
  constexpr int WPW = kDDma / 2;
  // Steps past the end are clamped to the first row past the range.
  auto issue = [&](int t, uint8_t *st) __attribute__((always_inline)) {
    const int tt = min(t, n);
    sfor<WPW>([&](auto i) __attribute__((always_inline)) {
      const int win = w * WPW + i;
      const uint32_t row = (uint32_t)(tt * kDK + 4 * win);
      dma16(rA, st + win * 1024, voA, row * lda_b);
      dma16(rB, st + kDOp + win * 1024, voB, row * ldb_b);
    });
  };

  // Does this wave's 64 x 64 piece hold a kept block?
  bool live[TM][TN], live_w = false;
#pragma unroll
  for (int tm = 0; tm < TM; ++tm)
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
      live[tm][tn] = oblk((wm * 64 + tm * 32) / BLK, (wn * 64 + tn * 32) / BLK) >= 0;
      live_w |= live[tm][tn];
    }

  f32x16 acc[TM][TN];
  sfor<TM>([&](auto tm) __attribute__((always_inline)) {
    sfor<TN>([&](auto tn) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[tm][tn][e] = 0.f;
    });
  });
  auto compute = [&](const uint8_t *st) __attribute__((always_inline)) {
    if (!live_w) return;
    sfor<kDK / 16>([&](auto kq) __attribute__((always_inline)) {
      bf16x8 af[TM], bfr[TN];
      sfor<TM>([&](auto tm) __attribute__((always_inline)) {
        af[tm] = frag_kn<256>(st, wm * 64 + tm * 32, kq, lane);
      });
      sfor<TN>([&](auto tn) __attribute__((always_inline)) {
        bfr[tn] = frag_kn<256>(st + kDOp, wn * 64 + tn * 32, kq, lane);
      });
      sfor<TM>([&](auto tm) __attribute__((always_inline)) {
        sfor<TN>([&](auto tn) __attribute__((always_inline)) {
          acc[tm][tn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[tn], af[tm], acc[tm][tn], 0, 0, 0);
        });
      });
    });
  };

  // Steps 0 .. 2 in flight before the loop; at step t the copies of step t + 3
  // go into the stage step t - 1 read (every wave is past it after the
  // barrier).  Whole groups of four steps; steps past the end add zeros.
  sfor<kDNS - 1>([&](auto j) __attribute__((always_inline)) { issue(j, stage(j)); });
  for (int s = 0; s < n; s += kDNS) {
    sfor<kDNS>([&](auto j) __attribute__((always_inline)) {
      wait_vm<2 * kDDma>();
      barrier();
      issue(s + j + kDNS - 1, stage(std::integral_constant<int, j + kDNS - 1>{}));
      compute(stage(j));
    });
  }
  wait_vm<0>();  // no copy outlives the workgroup

  // Lane l of (tm, tn): row tm * 32 + l % 32, columns tn * 32 + q * 8 + (l / 32) * 4
  // .. + 3 in registers 4 q .. 4 q + 3.
  if (a.nsplit > 1) {
    // Partials, 16 bytes a lane: [wave][tm][tn][q][lane][4].
    float *const part = a.partials + ((int64_t)item * a.nsplit + split) * (kDT * kDT) + w * 4096 + lane * 4;
    sfor<TM>([&](auto tm) __attribute__((always_inline)) {
      sfor<TN>([&](auto tn) __attribute__((always_inline)) {
        if (!live[tm][tn]) return;
        sfor<4>([&](auto q) __attribute__((always_inline)) {
          *(f32x4 *)(part + ((tm * 2 + tn) * 4 + q) * 256) =
              f32x4{acc[tm][tn][q * 4], acc[tm][tn][q * 4 + 1], acc[tm][tn][q * 4 + 2], acc[tm][tn][q * 4 + 3]};
        });
      });
    });
    return;
  }
  const float sc = sparse ? a.scale_w : a.scale_lr;
  float wd = 0.f;  // mixing weight: sum of (unscaled sum) x W over stored kept elements
  sfor<TM>([&](auto tm) __attribute__((always_inline)) {
    sfor<TN>([&](auto tn) __attribute__((always_inline)) {
      const int R = wm * 64 + tm * 32, C = wn * 64 + tn * 32, ga = R / BLK, gb = C / BLK;
      const int blk = oblk(ga, gb);
      if (blk < 0) return;
      const int rl = R % BLK + (lane & 31), cl = C % BLK + (lane >> 5) * 4;
      const int64_t po = (int64_t)blk * (BLK * BLK) + rl * BLK + cl;
      bf16_t *const dst = sparse ? (bf16_t *)a.Wout + po
                                 : (bf16_t *)d.out + ((int64_t)acol(ga) * BLK + rl) * d.ldo +
                                       (int64_t)bcol(gb) * BLK + cl;
      sfor<4>([&](auto q) __attribute__((always_inline)) {
        const f32x4 f = {acc[tm][tn][q * 4], acc[tm][tn][q * 4 + 1], acc[tm][tn][q * 4 + 2],
                         acc[tm][tn][q * 4 + 3]};
        if (a.wdot && sparse) {
          const u32x2 x = *(const u32x2 *)((const bf16_t *)a.wdot + po + q * 8);
          wd += (f[0] * bf(x[0] & 0xffffu) + f[1] * bf(x[0] >> 16)) +
                (f[2] * bf(x[1] & 0xffffu) + f[3] * bf(x[1] >> 16));
        }
        *(u32x2 *)(dst + q * 8) = u32x2{pack2(f[0] * sc, f[1] * sc), pack2(f[2] * sc, f[3] * sc)};
      });
    });
  });
  if (a.wdot) {
    // Workgroup sum in a fixed order (wave butterflies, then the waves).
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) wd += __shfl_xor(wd, o, 64);
    __shared__ float red[4];
    if (lane == 0) red[w] = wd;
    __syncthreads();
    if (tid == 0) a.wdot_out[item] = ((red[0] + red[1]) + red[2]) + red[3];
  }
}

}  // namespace

hipError_t launch_tnd(int blk, const TNArgs &a, hipStream_t s) {
  const int64_t grid = (int64_t)tn_items_total(a, blk) * a.nsplit;
  if (grid <= 0 || grid > 0x7fffffff) return hipErrorInvalidValue;
  if (blk == 32) launch_kernel(tnd_kernel<32>, dim3((unsigned)grid), dim3(256), s, a);
  else if (blk == 64) launch_kernel(tnd_kernel<64>, dim3((unsigned)grid), dim3(256), s, a);
  else if (blk == 128) launch_kernel(tnd_kernel<128>, dim3((unsigned)grid), dim3(256), s, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace pf

// Exact (erf) GELU and its derivative for kernels with bf16 outputs.
#pragma once

#include <hip/hip_runtime.h>

namespace pf {
namespace {

// Standard normal CDF: Phi(x) = 1 - tail for x >= 0 and tail for x < 0, with
//   tail = erfc(|x| / sqrt 2) / 2 = t P(t) exp(-x^2 / 2), t = 1 / (1 + p |x| / sqrt 2),
// P a degree-8 minimax fit (relative error 7e-9, iteratively reweighted
// least squares over |x| / sqrt 2 in [0, 8], p = 0.371) of erfcx(z) / (2 t).
// One reciprocal, one exponential and about fifteen other VALU instructions,
// where the library erff takes some fifty on both sides of its branch: the
// GELU epilogues of the 8192 x 1024 -> 4096 layer were bound by them (forward
// 87 -> 72 us, backward-data 101 -> 80 us).  fp32 error of gelu over
// |x| <= 3, 2-norm: 3.3e-8 (erff: 3.6e-8); the negative tail keeps its
// relative accuracy (2e-7, where 1 + erf cancels).  e: exp(-x^2 / 2).
__device__ __forceinline__ float normal_cdf(float x, float &e) {
  const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(fabsf(x), 0.262336612f, 1.0f));
  float q = 0.0319899283f;
  q = __builtin_fmaf(q, t, -0.155200198f);
  q = __builtin_fmaf(q, t, 0.248538524f);
  q = __builtin_fmaf(q, t, -0.149138957f);
  q = __builtin_fmaf(q, t, 0.160115287f);
  q = __builtin_fmaf(q, t, 0.0511091352f);
  q = __builtin_fmaf(q, t, 0.103993565f);
  q = __builtin_fmaf(q, t, 0.103897266f);
  q = __builtin_fmaf(q, t, 0.104695439f);
  e = __builtin_amdgcn_exp2f(x * x * -0.72134752f);
  const float tail = t * q * e;
  return x < 0.f ? tail : 1.0f - tail;
}
__device__ __forceinline__ float gelu_fast(float x) {
  float e;
  return x * normal_cdf(x, e);
}
__device__ __forceinline__ float gelu_grad_fast(float x) {
  float e;
  const float cdf = normal_cdf(x, e);
  return __builtin_fmaf(x * 0.39894228040143268f, e, cdf);
}

}  // namespace
}  // namespace pf

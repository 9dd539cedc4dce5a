// Exact (erf) GELU and its derivative for kernels with bf16 outputs.
#pragma once

#include <hip/hip_runtime.h>

namespace pf {
namespace {

// Standard normal CDF.  Near zero (|x| < 1.25) Phi(x) = 1/2 + x P(x^2), P of
// degree 5 (a minimax fit of erf, 2e-9 absolute).  Beyond, the form of
// Hastings (Abramowitz and Stegun 7.1.26): Phi(x) = 1 - tail for x > 0 and tail
// for x < 0, with
//   tail = erfc(|x| / sqrt 2) / 2 = t Q(t) exp(-x^2 / 2), t = 1 / (1 + p |x| / sqrt 2),
// Q of degree 5 to erfcx(z) / (2 t), p = 0.45 (fitted here over |x| in [1.25,
// 10]: within 5e-9 absolute and 4e-7 relative).
// One reciprocal, one exponential and about twenty other VALU instructions
// without a branch, where the library erff takes some fifty on both sides of
// its own (both GELU launches of the 8192-token 1024 - 4096 MLP step).  The tail
// form alone (degree 8, four instructions fewer, that step 397.5 us against
// 405.4) is no substitute near zero: the rounding of t enlarged threefold makes it
// 2.1e-7 off there.  Errors on the device, tail form alone / this / erff:
//   CDF, largest, |x| <= 6                  2.0e-7 / 6.1e-8 / 7.5e-8
//   gelu, 2-norm, |x| <= 0.5                9.0e-8 / 3.8e-8 / 4.0e-8
//   gelu, 2-norm, x from N(0, 1)            3.9e-8 / 3.4e-8 / 3.9e-8
//   derivative, 2-norm, x from N(0, 1)      6.4e-8 / 3.8e-8 / 4.0e-8
// The negative tail keeps a relative accuracy where 1 + erf cancels: 7e-7 for x in
// -3 .. -1.25, then growing with the rounding of x^2 to 3e-6 at -8; 2e-5 at -13.
// e: exp(-x^2 / 2).
__device__ __forceinline__ float normal_cdf(float x, float &e) {
  const float u = x * x;
  float q = -6.64486106e-06f;
  q = __builtin_fmaf(q, u, 0.000110327463f);
  q = __builtin_fmaf(q, u, -0.00118270959f);
  q = __builtin_fmaf(q, u, 0.00997150037f);
  q = __builtin_fmaf(q, u, -0.0664899871f);
  q = __builtin_fmaf(q, u, 0.398942262f);
  const float near = __builtin_fmaf(x, q, 0.5f);
  const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(fabsf(x), 0.318198055f, 1.0f));
  q = -0.0769115612f;
  q = __builtin_fmaf(q, t, 0.168941066f);
  q = __builtin_fmaf(q, t, 0.0227707624f);
  q = __builtin_fmaf(q, t, 0.134163529f);
  q = __builtin_fmaf(q, t, 0.123758964f);
  q = __builtin_fmaf(q, t, 0.127148032f);
  e = __builtin_amdgcn_exp2f(u * -0.72134752f);
  const float tail = t * q * e;
  const float far = x < 0.f ? tail : 1.0f - tail;
  return fabsf(x) < 1.25f ? near : far;
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

// Exact GELU, v * Phi(v), for the bf16 kernels' epilogues.
#pragma once

#include <hip/hip_runtime.h>

namespace dycl {
namespace k {

// Phi(-|v|) = erfc(z) / 2 with z = |v| / sqrt(2), t = 1 / (1 + z / 2) and u =
// 1 - t = (z / 2) t in [0, 1):  erfc(z) = t exp(-z^2) (erfcx(z) / t), and
// log2(erfcx(z) / t) = u S(u) with S a polynomial of degree 7 (Chebyshev
// interpolation on z <= 10, beyond which exp(-z^2) is below 1e-43).  One
// reciprocal, one exponential and 8 fused multiply-adds, no branch; erff takes
// both of its branches in every wave, several times that.  Against 64 bits over
// |v| <= 12, these operations rounded to 32 bits: largest error 3.8e-7, root mean
// square 5.0e-8 (0.5 v (1 + erf), rounded alike: 4.5e-7 and 5.6e-8), relative 3e-6
// for |v| <= 6, 5e-6 for 9 and 9e-6 for 12, from the rounding of an exponent of up
// to 104 (that form: 5e-2 for 5, and no digit left at -6).  4096 x 1024 outputs of a 2048-long
// contraction: 29.4 -> 26 us.
__device__ __forceinline__ float gelu_f32(float v) {
  const float h = fminf(fabsf(v) * 0.35355339059327376f, 10.0f);   // z / 2
  const float t = __builtin_amdgcn_rcpf(1.0f + h);
  const float u = h * t;
  float s = 0.17395517230033875f;
  s = fmaf(s, u, -0.30288174748420715f);
  s = fmaf(s, u, -0.04480735585093498f);
  s = fmaf(s, u, 0.09478182345628738f);
  s = fmaf(s, u, 0.2703500986099243f);
  s = fmaf(s, u, 0.23424099385738373f);
  s = fmaf(s, u, -0.43754667043685913f);
  s = fmaf(s, u, -1.8131184577941895f);
  // log2(exp(-z^2)) = -v^2 log2(e) / 2
  const float e = 0.5f * t * __builtin_amdgcn_exp2f(fmaf(s, u, -0.72134752044448170f * v * v));
  return v * (v > 0.0f ? 1.0f - e : e);
}

}  // namespace k
}  // namespace dycl

// Element arithmetic shared by the surrogate's kernels: the matrix-core operand
// types, the rounding to BF16, and the GELU with its derivative.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace sugg {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ __bf16 to_bf16(float x) { return (__bf16)x; }

// erf by Abramowitz and Stegun, Handbook of Mathematical Functions, formula
// 7.1.26: erf(a) = 1 - t (a1 + t (a2 + t (a3 + t (a4 + t a5)))) e^(-a^2) with
// t = 1 / (1 + p a) for a >= 0 (odd extension below 0), absolute error at
// most 1.5e-7 in exact arithmetic; in FP32 (hardware reciprocal and
// exponential) a few units of 1e-7 more, far below the BF16 rounding of
// every output it feeds.  Two transcendental and six fused operations in
// place of the library's erff.
__device__ __forceinline__ float erf_as(float x) {
  const float a = fabsf(x);
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, a, 1.0f));
  const float poly =
      t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, 1.061405429f, -1.453152027f), 1.421413741f), -0.284496736f), 0.254829592f);
  return copysignf(1.0f - poly * __expf(-a * a), x);
}
__device__ __forceinline__ float gelu_f(float x) { return 0.5f * x * (1.0f + erf_as(x * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float x) {
  return 0.5f * (1.0f + erf_as(x * 0.70710678118654752f)) + x * 0.39894228040143268f * __expf(-0.5f * x * x);
}

}  // namespace sugg

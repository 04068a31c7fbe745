// The ungated activations, shared by the activation kernels (nn.hip) and the projections that apply one to what they store.
#pragma once
#include <hip/hip_runtime.h>

#include "twist.h"

namespace {

// GELU in its tanh form, 0.5 u (1 + tanh y), y = k0 (u + k1 u^3).  FINE (fp32 values): as it stands.  Values that are rounded to bf16 (2^-9):
// u / (1 + e^-2y) on the hardware's exponential and reciprocal; seven instructions instead of the library tanh's thirty, which bound the
// kernels (8192 x 768, us: forward 8.3 -> 6.1, backward 8.7 -> 5.2).  Error before that rounding, relative, the library form in brackets:
//   value     u > -2: 3e-7 (9e-7)   [-4, -2]: 7e-7 (1.2e-3, from 1 + tanh y)   [-6, -4]: 2e-6 (all of it)   [-8, -6]: 4e-6   -10: 1e-5, the
//             rounding of an exponent that grows like u^3
//   gradient  as the value for u < -2; |u| < 2: 3e-7 (3e-7) but at its zero near -0.75; [2, 4]: 1.1e-6 (5e-7), [4, 8]: 1.9e-6 (1.2e-6), from 1 - s.
//             Stored products with all 128 mantissas of da, u in [0.5, 8): at most 2e-7 beyond a rounding to nearest (4e-7)
// (evaluated in fp32 arithmetic with exact exponentials and quotients; the instructions add an ulp each).
__device__ __forceinline__ float gelu_gate(float u) {  // 1 / (1 + e^-2y)
  constexpr float k1 = 0.044715f, l2 = -2.302208198f;  // l2 = -2 k0 log2(e)
  return __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(u * fmaf(l2 * k1, u * u, l2)));
}
template <bool FINE>
__device__ __forceinline__ float gelu_tanh(float u) {
  if (!FINE) return u * gelu_gate(u);
  const float k0 = 0.7978845608028654f, k1 = 0.044715f;
  return 0.5f * u * (1.f + tanhf(k0 * (u + k1 * u * u * u)));
}
template <bool FINE>
__device__ __forceinline__ float gelu_tanh_grad(float u) {
  const float k0 = 0.7978845608028654f, k1 = 0.044715f;
  if (!FINE) {
    const float s = gelu_gate(u);
    return fmaf(u * s * (1.f - s), 2.f * k0 * fmaf(3.f * k1, u * u, 1.f), s);
  }
  const float t = tanhf(k0 * (u + k1 * u * u * u));
  return 0.5f * (1.f + t) + 0.5f * u * (1.f - t * t) * k0 * (1.f + 3.f * k1 * u * u);
}
// f(u) of an ungated activation
template <bool FINE>
__device__ __forceinline__ float act_value(int act, float u) { return act == TWIST_ACT_RELU ? fmaxf(u, 0.f) : gelu_tanh<FINE>(u); }

}  // namespace

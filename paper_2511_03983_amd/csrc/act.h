// The ungated activations, shared by the activation kernels (nn.hip) and the projections that apply one to what they store.
#pragma once
#include <hip/hip_runtime.h>

#include "twist.h"

namespace {

// GELU in its tanh form, 0.5 u (1 + tanh y), y = k0 (u + k1 u^3).  FINE (fp32 values): as it stands.  Values that are rounded to bf16:
// u / (1 + e^-2y) on the hardware's exponential and reciprocal, 1e-6 of the result and without the cancellation of 1 + tanh y where u is
// negative; seven instructions instead of the library tanh's thirty, which bound the kernels (8192 x 768, us: forward 8.3 -> 6.1,
// backward 8.7 -> 5.2).
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

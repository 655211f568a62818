// GeLU and its derivative, for the element-wise kernels and the epilogues that apply them to a product's results.
#pragma once
#include <math.h>

#include "common.h"

namespace tmk {

__device__ __forceinline__ float gelu_tanh_f(float u) {
  const float k = 0.7978845608028654f;  // sqrt(2/pi)
  return 0.5f * u * (1.f + tanhf(k * (u + 0.044715f * u * u * u)));
}
__device__ __forceinline__ float gelu_tanh_grad_f(float u) {
  const float k = 0.7978845608028654f;
  const float th = tanhf(k * (u + 0.044715f * u * u * u));
  return 0.5f * (1.f + th) + 0.5f * u * (1.f - th * th) * k * (1.f + 0.134145f * u * u);
}
__device__ __forceinline__ float gelu_erf_f(float u) { return 0.5f * u * (1.f + erff(u * 0.7071067811865476f)); }
__device__ __forceinline__ float gelu_erf_grad_f(float u) {
  const float pdf = 0.3989422804014327f * expf(-0.5f * u * u);
  return 0.5f * (1.f + erff(u * 0.7071067811865476f)) + u * pdf;
}
__device__ __forceinline__ float gelu_f(int act, float u) { return act == TM_ACT_GELU_TANH ? gelu_tanh_f(u) : gelu_erf_f(u); }
__device__ __forceinline__ float gelu_grad_f(int act, float u) {
  return act == TM_ACT_GELU_TANH ? gelu_tanh_grad_f(u) : gelu_erf_grad_f(u);
}

}  // namespace tmk

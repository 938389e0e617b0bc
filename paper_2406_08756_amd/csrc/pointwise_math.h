// Per-element arithmetic that more than one kernel must perform bit-identically: the
// stand-alone elementwise kernels and the matrix-product epilogues that absorb them.
// Floating-point contraction is off inside these functions and every fused multiply-add is written
// out, so the instruction sequence, and with it every rounding, is the same wherever
// these functions are inlined.
#pragma once
#include "device_common.h"

namespace lynx {

// tanh-form GeLU (operator 11) and its derivative.
constexpr float kGeluKappa = 0.7978845608028654f;  // sqrt(2/pi)
constexpr float kGeluC = 0.044715f;

// 1 / (1 + 2^x) from the hardware exponential and reciprocal, the latter with one Newton step: a third of the
// instructions of an IEEE division, which were half of the GeLU kernels' work.  Forward, 16384 x 2560:
// 32.6 -> 27.8 us (6.0 TB/s), 8192 x 4096: 28.5 -> 23.2; the gradient, in the store pass of the FC2 gradient
// pair, 8192 tokens, h 1024, f 4096: 178 -> 171 us for the launch.
__device__ __forceinline__ float inv_1p_exp2(float x) {
#pragma clang fp contract(off)
  const float d = fminf(1.0f + __builtin_amdgcn_exp2f(x), 3.0e38f);  // (of infinity the Newton step makes NaN)
  const float r = __builtin_amdgcn_rcpf(d);
  return __builtin_fmaf(__builtin_fmaf(-d, r, 1.0f), r, r);
}
constexpr float kLog2e = 1.4426950408889634f;
// y = kappa (u + c u^3) = u (kappa + kappa c u^2)
__device__ __forceinline__ float gelu_inner(float u) {
#pragma clang fp contract(off)
  return u * __builtin_fmaf(kGeluKappa * kGeluC, u * u, kGeluKappa);
}
// u (1 + tanh y) / 2, tanh y = 1 - 2 / (1 + e^(2y)).  Error against 64 bits as with the division (4 M
// normal deviates of deviation 0.05 to 20: 2-norm 3.4e-9 to 5.8e-8).
__device__ __forceinline__ float gelu_f(float u) {
#pragma clang fp contract(off)
  const float th = __builtin_fmaf(-2.0f, inv_1p_exp2(gelu_inner(u) * (2.0f * kLog2e)), 1.0f);
  return 0.5f * u * (1.0f + th);
}
// With sigma = (1 + tanh y) / 2 = 1 / (1 + e^(-2y)): gelu' = sigma + 2 u y' sigma (1 - sigma), in which
// nothing cancels for u < 0: error in the 2-norm 0.86 to 0.97 of the tanh form's (deviates of deviation 0.05 to 20);
// largest 0.7 of it at 0.05, 1.3 and 1.1 times at 0.5 and 1 (3.7e-7 and 1.4e-6), the same beyond.
// sigma (1 - sigma) comes first: it is 0 from |u| of about 10 on, where u y' grows with u^3 and overflows at 1e13
// (for u < 0 too: the hardware reciprocal of anything beyond 2^126, whose reciprocal is subnormal, is 0).
__device__ __forceinline__ float gelu_grad_f(float u) {
#pragma clang fp contract(off)
  const float sg = inv_1p_exp2(gelu_inner(u) * (-2.0f * kLog2e));
  const float two_dinner = __builtin_fmaf(6.0f * kGeluKappa * kGeluC, u * u, 2.0f * kGeluKappa);
  return __builtin_fmaf(u * (sg * (1.0f - sg)), two_dinner, sg);
}

// du = round(dg gelu'(u)) for 8 elements.
template <typename T>
__device__ __forceinline__ void gelu_bwd8(const float (&dg)[8], const float (&u)[8], float (&du)[8]) {
#pragma clang fp contract(off)
#pragma unroll
  for (int i = 0; i < 8; ++i) du[i] = round_to_storage(dg[i] * gelu_grad_f(u[i]), static_cast<T*>(nullptr));
}

// out = res + keep (in + bias) c for the 8 elements of dropout group `group` (operators
// 8 and 13); `in` is the storage-rounded product of the preceding linear layer.
__device__ __forceinline__ void bias_dropout_add8(const float (&in)[8], const float (&bias)[8],
                                                  const float (&res)[8], const DropoutKey& key,
                                                  uint64_t group, float (&out)[8]) {
#pragma clang fp contract(off)
  float a[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = in[i] + bias[i];
  dropout_apply8(key, group, a);
#pragma unroll
  for (int i = 0; i < 8; ++i) out[i] = res[i] + a[i];
}

}  // namespace lynx

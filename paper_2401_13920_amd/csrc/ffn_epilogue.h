// The expert FFN's epilogues, shared by its GEMM kernels.
#pragma once
#include "common.h"
#include "gelu_coef.h"

namespace locmoe {
namespace {

// GeLU for outputs that are rounded to bf16: GeLU(v) = max(v,0) - |v| Phi(-|v|), with
// 2 Phi(-x) = exp2(q(x)), q the degree-6 polynomial of gelu_coef.h on [0, 6] (argument clamped: the
// tail beyond is below 6e-9).  Relative error below 5e-5, absolute below 7e-6: forty times finer than
// the bf16 rounding that follows, at 10 vector ops and one transcendental per value (a rational erfc
// form with the same tail behaviour costs 15 and two; the epilogue's vector work was a tenth of the
// first GEMM's time with it).
// max(v,0) is formed as (v + |v|)/2 so that a NaN input stays a NaN.
__device__ __forceinline__ float gelu_bf16(float v) {
  const float x = fminf(fabsf(v), kGeluXMax);
  float q = kGeluCoef[kGeluDegree];
#pragma unroll
  for (int k = kGeluDegree - 1; k >= 0; --k) q = fmaf(q, x, kGeluCoef[k]);
  return 0.5f * fmaf(-x, __builtin_amdgcn_exp2f(q), v + fabsf(v));
}

// GeLU'(v) = Phi(v) + v phi(v) for factors of outputs that are rounded to bf16, from the same polynomial:
// Phi(-|v|) = exp2(q(|v|)) / 2 (absolute error below 2.3e-5), phi(v) = exp2(-v^2 log2(e)/2) / sqrt(2 pi).
__device__ __forceinline__ float gelu_grad_bf16(float v) {
  const float x = fminf(fabsf(v), kGeluXMax);
  float q = kGeluCoef[kGeluDegree];
#pragma unroll
  for (int k = kGeluDegree - 1; k >= 0; --k) q = fmaf(q, x, kGeluCoef[k]);
  const float tail = 0.5f * __builtin_amdgcn_exp2f(q);  // Phi(-|v|)
  const float Phi = v >= 0.f ? 1.0f - tail : tail;
  const float phi = 0.3989422804f * __builtin_amdgcn_exp2f(-0.7213475204f * v * v);
  return fmaf(v, phi, Phi);
}

// What happens to an accumulator on its way to memory
constexpr int kEpiNone = 0;      // rounded and stored
constexpr int kEpiGelu = 1;      // GeLU, then rounded and stored (H of Eq. 1)
constexpr int kEpiGeluSave = 2;  // the same, and the pre-activation Z is stored (bf16) to `aux` for the backward
constexpr int kEpiGeluGrad = 3;  // multiplied by GeLU'(Z), Z read from `aux` (bf16): dZ = dH * GeLU'(Z)

// One accumulator quad -> memory.  q holds D[n0..n0+3][m] for one row m.
template <int EPI, bool OUT_F32>
__device__ __forceinline__ void store_quad(void* C, uint16_t* aux, size_t row, int ldc, int n0, float q0, float q1,
                                           float q2, float q3) {
  static_assert(!(EPI != kEpiNone && OUT_F32), "the hidden activations and their gradients are stored as bf16");
  if (EPI == kEpiGeluSave) *(uint2*)(aux + row * ldc + n0) = make_uint2(pack_bf16x2(q0, q1), pack_bf16x2(q2, q3));
  if (EPI == kEpiGelu || EPI == kEpiGeluSave) {
    q0 = gelu_bf16(q0); q1 = gelu_bf16(q1); q2 = gelu_bf16(q2); q3 = gelu_bf16(q3);
  }
  if (EPI == kEpiGeluGrad) {
    const uint2 z = *(const uint2*)(aux + row * ldc + n0);
    q0 *= gelu_grad_bf16(bf16_bits_to_f32(z.x & 0xFFFFu));
    q1 *= gelu_grad_bf16(__uint_as_float(z.x & 0xFFFF0000u));
    q2 *= gelu_grad_bf16(bf16_bits_to_f32(z.y & 0xFFFFu));
    q3 *= gelu_grad_bf16(__uint_as_float(z.y & 0xFFFF0000u));
  }
  if (OUT_F32) {
    *(float4*)((float*)C + row * ldc + n0) = make_float4(q0, q1, q2, q3);
  } else {
    *(uint2*)((uint16_t*)C + row * ldc + n0) = make_uint2(pack_bf16x2(q0, q1), pack_bf16x2(q2, q3));
  }
}

}  // namespace
}  // namespace locmoe

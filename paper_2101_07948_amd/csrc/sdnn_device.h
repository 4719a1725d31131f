// Device code shared by the kernels: the fused epilogue and the stores of C.
#ifndef SDNN_DEVICE_H_
#define SDNN_DEVICE_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/sdnn.h"

namespace sdnn {
namespace {

// GELU(x) = x Phi(x) = 0.5 x (1 + erf(x / sqrt 2)) (the exact erf form).  erf(z) for
// z >= 0 comes from Abramowitz & Stegun 7.1.26 (Hastings' approximation, absolute error
// at most 1.5e-7): erf(z) = 1 - q, q = t (a1 + t (a2 + t (a3 + t (a4 + t a5)))) e^(-z^2),
// t = 1 / (1 + p z); with erf(-z) = -erf(z), GELU(x) = 0.5 x (2 - q) for x >= 0 and
// 0.5 x q for x < 0 (no cancellation on the negative side).  The reciprocal and the
// exponential are the hardware's (v_rcp_f32, v_exp_f32, about 1 ulp); the result is within
// 0.5 |x| * 4e-7 of the exact GELU, far inside the 1e-6 floor of the parity bar at the
// |x| these layers reach, and costs about a third of the library erff's instructions.
__device__ __forceinline__ float gelu(float x) {
  const float z = fabsf(x) * 0.70710678118654752f;
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, z, 1.0f));
  float poly = fmaf(t, 1.061405429f, -1.453152027f);
  poly = fmaf(t, poly, 1.421413741f);
  poly = fmaf(t, poly, -0.284496736f);
  poly = fmaf(t, poly, 0.254829592f);
  poly *= t;
  const float q = poly * __builtin_amdgcn_exp2f(-z * z * 1.4426950408889634f);
  return 0.5f * x * (x >= 0.0f ? 2.0f - q : q);
}

// C is written once and not read again by the kernel: its stores are non-temporal, so the
// output stream does not evict the B tiles and the packed stream from L2 (the stores of the
// 201 MB output of the 3072 x 768 layer at N = 16384 otherwise push the 0.57 MB stream out
// between tiles).
typedef float nt_float4 __attribute__((ext_vector_type(4)));
typedef float nt_float2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void store_c4(float* p, float x, float y, float z, float w) {
  const nt_float4 v = {x, y, z, w};
  __builtin_nontemporal_store(v, reinterpret_cast<nt_float4*>(p));
}
__device__ __forceinline__ void store_c2(float* p, float x, float y) {
  const nt_float2 v = {x, y};
  __builtin_nontemporal_store(v, reinterpret_cast<nt_float2*>(p));
}
__device__ __forceinline__ void store_c1(float* p, float x) { __builtin_nontemporal_store(x, p); }

__device__ __forceinline__ float activation(float x, int epi) {
  if (epi == SDNN_EPI_RELU) return fmaxf(x, 0.0f);
  if (epi == SDNN_EPI_GELU) return gelu(x);
  return x;
}

}  // namespace
}  // namespace sdnn

#endif  // SDNN_DEVICE_H_

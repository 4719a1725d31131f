// Device code shared by the kernels: the fused epilogue and the stores of C.
#ifndef SDNN_DEVICE_H_
#define SDNN_DEVICE_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/sdnn.h"

namespace sdnn {
namespace {

// GELU(x) = x Phi(x) = 0.5 x (1 + erf(x / sqrt 2)) (the exact erf form).  With z = |x| / sqrt 2
// and erfc(z) = t (a1 + t (a2 + t (a3 + t (a4 + t a5)))) e^(-z^2), t = 1 / (1 + p z) (Abramowitz &
// Stegun 7.1.26, Hastings' approximation, absolute error at most 1.5e-7),
//     GELU(x) = max(x, 0) - 0.5 |x| erfc(z)
// for either sign (no cancellation: the second term is at most half the first, or alone).
// Evaluated on y = |x| sqrt(0.5 log2 e), so that e^(-z^2) = 2^(-y^2), with the factor 0.5 |x| / y
// folded into the coefficients; their last bits (and p's) were then searched on the GPU for the
// smallest error, because the rounded ones no longer sum to erfc(0) = 1.  The reciprocal and the
// exponential are the hardware's (v_rcp_f32, v_exp_f32, about 1 ulp).  Over every float of 1e-7 <=
// |x| <= 14 the result is within 0.5 |x| * 6.31e-7 of the exact GELU (6.43e-7 with the coefficients
// as printed, in the two-sided form), far inside the 1e-6 floor of the parity bar at the |x| these
// layers reach; over x distributed N(0, 0.01^2) to N(0, 5^2) the 2-norm of the error is 0.93-1.007
// of theirs, 1.05 at N(0, 0.003^2).  12 plain instructions and the two special ones, where the
// two-sided form took 18: on the 3072 x 768 layer at N = 16384 the GELU of 50 M outputs is a third
// of the vector instructions (107.7 -> 103.1 us).
__device__ __forceinline__ float gelu(float x) {
  // (an infinite x: its factor stays finite at +inf, whose q is 0, and gives NaN at -inf)
  const float y = fabsf(__builtin_elementwise_minimum(x, 3.0e38f)) * 0.849321783f;
  const float e = __builtin_amdgcn_exp2f(-(y * y));
  const float t = __builtin_amdgcn_rcpf(fmaf(y, 0.272737592f, 1.0f));
  float q = fmaf(t, 0.624854565f, -0.855477035f);
  q = fmaf(t, q, 0.836792111f);
  q = fmaf(t, q, -0.167484373f);
  q = fmaf(t, q, 0.15001978f);
  q *= t;
  q *= e;
  return fmaf(-y, q, fmaxf(x, 0.0f));
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

// What a consumer wave leaves in all of its accumulators when it went on without waiting, or
// its chunks may have been overwritten: a NaN whose payload no arithmetic makes.  Its rows are
// stored as NaN whatever the activation is (fmaxf(NaN, 0) = 0: a ReLU would otherwise turn the
// rows into plausible zeros).  The value is the same in every accumulator, so one is looked at.
constexpr uint32_t kPoison = 0x7fc0deadu;
__device__ __forceinline__ int epilogue_of(float acc, int epi) {  // of a wave
  return (uint32_t)__builtin_amdgcn_readfirstlane(__float_as_int(acc)) == kPoison ? (int)SDNN_EPI_NONE : epi;
}

}  // namespace
}  // namespace sdnn

#endif  // SDNN_DEVICE_H_

// Shared device/host helpers for the stage kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace zs {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16;
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

enum DType { F32 = 0, BF16 = 1, F16 = 2 };   // F16: IEEE half (the precision the paper trains in, Section 6.1)

constexpr int WAVE = 64;

__device__ __forceinline__ float to_f(float x) { return x; }
__device__ __forceinline__ float to_f(bf16 x) { return (float)x; }
__device__ __forceinline__ float to_f(f16 x) { return (float)x; }
template <typename T> __device__ __forceinline__ T from_f(float x);
template <> __device__ __forceinline__ float from_f<float>(float x) { return x; }
template <> __device__ __forceinline__ bf16 from_f<bf16>(float x) { return (bf16)x; }  // round-to-nearest-even
template <> __device__ __forceinline__ f16 from_f<f16>(float x) { return (f16)x; }     // round-to-nearest-even, overflow to inf

// Between LDS writes of a wave and reads of what other lanes of it wrote, and between those reads and the next writes there.  The hardware
// keeps a wave's LDS accesses in order; the compiler sees one lane, whose own addresses it may find distinct and its accesses free to move.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// x as an fp32 value of its own: without this the compiler may fold the multiply-add that gives x and the rounding to half that follows into
// one instruction (v_fma_mixlo_f16), which rounds once, and does or does not with the code around.
__device__ __forceinline__ float fp32_value(float x) {
  asm("" : "+v"(x));
  return x;
}

// Elements moved per 16-byte access.
template <typename T> struct Vec;
template <> struct Vec<float> { static constexpr int N = 4; typedef f32x4 type; };
template <> struct Vec<bf16> { static constexpr int N = 8; typedef bf16x8 type; };
template <> struct Vec<f16> { static constexpr int N = 8; typedef f16x8 type; };

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// Sum over a workgroup of NW waves; every thread gets the result.  red must hold NW floats.
template <int NW> __device__ __forceinline__ float block_sum(float v, float* red) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  __syncthreads();
  if (l == 0) red[w] = v;
  __syncthreads();
  float t = 0.f;
#pragma unroll
  for (int i = 0; i < NW; ++i) t += red[i];
  return t;
}

// GELU(z) = z Phi(z) with Phi the normal distribution function (the erf form) and its derivative Phi(z) + z phi(z).
// erf comes from the rational approximation 7.1.26 of Abramowitz and Stegun, |error| <= 1.5e-7, i.e. fp32 rounding level:
// erf(x) = 1 - (a1 t + ... + a5 t^5) exp(-x^2), t = 1 / (1 + p x), x >= 0.  With x = |z| / sqrt(2) its exponential is
// exp(-z^2 / 2), the one the density phi needs as well, so value and derivative cost one hardware exp2 and one hardware
// reciprocal instead of erff and expf (these kernels were bound by that arithmetic, not by memory).
__device__ __forceinline__ void gelu_parts(float z, float& Phi, float& phi) {
  const float x = fabsf(z) * 0.70710678118654752f;
  const float e = __builtin_amdgcn_exp2f(-1.4426950408889634f * x * x);
  const float t = __builtin_amdgcn_rcpf(1.0f + 0.3275911f * x);
  const float poly = t * (0.254829592f + t * (-0.284496736f + t * (1.421413741f + t * (-1.453152027f + t * 1.061405429f))));
  Phi = 0.5f * (1.0f + copysignf(1.0f - poly * e, z));
  phi = 0.39894228040143268f * e;
}
__device__ __forceinline__ float gelu_f(float z) {
  float Phi, phi;
  gelu_parts(z, Phi, phi);
  return z * Phi;
}
__device__ __forceinline__ float gelu_df(float z) {
  float Phi, phi;
  gelu_parts(z, Phi, phi);
  return Phi + z * phi;
}

// Gated FFN unit of the Llama-style layer: a = silu(gate) * up, and (dgate, dup) from da.  One definition, so that
// the stand-alone kernels and the GEMM epilogues that fuse them produce the same bits.
// exp through the hardware's exp2 and a hardware reciprocal (each good to about one fp32 ulp, far below the 16-bit
// rounding of whatever is stored): a fifth of the instructions of expf and an IEEE division, which matters where this runs
// 65 536 times in the store phase of a GEMM tile with the matrix cores waiting.
__device__ __forceinline__ float sigmoid_f(float z) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * z));
}
__device__ __forceinline__ float glu_f(float g, float u) { return g * sigmoid_f(g) * u; }
__device__ __forceinline__ void glu_df(float d, float g, float u, float& dg, float& du) {
  const float s = sigmoid_f(g);
  du = d * g * s;
  dg = d * u * s * (1.0f + g * (1.0f - s));
}

static inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

}  // namespace zs

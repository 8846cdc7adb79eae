// Causal softmax attention, forward and backward, one wavefront per query (or key) row, fp32
// arithmetic, no atomics.  This is the path of head sizes above 128 and of unaligned rows, which the matrix-core
// kernels do not take; it never materialises the S x S matrix (online softmax over tiles of
// 64 keys) but makes no attempt to reuse K/V across rows.
#include "kernels.h"
#include "attention_rows.h"

namespace zs {

constexpr int MAXD = 256;  // head dim limit of this kernel

// grid (ceil(S/4), nh, mb), 256 threads: wave w handles query row blockIdx.x*4+w.
template <typename T>
__global__ __launch_bounds__(256) void attn_fwd_simple(int S, int d, const T* __restrict__ q, const T* __restrict__ k,
                                                       const T* __restrict__ v, int64_t ld, T* __restrict__ o,
                                                       int64_t ldo, float* __restrict__ lse, float scale) {
  __shared__ float qs[4][MAXD];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + w;
  const int h = blockIdx.y, b = blockIdx.z, nh = gridDim.y;
  if (i >= S) return;                       // whole wave leaves together; no block barrier below
  const int64_t tok0 = (int64_t)b * S, at = tok0 * ld + h * d;
  T* oi = o + (tok0 + i) * ldo + h * d;
  const float l = attn_fwd_row<MAXD / 64>(qs[w], i, d, q + at, k + at, v + at, ld, scale, lane, [&](int c, float x) { oi[c] = from_f<T>(x); });
  if (lane == 0) lse[((int64_t)b * nh + h) * S + i] = l;
}

// delta[b,h,i] = sum_c do[i,c] * o[i,c]
template <typename T>
__global__ __launch_bounds__(256) void attn_delta_kernel(int S, int d, const T* __restrict__ o, const T* __restrict__ dout,
                                                         int64_t ldo, float* __restrict__ delta) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + w;
  const int h = blockIdx.y, b = blockIdx.z, nh = gridDim.y;
  if (i >= S) return;
  const int64_t off = ((int64_t)b * S + i) * ldo + h * d;
  float s = 0.f;
  for (int c = lane; c < d; c += 64) s += to_f(o[off + c]) * to_f(dout[off + c]);
  s = wave_sum(s);
  if (lane == 0) delta[((int64_t)b * nh + h) * S + i] = s;
}

template <typename T>
__global__ __launch_bounds__(256) void attn_bwd_dq_simple(int S, int d, const T* __restrict__ q, const T* __restrict__ k,
                                                          const T* __restrict__ v, int64_t ld,
                                                          const T* __restrict__ dout, int64_t ldo,
                                                          const float* __restrict__ lse, const float* __restrict__ delta,
                                                          T* __restrict__ dq, int64_t ldd, float scale) {
  __shared__ float rows[4][2 * MAXD];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + w;
  const int h = blockIdx.y, b = blockIdx.z, nh = gridDim.y;
  if (i >= S) return;
  const int64_t tok0 = (int64_t)b * S, at = tok0 * ld + h * d, stat = ((int64_t)b * nh + h) * S + i;
  T* dqi = dq + (tok0 + i) * ldd + h * d;
  attn_dq_row<MAXD / 64>(rows[w], i, d, q + at, k + at, v + at, ld, dout + tok0 * ldo + h * d, ldo, lse[stat], delta[stat], scale, lane,
                         [&](int c, float x) { dqi[c] = from_f<T>(x); });
}

template <typename T>
__global__ __launch_bounds__(256) void attn_bwd_dkv_simple(int S, int d, const T* __restrict__ q, const T* __restrict__ k,
                                                           const T* __restrict__ v, int64_t ld,
                                                           const T* __restrict__ dout, int64_t ldo,
                                                           const float* __restrict__ lse, const float* __restrict__ delta,
                                                           T* __restrict__ dk, T* __restrict__ dv, int64_t ldd, float scale) {
  __shared__ float rows[4][2 * MAXD];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int j = blockIdx.x * 4 + w;
  const int h = blockIdx.y, b = blockIdx.z, nh = gridDim.y;
  if (j >= S) return;
  const int64_t tok0 = (int64_t)b * S, at = tok0 * ld + h * d, stat = ((int64_t)b * nh + h) * S, to = (tok0 + j) * ldd + h * d;
  attn_dkv_row<MAXD / 64>(rows[w], j, S, d, q + at, k + at, v + at, ld, dout + tok0 * ldo + h * d, ldo, lse + stat, [&](int i) { return delta[stat + i]; }, scale,
                          lane, [&](int c, float xk, float xv) { dk[to + c] = from_f<T>(xk); dv[to + c] = from_f<T>(xv); });
}

template <typename T>
static hipError_t fwd_simple(hipStream_t st, int mb, int S, int nh, int d, const void* q, const void* k, const void* v,
                             int64_t ld, void* o, int64_t ldo, float* lse) {
  dim3 grid((unsigned)cdiv(S, 4), (unsigned)nh, (unsigned)mb), blk(256);
  hipLaunchKernelGGL(attn_fwd_simple<T>, grid, blk, 0, st, S, d, (const T*)q, (const T*)k, (const T*)v, ld, (T*)o, ldo,
                     lse, 1.0f / sqrtf((float)d));
  return hipGetLastError();
}
template <typename T>
static hipError_t bwd_simple(hipStream_t st, int mb, int S, int nh, int d, const void* q, const void* k, const void* v,
                             int64_t ld, const void* o, const void* dout, int64_t ldo, const float* lse, float* delta,
                             void* dq, void* dk, void* dv, int64_t ldd) {
  dim3 grid((unsigned)cdiv(S, 4), (unsigned)nh, (unsigned)mb), blk(256);
  const float scale = 1.0f / sqrtf((float)d);
  hipLaunchKernelGGL(attn_delta_kernel<T>, grid, blk, 0, st, S, d, (const T*)o, (const T*)dout, ldo, delta);
  hipLaunchKernelGGL(attn_bwd_dq_simple<T>, grid, blk, 0, st, S, d, (const T*)q, (const T*)k, (const T*)v, ld,
                     (const T*)dout, ldo, lse, delta, (T*)dq, ldd, scale);
  hipLaunchKernelGGL(attn_bwd_dkv_simple<T>, grid, blk, 0, st, S, d, (const T*)q, (const T*)k, (const T*)v, ld,
                     (const T*)dout, ldo, lse, delta, (T*)dk, (T*)dv, ldd, scale);
  return hipGetLastError();
}

typedef hipError_t AttnFwd(hipStream_t st, int mb, int S, int nh, int d, const void* q, const void* k, const void* v, int64_t ld, void* o,
                           int64_t ldo, float* lse);
typedef hipError_t AttnBwd(hipStream_t st, int mb, int S, int nh, int d, const void* q, const void* k, const void* v, int64_t ld,
                           const void* o, const void* dout, int64_t ldo, const float* lse, float* delta, void* dq, void* dk, void* dv,
                           int64_t ldd, const float2* rope);
AttnFwd attn_fwd_mfma, attn_fwd_mfma_f16, attn_fwd_split, attn_fwd_split_f16, attn_fwd_f32;
AttnBwd attn_bwd_mfma, attn_bwd_mfma_f16, attn_bwd_split, attn_bwd_split_f16, attn_bwd_f32;
bool attn_mfma_supported(DType dt, int S, int d);
bool attn_f32_supported(int mb, int S, int nh, int d, int64_t ld_max, uintptr_t pointers, int64_t strides);

int attn_select(DType dt, int S, int d, int force) {
  if (force == ATTN_SIMPLE) return ATTN_SIMPLE;
  return attn_mfma_supported(dt, S, d) ? ATTN_MFMA : ATTN_SIMPLE;
}

// Sequences so short that a wave per row is faster.  Its time grows with the keys; a matrix-core kernel takes the same for any
// number of them up to a tile, once per round of workgroups on the 256 CUs (one or two rounds up to 256 heads).  Measured at 1 to
// 2048 heads, S = 1 to 64 and d = 8 to 128 (us, wave per row : matrix cores): fp32 forward, d = 64, one head S = 4 4.9 : 6.1, S = 16
// 6.7 : 6.1; bf16 forward, 16 heads, d = 8 S = 8 5.1 : 5.2, d = 64 S = 2 4.8 : 5.4; with 2048 heads of 64 the matrix cores lose by 2.3
// to 4.3 at S = 2 and win from S = 12 on.  The half backward of d > 96, whose registers spill, takes 27 us up to S = 32 (16 heads;
// wave per row 24.7 at S = 24).  fp32 blocks hold 16 rows, so many heads pay a second round from S = 17 on.  Of 3900
// measured points 8 are left more than 10 % slower than the wave per row, by at most 27 %.  A rotation (rope) is another two
// launches after the wave per row.
static bool few_keys(DType dt, bool bwd, bool rope, int64_t heads, int d, int S) {
  const bool wide = d > 64, many = heads > 256;
  int most;
  if (dt == F32) {
    if (heads >= 256 && !rope && S > 16 && S <= (bwd ? 24 : 20) && (bwd ? d <= 32 : wide)) return true;
    most = many ? (!bwd && d > 32 && !wide ? 8 : 12) : (wide ? 16 : 20 - d / 8) - (heads >= 128 ? 5 : 0);
  } else if (!bwd) {
    most = many ? 10 : wide ? (dt == BF16 ? 4 : 5) : 11 - 3 * d / 32;
  } else if (dt == BF16) {
    most = many ? (d <= 32 ? 14 : 10) : wide ? 2 : 8 - d / 8;
  } else {
    most = d > 96 ? 24 : many ? (d <= 32 ? 14 : wide ? 16 : 12) : wide ? 10 : 12 - 5 * d / 32;
  }
  return S <= most - (rope ? (many ? 4 : 16) : 0);
}

// Heads of 128 in 16 bits always run on the matrix cores.  Narrower 16-bit heads (their fp32 probabilities split in two 16-bit
// parts) and fp32 heads do when there are more than a few keys and rows can be read in aligned 16-byte pieces through 32-bit
// offsets; else, and for wider heads, a wavefront per row.
AttnRoute attn_route(DType dt, bool bwd, bool rope, int mb, int S, int nh, int d, int64_t ld_max, uintptr_t pointers, int64_t strides, int force) {
  if (attn_select(dt, S, d, force) == ATTN_MFMA) return ATTN_ROUTE_MFMA;
  if (force == ATTN_SIMPLE || few_keys(dt, bwd, rope, mb * (int64_t)nh, d, S)) return ATTN_ROUTE_SIMPLE;
  if (dt == F32) return attn_f32_supported(mb, S, nh, d, ld_max, pointers, strides) ? ATTN_ROUTE_F32 : ATTN_ROUTE_SIMPLE;
  return d < 128 && (pointers & 15) == 0 && strides % 8 == 0 && (int64_t)S * ld_max * 2 < (1ll << 31) ? ATTN_ROUTE_SPLIT : ATTN_ROUTE_SIMPLE;
}

hipError_t attn_fwd(hipStream_t st, DType dt, int mb, int S, int nh, int d, const void* q, const void* k,
                    const void* v, int64_t ld, void* o, int64_t ldo, float* lse, int force) {
  const AttnRoute route = attn_route(dt, false, false, mb, S, nh, d, ld, (uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o, ld | ldo, force);
  if (route == ATTN_ROUTE_MFMA) return (dt == F16 ? attn_fwd_mfma_f16 : attn_fwd_mfma)(st, mb, S, nh, d, q, k, v, ld, o, ldo, lse);
  if (route == ATTN_ROUTE_SPLIT) return (dt == F16 ? attn_fwd_split_f16 : attn_fwd_split)(st, mb, S, nh, d, q, k, v, ld, o, ldo, lse);
  if (route == ATTN_ROUTE_F32) return attn_fwd_f32(st, mb, S, nh, d, q, k, v, ld, o, ldo, lse);
  return dt == F32    ? fwd_simple<float>(st, mb, S, nh, d, q, k, v, ld, o, ldo, lse)
         : dt == BF16 ? fwd_simple<bf16>(st, mb, S, nh, d, q, k, v, ld, o, ldo, lse)
                      : fwd_simple<f16>(st, mb, S, nh, d, q, k, v, ld, o, ldo, lse);
}
hipError_t attn_bwd(hipStream_t st, DType dt, int mb, int S, int nh, int d, const void* q, const void* k,
                    const void* v, int64_t ld, const void* o, const void* dout, int64_t ldo, const float* lse,
                    float* delta, void* dq, void* dk, void* dv, int64_t ldd, const float2* rope, int force) {
  const uintptr_t at = (uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o | (uintptr_t)dout | (uintptr_t)dq | (uintptr_t)dk |
                       (uintptr_t)dv | (uintptr_t)rope;
  const AttnRoute route = attn_route(dt, true, rope != nullptr, mb, S, nh, d, ld > ldo ? ld : ldo, at, ld | ldo | ldd, force);
  if (route != ATTN_ROUTE_SIMPLE) {   // rotation fused into the kernels' stores
    AttnBwd* run = route == ATTN_ROUTE_F32 ? attn_bwd_f32 : route == ATTN_ROUTE_MFMA ? (dt == F16 ? attn_bwd_mfma_f16 : attn_bwd_mfma)
                                                                                  : (dt == F16 ? attn_bwd_split_f16 : attn_bwd_split);
    return run(st, mb, S, nh, d, q, k, v, ld, o, dout, ldo, lse, delta, dq, dk, dv, ldd, rope);
  }
  hipError_t e = dt == F32    ? bwd_simple<float>(st, mb, S, nh, d, q, k, v, ld, o, dout, ldo, lse, delta, dq, dk, dv, ldd)
                 : dt == BF16 ? bwd_simple<bf16>(st, mb, S, nh, d, q, k, v, ld, o, dout, ldo, lse, delta, dq, dk, dv, ldd)
                              : bwd_simple<f16>(st, mb, S, nh, d, q, k, v, ld, o, dout, ldo, lse, delta, dq, dk, dv, ldd);
  if (e == hipSuccess && rope) e = rope_apply(st, dt, mb * S, S, nh * d, d, dq, ldd, rope, -1.0f);
  if (e == hipSuccess && rope) e = rope_apply(st, dt, mb * S, S, nh * d, d, dk, ldd, rope, -1.0f);
  return e;
}

}  // namespace zs

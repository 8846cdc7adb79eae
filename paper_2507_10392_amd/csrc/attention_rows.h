// Causal attention of ONE row by one wavefront in fp32 arithmetic, forward and backward: what the wave-per-row kernels run for
// every row, and what the matrix-core kernels fall back to for a row whose result did not come out finite (see below).
//
// A matrix instruction multiplies a whole tile: a key in the future of a query takes part with weight zero instead of being
// skipped, and 0 * inf and 0 * NaN are NaN, so one non-finite value of a token would reach rows that do not see that token.
// A product of that kind always leaves NaN in the accumulators of the row it reaches.  The kernels therefore look at their
// accumulators once, before the store, and redo the rows that hold anything non-finite here, where masked keys are not read.
// The rows of a workgroup are dealt out over its waves; rows that are NaN throughout in any case, because a row
// statistic they depend on is NaN, are left as they are.
#pragma once
#include "common.h"

namespace zs {

template <typename T> __device__ __forceinline__ float dot_row(const float* __restrict__ vec, const T* __restrict__ row, int d) {
  constexpr int V = Vec<T>::N;
  float s = 0.f;
  for (int c = 0; c < d; c += V) {
    typename Vec<T>::type r = *reinterpret_cast<const typename Vec<T>::type*>(row + c);
#pragma unroll
    for (int i = 0; i < V; ++i) s += vec[c + i] * to_f(r[i]);
  }
  return s;
}

// Query i of a head with rows q, k, v (stride ld): out(c, o[i][c]) for the columns c < d that the lane owns (c = 64 n + lane,
// d <= 64 NC); returns the row's log-sum-exp.  qs: LDS of the wave's own, 64 NC floats.
template <int NC, typename T, typename F>
__device__ __forceinline__ float attn_fwd_row(float* qs, int i, int d, const T* __restrict__ q, const T* __restrict__ k,
                                              const T* __restrict__ v, int64_t ld, float scale, int lane, F&& out) {
  for (int c = lane; c < d; c += 64) qs[c] = to_f(q[(int64_t)i * ld + c]) * scale;
  __builtin_amdgcn_wave_barrier();
  float m = -INFINITY, l = 0.f;
  float acc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) acc[c] = 0.f;
  for (int j0 = 0; j0 <= i; j0 += 64) {
    const int j = j0 + lane;
    float s = -INFINITY;
    if (j <= i) s = dot_row(qs, k + (int64_t)j * ld, d);
    const float mn = fmaxf(m, wave_max(s));
    const float p = (j <= i) ? expf(s - mn) : 0.f;
    const float alpha = expf(m - mn);
    l = l * alpha + wave_sum(p);
    m = mn;
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] *= alpha;
    const int jn = min(64, i - j0 + 1);
    for (int jj = 0; jj < jn; ++jj) {
      const float pj = __shfl(p, jj, 64);
      const T* vr = v + (int64_t)(j0 + jj) * ld;
#pragma unroll
      for (int c = 0; c < NC; ++c)
        if (c * 64 + lane < d) acc[c] += pj * to_f(vr[c * 64 + lane]);
    }
  }
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (c * 64 + lane < d) out(c * 64 + lane, acc[c] / l);
  return m + logf(l);
}

// dq_i = scale * sum_{j<=i} ds_ij k_j,  ds_ij = p_ij (do_i.v_j - delta_i),  p_ij = exp(scale q_i.k_j - lse_i), with li = lse_i and
// di = delta_i.  rows: LDS of the wave's own, 128 NC floats.
template <int NC, typename T, typename F>
__device__ __forceinline__ void attn_dq_row(float* rows, int i, int d, const T* __restrict__ q, const T* __restrict__ k,
                                            const T* __restrict__ v, int64_t ld, const T* __restrict__ dout, int64_t ldo, float li,
                                            float di, float scale, int lane, F&& out) {
  float *qs = rows, *dos = rows + 64 * NC;
  for (int c = lane; c < d; c += 64) {
    qs[c] = to_f(q[(int64_t)i * ld + c]) * scale;
    dos[c] = to_f(dout[(int64_t)i * ldo + c]);
  }
  __builtin_amdgcn_wave_barrier();
  float acc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) acc[c] = 0.f;
  for (int j0 = 0; j0 <= i; j0 += 64) {
    const int j = j0 + lane;
    float ds = 0.f;
    if (j <= i) {
      const float s = dot_row(qs, k + (int64_t)j * ld, d);
      const float dp = dot_row(dos, v + (int64_t)j * ld, d);
      ds = expf(s - li) * (dp - di);
    }
    const int jn = min(64, i - j0 + 1);
    for (int jj = 0; jj < jn; ++jj) {
      const float dsj = __shfl(ds, jj, 64);
      const T* kr = k + (int64_t)(j0 + jj) * ld;
#pragma unroll
      for (int c = 0; c < NC; ++c)
        if (c * 64 + lane < d) acc[c] += dsj * to_f(kr[c * 64 + lane]);
    }
  }
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (c * 64 + lane < d) out(c * 64 + lane, acc[c] * scale);
}

// dv_j = sum_{i>=j} p_ij do_i,  dk_j = scale * sum_{i>=j} ds_ij q_i: out(c, dk[j][c], dv[j][c]).  lse: the head's rows, delta(i): row i's.
// rows: LDS of the wave's own, 128 NC floats.
template <int NC, typename T, typename Delta, typename F>
__device__ __forceinline__ void attn_dkv_row(float* rows, int j, int S, int d, const T* __restrict__ q, const T* __restrict__ k,
                                             const T* __restrict__ v, int64_t ld, const T* __restrict__ dout, int64_t ldo,
                                             const float* __restrict__ lse, Delta&& delta, float scale, int lane,
                                             F&& out) {
  float *ks = rows, *vs = rows + 64 * NC;
  for (int c = lane; c < d; c += 64) {
    ks[c] = to_f(k[(int64_t)j * ld + c]) * scale;
    vs[c] = to_f(v[(int64_t)j * ld + c]);
  }
  __builtin_amdgcn_wave_barrier();
  float acck[NC], accv[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) acck[c] = accv[c] = 0.f;
  for (int i0 = j; i0 < S; i0 += 64) {
    const int i = i0 + lane;
    float p = 0.f, ds = 0.f;
    if (i < S) {
      const float s = dot_row(ks, q + (int64_t)i * ld, d);
      const float dp = dot_row(vs, dout + (int64_t)i * ldo, d);
      p = expf(s - lse[i]);
      ds = p * (dp - delta(i));
    }
    const int in = min(64, S - i0);
    for (int ii = 0; ii < in; ++ii) {
      const float pi = __shfl(p, ii, 64);
      const float dsi = __shfl(ds, ii, 64);
      const T* qr = q + (int64_t)(i0 + ii) * ld;
      const T* dor = dout + (int64_t)(i0 + ii) * ldo;
#pragma unroll
      for (int c = 0; c < NC; ++c)
        if (c * 64 + lane < d) {
          accv[c] += pi * to_f(dor[c * 64 + lane]);
          acck[c] += dsi * to_f(qr[c * 64 + lane]);
        }
    }
  }
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (c * 64 + lane < d) out(c * 64 + lane, acck[c] * scale, accv[c]);
}

// True when key j has NaN in every column of dk and dv because a query that sees it has a log-sum-exp of NaN.
__device__ __forceinline__ bool dkv_row_is_nan(int j, int S, const float* __restrict__ lse, int lane) {
  bool nan = false;
  for (int i = j + lane; i < S; i += 64) nan |= lse[i] != lse[i];
  return __any(nan);
}

// Whether any of masks[0 .. groups-1] in LDS has a bit: one read, where the words one after the other are as many LDS latencies.
__device__ __forceinline__ bool any_row(const unsigned* masks, int groups, int lane) { return __any(masks[min(lane, groups - 1)] != 0); }
// Calls f(group, bit) for the set bits of masks[0 .. groups-1], dealt out over `waves` waves.
template <typename F> __device__ __forceinline__ void for_dealt_rows(const unsigned* masks, int groups, int waves, int wave, F&& f) {
  int n = 0;
  for (int g = 0; g < groups; ++g)
    for (unsigned m = __builtin_amdgcn_readfirstlane(masks[g]); m; m &= m - 1)
      if (n++ % waves == wave) f(g, __ffs(m) - 1);
}

// Column c of a row at position pos rotated back by the rotary angles of a d-wide head: (u, w) -> (u c + w s, w c - u s).  Lane
// l ^ 1 holds the other column of the pair.
__device__ __forceinline__ float unrotate_column(float x, const float2* __restrict__ rope, int pos, int c, int d) {
  const float other = __shfl_xor(x, 1, 64);
  const float2 t = rope[(int64_t)pos * (d / 2) + c / 2];
  return c & 1 ? x * t.x - other * t.y : x * t.x + other * t.y;
}

// 0 while every value added is finite, NaN from the first other one on.
__device__ __forceinline__ float mark_non_finite(float mark, float x) { return fmaf(x, 0.f, mark); }

}  // namespace zs

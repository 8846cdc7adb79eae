// Bandwidth-bound kernels of the stage step: norms, activations, RoPE, embedding, cross
// entropy, vector-gradient reductions and the fused AdamW.  Statistics and all arithmetic are
// fp32; storage is float or bf16.  Every global access is a 16-byte vector per lane where the
// shape allows it, consecutive lanes touching consecutive vectors.
#include "kernels.h"

namespace zs {

template <typename T> struct VT { typedef typename Vec<T>::type type; };

template <typename T> __device__ __forceinline__ void load_vec(const T* p, float (&out)[Vec<T>::N]) {
  typename Vec<T>::type v = *reinterpret_cast<const typename Vec<T>::type*>(p);
#pragma unroll
  for (int i = 0; i < Vec<T>::N; ++i) out[i] = to_f(v[i]);
}
template <typename T> __device__ __forceinline__ void store_vec(T* p, const float (&in)[Vec<T>::N]) {
  typename Vec<T>::type v;
#pragma unroll
  for (int i = 0; i < Vec<T>::N; ++i) v[i] = from_f<T>(in[i]);
  *reinterpret_cast<typename Vec<T>::type*>(p) = v;
}

// ------------------------------------------------------------------ norm forward
// One wave per row; three passes over a row that stays in cache (mean, variance, output).
template <typename T, int KIND>
__global__ __launch_bounds__(256) void norm_fwd_kernel(int Trows, int H, const T* __restrict__ x,
                                                       const T* __restrict__ g, const T* __restrict__ b, float eps,
                                                       T* __restrict__ n, float* __restrict__ rstd,
                                                       float* __restrict__ mean, T* __restrict__ copy) {
  constexpr int V = Vec<T>::N;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= Trows) return;
  const T* xr = x + (int64_t)row * H;
  float mu = 0.f;
  if (KIND == 0) {
    float s = 0.f;
    for (int c = lane * V; c < H; c += 64 * V) {
      float a[V];
      load_vec(xr + c, a);
#pragma unroll
      for (int i = 0; i < V; ++i) s += a[i];
    }
    mu = wave_sum(s) / (float)H;
  }
  float s2 = 0.f;
  for (int c = lane * V; c < H; c += 64 * V) {
    float a[V];
    load_vec(xr + c, a);
#pragma unroll
    for (int i = 0; i < V; ++i) s2 += (a[i] - mu) * (a[i] - mu);
  }
  const float r = 1.0f / sqrtf(wave_sum(s2) / (float)H + eps);
  if (lane == 0) {
    rstd[row] = r;
    if (KIND == 0) mean[row] = mu;
  }
  T* nr = n + (int64_t)row * H;
  for (int c = lane * V; c < H; c += 64 * V) {
    float a[V], gg[V], bb[V], o[V];
    load_vec(xr + c, a);
    load_vec(g + c, gg);
    if (KIND == 0) load_vec(b + c, bb);
    if (copy) store_vec(copy + (int64_t)row * H + c, a);
#pragma unroll
    for (int i = 0; i < V; ++i) o[i] = (a[i] - mu) * r * gg[i] + (KIND == 0 ? bb[i] : 0.f);
    store_vec(nr + c, o);
  }
}

// Same arithmetic with the row kept in registers (one global read): H <= 64 lanes x V x J, FULL: exactly that.  The
// element -> lane assignment and the order of every sum equal the kernel above, so the results are identical.
template <typename T, int KIND, int J, bool FULL>
__global__ __launch_bounds__(256) void norm_fwd_reg_kernel(int Trows, int width, const T* __restrict__ x, const T* __restrict__ g,
                                                           const T* __restrict__ b, float eps, T* __restrict__ n,
                                                           float* __restrict__ rstd, float* __restrict__ mean, T* __restrict__ copy) {
  constexpr int V = Vec<T>::N;
  const int H = FULL ? 64 * V * J : width;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= Trows) return;
  const T* xr = x + (int64_t)row * H;
  float a[J][V];
#pragma unroll
  for (int j = 0; j < J; ++j)
    if (FULL || (j * 64 + lane) * V < H) load_vec(xr + (j * 64 + lane) * V, a[j]);
  float mu = 0.f;
  if (KIND == 0) {
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < J; ++j)
      if (FULL || (j * 64 + lane) * V < H) {
#pragma unroll
        for (int i = 0; i < V; ++i) s += a[j][i];
      }
    mu = wave_sum(s) / (float)H;
  }
  float s2 = 0.f;
#pragma unroll
  for (int j = 0; j < J; ++j)
    if (FULL || (j * 64 + lane) * V < H) {
#pragma unroll
      for (int i = 0; i < V; ++i) s2 += (a[j][i] - mu) * (a[j][i] - mu);
    }
  const float r = 1.0f / sqrtf(wave_sum(s2) / (float)H + eps);
  if (lane == 0) {
    rstd[row] = r;
    if (KIND == 0) mean[row] = mu;
  }
  T* nr = n + (int64_t)row * H;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int c = (j * 64 + lane) * V;
    if (!FULL && c >= H) continue;
    float gg[V], bb[V], o[V];
    load_vec(g + c, gg);
    if (KIND == 0) load_vec(b + c, bb);
    if (copy) store_vec(copy + (int64_t)row * H + c, a[j]);   // the values as loaded: bit for bit
#pragma unroll
    for (int i = 0; i < V; ++i) o[i] = (a[j][i] - mu) * r * gg[i] + (KIND == 0 ? bb[i] : 0.f);
    store_vec(nr + c, o);
  }
}

// Which register-resident norm kernel takes rows of H elements: J vectors per lane, `full` when they are exactly the row, and
// for the backward the waves that share a row.  The row lengths of the usual model widths have exact variants; any other row
// up to 16 (backward: 32) vectors per lane of one wave runs with its last vectors masked.  J = 0: none, longer rows take the
// kernels that re-read the row.
struct NormPlan { int J = 0; bool full = false; int waves = 1; };
static int per_chunk(DType dt) { return 64 * (dt == F32 ? 4 : 8); }   // elements that a wave moves per access
static NormPlan norm_plan_fwd(DType dt, int H) {
  const int per = per_chunk(dt), need = (int)cdiv(H, per);
  NormPlan p;
  p.full = H % per == 0 && (need == 1 || need == 2 || need == 4 || need == 8 || need == 10);
  if (need <= 8 || p.full) p.J = need;
  else if (need <= 16) p.J = (need + 1) / 2 * 2;
  return p;
}
static NormPlan norm_plan_bwd(DType dt, int H) {
  const int per = per_chunk(dt), need = (int)cdiv(H, per);
  NormPlan p;
  p.full = H % per == 0 && (need == 1 || need == 2 || need == 4 || need == 8 || need == 10);
  p.waves = need <= 4 || p.full ? 1 : need <= 8 ? 2 : need <= 16 ? 4 : 8;
  if (need <= 32) p.J = (int)cdiv(need, p.waves);
  return p;
}

hipError_t norm_fwd(hipStream_t st, DType dt, int kind, int T, int H, const void* x, const void* g, const void* b,
                    float eps, void* n, float* rstd, float* mean, void* copy) {
  dim3 grid((unsigned)cdiv(T, 4)), blk(256);
  const NormPlan p = norm_plan_fwd(dt, H);
#define LR(TT, KK, JJ, FF) \
  hipLaunchKernelGGL((norm_fwd_reg_kernel<TT, KK, JJ, FF>), grid, blk, 0, st, T, H, (const TT*)x, (const TT*)g, (const TT*)b, eps, (TT*)n, rstd, mean, (TT*)copy)
#define LJ(TT, KK) \
  if (p.full) switch (p.J) { case 1: LR(TT, KK, 1, true); break; case 2: LR(TT, KK, 2, true); break; case 4: LR(TT, KK, 4, true); break; \
                             case 8: LR(TT, KK, 8, true); break; default: LR(TT, KK, 10, true); break; } \
  else switch (p.J) { case 1: LR(TT, KK, 1, false); break; case 2: LR(TT, KK, 2, false); break; case 3: LR(TT, KK, 3, false); break; \
                      case 4: LR(TT, KK, 4, false); break; case 5: LR(TT, KK, 5, false); break; case 6: LR(TT, KK, 6, false); break; \
                      case 7: LR(TT, KK, 7, false); break; case 8: LR(TT, KK, 8, false); break; case 10: LR(TT, KK, 10, false); break; \
                      case 12: LR(TT, KK, 12, false); break; case 14: LR(TT, KK, 14, false); break; default: LR(TT, KK, 16, false); break; }
#define L(TT, KK) \
  hipLaunchKernelGGL((norm_fwd_kernel<TT, KK>), grid, blk, 0, st, T, H, (const TT*)x, (const TT*)g, (const TT*)b, eps, (TT*)n, rstd, mean, (TT*)copy)
  if (p.J) {
    if (dt == F32) { if (kind == 0) { LJ(float, 0) } else { LJ(float, 1) } }
    else if (dt == BF16) { if (kind == 0) { LJ(bf16, 0) } else { LJ(bf16, 1) } }
    else { if (kind == 0) { LJ(f16, 0) } else { LJ(f16, 1) } }
  } else {
    if (dt == F32) { if (kind == 0) L(float, 0); else L(float, 1); }
    else if (dt == BF16) { if (kind == 0) L(bf16, 0); else L(bf16, 1); }
    else { if (kind == 0) L(f16, 0); else L(f16, 1); }
  }
#undef L
#undef LJ
#undef LR
  return hipGetLastError();
}

// ------------------------------------------------------------------ norm backward (dx only)
// u = dn*g; dx = r*(u - mean(u) [LN] - xhat*mean(u*xhat)) + dres
template <typename T, int KIND>
__global__ __launch_bounds__(256) void norm_bwd_kernel(int Trows, int H, const T* __restrict__ dn,
                                                       const T* __restrict__ x, const T* __restrict__ g,
                                                       const float* __restrict__ rstd, const float* __restrict__ mean,
                                                       const T* dres, T* dx) {
  constexpr int V = Vec<T>::N;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= Trows) return;
  const float r = rstd[row];
  const float mu = (KIND == 0) ? mean[row] : 0.f;
  const T* xr = x + (int64_t)row * H;
  const T* dr = dn + (int64_t)row * H;
  float su = 0.f, sux = 0.f;
  for (int c = lane * V; c < H; c += 64 * V) {
    float a[V], d[V], gg[V];
    load_vec(xr + c, a);
    load_vec(dr + c, d);
    load_vec(g + c, gg);
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const float u = d[i] * gg[i];
      su += u;
      sux += u * (a[i] - mu) * r;
    }
  }
  const float mu_u = (KIND == 0) ? wave_sum(su) / (float)H : 0.f;
  const float mu_ux = wave_sum(sux) / (float)H;
  for (int c = lane * V; c < H; c += 64 * V) {
    float a[V], d[V], gg[V], o[V], rs[V];
    load_vec(xr + c, a);
    load_vec(dr + c, d);
    load_vec(g + c, gg);
    if (dres) load_vec(dres + (int64_t)row * H + c, rs);
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const float u = d[i] * gg[i];
      o[i] = r * (u - mu_u - (a[i] - mu) * r * mu_ux) + (dres ? rs[i] : 0.f);
    }
    store_vec(dx + (int64_t)row * H + c, o);
  }
}

static hipError_t norm_bwd(hipStream_t st, DType dt, int kind, int T, int H, const void* dn, const void* x, const void* g,
                           const float* rstd, const float* mean, const void* dres, void* dx) {
  dim3 grid((unsigned)cdiv(T, 4)), blk(256);
#define L(TT, KK) \
  hipLaunchKernelGGL((norm_bwd_kernel<TT, KK>), grid, blk, 0, st, T, H, (const TT*)dn, (const TT*)x, (const TT*)g, rstd, mean, (const TT*)dres, (TT*)dx)
  if (dt == F32) { if (kind == 0) L(float, 0); else L(float, 1); }
  else if (dt == BF16) { if (kind == 0) L(bf16, 0); else L(bf16, 1); }
  else { if (kind == 0) L(f16, 0); else L(f16, 1); }
#undef L
  return hipGetLastError();
}

// ------------------------------------------------------------------ column partial sums
// grid (column chunks of 64*V, nblk).  A workgroup is 64 column threads (V columns each) x 4 row groups:
// row group q walks rows r0+q, r0+q+4, ... of the block, four rows in flight per thread, and the four
// groups' sums are added in the order 0..3 through LDS, so the result does not depend on timing.
template <typename T>
__device__ __forceinline__ void colsum_block(int chunk, int Trows, int N, const T* __restrict__ a, int64_t lda, const T* __restrict__ x, int64_t ldx,
                                             const float* __restrict__ rstd, const float* __restrict__ mean, float* __restrict__ part,
                                             int rows_per_blk) {
  constexpr int V = Vec<T>::N;
  __shared__ float red[3][64][V];
  const int ct = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int col = (chunk * 64 + ct) * V;
  const bool live = col < N;
  const int r0 = blockIdx.y * rows_per_blk;
  const int r1 = min(Trows, r0 + rows_per_blk);
  float acc[V];
#pragma unroll
  for (int i = 0; i < V; ++i) acc[i] = 0.f;
  if (live) {
    for (int t0 = r0 + q; t0 < r1; t0 += 16) {
      float av[4][V], xv[4][V];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int t = t0 + 4 * u;
        if (t < r1) {
          load_vec(a + (int64_t)t * lda + col, av[u]);
          if (x) load_vec(x + (int64_t)t * ldx + col, xv[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int t = t0 + 4 * u;
        if (t < r1) {
          if (x) {
            const float r = rstd[t];
            const float mu = mean ? mean[t] : 0.f;
#pragma unroll
            for (int i = 0; i < V; ++i) acc[i] += av[u][i] * ((xv[u][i] - mu) * r);
          } else {
#pragma unroll
            for (int i = 0; i < V; ++i) acc[i] += av[u][i];
          }
        }
      }
    }
  }
  if (q > 0) {
#pragma unroll
    for (int i = 0; i < V; ++i) red[q - 1][ct][i] = acc[i];
  }
  __syncthreads();
  if (q == 0 && live) {
    float* p = part + (int64_t)blockIdx.y * N + col;
#pragma unroll
    for (int i = 0; i < V; ++i) p[i] = ((acc[i] + red[0][ct][i]) + red[1][ct][i]) + red[2][ct][i];
  }
}
template <typename T>
__global__ __launch_bounds__(256) void colsum_kernel(int Trows, int N, const T* __restrict__ a, int64_t lda,
                                                     const T* __restrict__ x, int64_t ldx,
                                                     const float* __restrict__ rstd, const float* __restrict__ mean,
                                                     float* __restrict__ part, int rows_per_blk) {
  colsum_block<T>(blockIdx.x, Trows, N, a, lda, x, ldx, rstd, mean, part, rows_per_blk);
}
// The plain sums of up to four arrays over the same rows in one launch: the bias gradients of a layer, whose launches on their
// own are too short to be worth one each (GPT step of 1024 tokens in fp32, hidden 256: 942 -> 895 us).
struct ColsumJobs { ColsumJob job[4]; int first[4]; };   // first: column chunk with which a job begins
template <typename T> __global__ __launch_bounds__(256) void colsum_jobs_kernel(int Trows, int njobs, ColsumJobs js, int rows_per_blk) {
  int k = 0;
#pragma unroll
  for (int i = 1; i < 4; ++i)
    if (i < njobs && (int)blockIdx.x >= js.first[i]) k = i;
  const ColsumJob& j = js.job[k];
  colsum_block<T>(blockIdx.x - js.first[k], Trows, j.width, (const T*)j.a, j.lda, nullptr, 0, nullptr, nullptr, j.part, rows_per_blk);
}

hipError_t colsum_partial(hipStream_t st, DType dt, int T, int N, const void* a, int64_t lda, const void* x,
                          int64_t ldx, const float* rstd, const float* mean, float* part, int nblk) {
  const int rows_per_blk = (int)cdiv(T, nblk);
  const int V = dt == F32 ? 4 : 8;
  dim3 grid((unsigned)cdiv(N, 64 * V), (unsigned)nblk), blk(256);
  if (dt == F32)
    hipLaunchKernelGGL(colsum_kernel<float>, grid, blk, 0, st, T, N, (const float*)a, lda, (const float*)x, ldx, rstd, mean, part, rows_per_blk);
  else if (dt == BF16)
    hipLaunchKernelGGL(colsum_kernel<bf16>, grid, blk, 0, st, T, N, (const bf16*)a, lda, (const bf16*)x, ldx, rstd, mean, part, rows_per_blk);
  else
    hipLaunchKernelGGL(colsum_kernel<f16>, grid, blk, 0, st, T, N, (const f16*)a, lda, (const f16*)x, ldx, rstd, mean, part, rows_per_blk);
  return hipGetLastError();
}

hipError_t colsum_partials(hipStream_t st, DType dt, int T, const ColsumJob* jobs, int njobs, int nblk) {
  if (njobs < 1 || njobs > 4) return hipErrorInvalidValue;
  const int rows_per_blk = (int)cdiv(T, nblk), V = dt == F32 ? 4 : 8;
  ColsumJobs js = {};
  int chunks = 0;
  for (int i = 0; i < njobs; ++i) {
    js.job[i] = jobs[i];
    js.first[i] = chunks;
    chunks += (int)cdiv(jobs[i].width, 64 * V);
  }
  const dim3 grid((unsigned)chunks, (unsigned)nblk), blk(256);
  if (dt == F32) hipLaunchKernelGGL(colsum_jobs_kernel<float>, grid, blk, 0, st, T, njobs, js, rows_per_blk);
  else if (dt == BF16) hipLaunchKernelGGL(colsum_jobs_kernel<bf16>, grid, blk, 0, st, T, njobs, js, rows_per_blk);
  else hipLaunchKernelGGL(colsum_jobs_kernel<f16>, grid, blk, 0, st, T, njobs, js, rows_per_blk);
  return hipGetLastError();
}

// ------------------------------------------------------------------ norm backward + partial sums, row in registers
// norm_bwd_kernel and the two colsum_kernel passes over the same rows in one kernel: dn and x are read once.
// One workgroup per row block (the blocks of colsum_partial).  WPR = 1: four waves, wave q walks rows r0+q, r0+q+4, ... of the
// block, computes dx of each row and keeps the running column sums of dn*xhat (and dn) of its rows in registers; the waves'
// sums are then added in the order 0..3 through LDS: colsum_kernel's order of additions per column.  WPR = 2, 4, 8: eight
// waves, that many of them share a row (vector j of part p covers chunk j WPR + p), their sums of u and u*xhat meet in LDS
// once per row, and 8 / WPR rows are walked side by side.  A wave thereby holds at most 4 vectors per lane and two waves fit
// a SIMD, one's loads under the other's arithmetic (20 instructions per element).  FULL: H = 64 V J exactly (WPR = 1); else
// the vectors past the row's end are masked.  With up to 4 vectors per lane the next row's loads are in flight beside a row's sums (with 8
// or 10, FULL only, there are no registers for them): without, a workgroup went through load, reduce, barrier and store 17 times with nothing
// in flight in between.  bf16, us, without : with: LayerNorm, 4097 rows of 3080 28.0 : 23.4 (48 as three kernels), 8200 rows of 600
// 16.7 : 13.8; RMSNorm, 4100 rows of 1288 13.7 : 10.4, 700 rows of 8192 13.8 : 11.9.  Exact rows of 4096 and 5120 elements stay with
// one wave per row (LayerNorm 30 and 42 us, RMSNorm 24 and 18 for 4096 and 2048 rows).
template <typename T, int KIND, int J, int WPR, bool FULL>
__global__ __launch_bounds__(WPR == 1 ? 256 : 512) void norm_bwd_partials_reg_kernel(int Trows, int width, const T* __restrict__ dn, const T* __restrict__ x,
                                                                    const T* __restrict__ g, const float* __restrict__ rstd,
                                                                    const float* __restrict__ mean, const T* dres, T* dx,
                                                                    float* __restrict__ part_g, float* __restrict__ part_b,
                                                                    int rows_per_blk) {
  constexpr int V = Vec<T>::N, NW = WPR == 1 ? 4 : 8, RG = NW / WPR;      // waves; rows walked side by side
  const int H = FULL ? 64 * V * J : width;
  extern __shared__ __align__(16) float red[];   // [RG - 1][WPR J][64 V]: the sums of the later rows, for part_g and then for part_b
  __shared__ float cross[2][NW][2];              // WPR > 1: the waves' sums of a row, two buffers in turn
  // Rows in scalar registers, so that a wave branches past the loads of a row that is not there: fp32 RMSNorm, 2048 rows of 1024 5.6 -> 5.4 us
  // with it.  Rows whose last vectors are masked lose by it (fp32 LayerNorm, 8200 of 600 17.9 -> 21.1).
  const int lane = threadIdx.x & 63, wave = FULL && J <= 4 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : threadIdx.x >> 6;
  const int q = wave / WPR, part = wave % WPR;
  const int r0 = blockIdx.x * rows_per_blk;
  const int r1 = min(Trows, r0 + rows_per_blk);
  auto col = [&](int j) { return ((j * WPR + part) * 64 + lane) * V; };
  auto in = [&](int j) { return FULL || col(j) < H; };
  float pg[J][V], pb[KIND == 0 ? J : 1][V];
#pragma unroll
  for (int j = 0; j < J; ++j)
#pragma unroll
    for (int i = 0; i < V; ++i) { pg[j][i] = 0.f; if (KIND == 0) pb[j][i] = 0.f; }
  typedef typename Vec<T>::type TV;
  if constexpr (J > 4) {   // exact rows in one wave each.  A loop of its own: which product of a sum is fused into a multiply-add, and so the
                           // last bit of dx, is the compiler's choice and changes with the code around it
    for (int row = r0 + q; row < r1; row += RG) {
      const float r = rstd[row];
      const float mu = KIND == 0 ? mean[row] : 0.f;
      const int64_t off = (int64_t)row * H;
      TV xv[J], dv[J], rv[J];
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int c = col(j);
        xv[j] = *reinterpret_cast<const TV*>(x + off + c);
        dv[j] = *reinterpret_cast<const TV*>(dn + off + c);
        if (dres) rv[j] = *reinterpret_cast<const TV*>(dres + off + c);
      }
      float su = 0.f, sux = 0.f;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        float gg[V];
        load_vec(g + col(j), gg);
#pragma unroll
        for (int i = 0; i < V; ++i) {
          const float d = to_f(dv[j][i]), xx = to_f(xv[j][i]);
          const float u = d * gg[i];
          su += u;
          sux += u * (xx - mu) * r;
          pg[j][i] += d * ((xx - mu) * r);
          if (KIND == 0) pb[j][i] += d;
        }
      }
      su = (KIND == 0) ? wave_sum(su) : 0.f;
      sux = wave_sum(sux);
      const float mu_u = su / (float)H;
      const float mu_ux = sux / (float)H;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int c = col(j);
        float o[V], gg[V];
        load_vec(g + c, gg);
#pragma unroll
        for (int i = 0; i < V; ++i) {
          const float u = to_f(dv[j][i]) * gg[i];
          o[i] = r * (u - mu_u - (to_f(xv[j][i]) - mu) * r * mu_ux) + (dres ? to_f(rv[j][i]) : 0.f);
        }
        store_vec(dx + off + c, o);
      }
    }
  } else {
    // The next row's loads go out before this row's sums, and the gains stay in registers.  dx may lie over dres: other rows.
    struct Row { TV x[J], d[J], r[J]; float rstd, mean; };
    auto load = [&](Row& w, int row) {
      const bool live = row < r1;
      w.rstd = live ? rstd[row] : 0.f;
      w.mean = (KIND == 0 && live) ? mean[row] : 0.f;
      const int64_t off = (int64_t)row * H;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        if (!live || !in(j)) continue;
        w.x[j] = *reinterpret_cast<const TV*>(x + off + col(j));
        w.d[j] = *reinterpret_cast<const TV*>(dn + off + col(j));
        if (dres) w.r[j] = *reinterpret_cast<const TV*>(dres + off + col(j));
      }
    };
    TV gains[J];
#pragma unroll
    for (int j = 0; j < J; ++j)
      if (in(j)) gains[j] = *reinterpret_cast<const TV*>(g + col(j));
    auto gain = [&](int j, float (&gg)[V]) {
#pragma unroll
      for (int i = 0; i < V; ++i) gg[i] = to_f(gains[j][i]);
    };
    int turn = 0;
    Row cur, next;
    load(cur, r0 + q);
    for (int row = r0 + q; (WPR == 1 ? row : row - q) < r1; row += RG) {   // WPR > 1: the same steps in every wave, for the barrier
      load(next, row + RG);
      const bool live = WPR == 1 || row < r1;
      const float r = cur.rstd, mu = cur.mean;
      const int64_t off = (int64_t)row * H;
      const TV (&xv)[J] = cur.x, (&dv)[J] = cur.d, (&rv)[J] = cur.r;
      float su = 0.f, sux = 0.f;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        if (!live || !in(j)) continue;
        float gg[V];
        gain(j, gg);
#pragma unroll
        for (int i = 0; i < V; ++i) {
          const float d = to_f(dv[j][i]), xx = to_f(xv[j][i]);
          const float u = d * gg[i];
          su += u;
          sux += u * (xx - mu) * r;
          pg[j][i] += d * ((xx - mu) * r);
          if (KIND == 0) pb[j][i] += d;
        }
      }
      su = (KIND == 0) ? wave_sum(su) : 0.f;
      sux = wave_sum(sux);
      if constexpr (WPR > 1) {
        if (lane == 0) { cross[turn][wave][0] = su; cross[turn][wave][1] = sux; }
        __syncthreads();   // the other buffer was read before this barrier, so it may be written after it
        su = sux = 0.f;
#pragma unroll
        for (int w = 0; w < WPR; ++w) { su += cross[turn][q * WPR + w][0]; sux += cross[turn][q * WPR + w][1]; }
        turn ^= 1;
      }
      const float mu_u = su / (float)H;
      const float mu_ux = sux / (float)H;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        if (!live || !in(j)) continue;
        const int c = col(j);
        float o[V], gg[V];
        gain(j, gg);
#pragma unroll
        for (int i = 0; i < V; ++i) {
          const float u = to_f(dv[j][i]) * gg[i];
          o[i] = r * (u - mu_u - (to_f(xv[j][i]) - mu) * r * mu_ux) + (dres ? to_f(rv[j][i]) : 0.f);
        }
        store_vec(dx + off + c, o);
      }
      cur = next;
    }
  }
  // sums over the rows walked side by side, in order, first of dn*xhat, then (LayerNorm) of dn
#pragma unroll
  for (int pass = 0; pass < (KIND == 0 ? 2 : 1); ++pass) {
    if (pass) __syncthreads();
    // LDS layout [row][chunk][quad of 4 columns][lane]: consecutive lanes 16 bytes apart, no bank conflicts
    constexpr int Q4 = V / 4;
    f32x4* red4 = reinterpret_cast<f32x4*>(red);
    auto at = [&](int u, int j, int h) { return (((u - 1) * (J * WPR) + j * WPR + part) * Q4 + h) * 64 + lane; };
    if (q > 0) {
#pragma unroll
      for (int j = 0; j < J; ++j)
#pragma unroll
        for (int h = 0; h < Q4; ++h) {
          f32x4 t;
#pragma unroll
          for (int e = 0; e < 4; ++e) t[e] = pass ? pb[KIND == 0 ? j : 0][4 * h + e] : pg[j][4 * h + e];
          red4[at(q, j, h)] = t;
        }
    }
    if (RG > 1) __syncthreads();
    if (q == 0) {
      float* p = (pass ? part_b : part_g) + (int64_t)blockIdx.x * H;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        if (!in(j)) continue;
#pragma unroll
        for (int h = 0; h < Q4; ++h) {
          f32x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = pass ? pb[KIND == 0 ? j : 0][4 * h + e] : pg[j][4 * h + e];
#pragma unroll
          for (int u = 1; u < RG; ++u) o += red4[at(u, j, h)];
          *reinterpret_cast<f32x4*>(p + col(j) + 4 * h) = o;
        }
      }
    }
  }
}

hipError_t norm_bwd_partials(hipStream_t st, DType dt, int kind, int T, int H, const void* dn, const void* x, const void* g,
                             const float* rstd, const float* mean, const void* dres, void* dx, float* part_g,
                             float* part_b, int nblk) {
  const NormPlan p = norm_plan_bwd(dt, H);
  if (p.J && nblk >= 1 && part_g && (kind != 0 || part_b)) {   // one pass over the rows
    const int rows_per_blk = (int)cdiv(T, nblk);
    const int nw = p.waves == 1 ? 4 : 8;
    dim3 grid((unsigned)nblk), blk(64 * nw);
    const size_t smem = (size_t)(nw / p.waves - 1) * p.waves * p.J * per_chunk(dt) * sizeof(float);
#define LR(TT, KK, JJ, WW, FF) \
  hipLaunchKernelGGL((norm_bwd_partials_reg_kernel<TT, KK, JJ, WW, FF>), grid, blk, smem, st, T, H, (const TT*)dn, (const TT*)x, (const TT*)g, rstd, mean, (const TT*)dres, (TT*)dx, part_g, part_b, rows_per_blk)
#define LJ(TT, KK) \
  if (p.full) switch (p.J) { case 1: LR(TT, KK, 1, 1, true); break; case 2: LR(TT, KK, 2, 1, true); break; case 4: LR(TT, KK, 4, 1, true); break; \
                             case 8: LR(TT, KK, 8, 1, true); break; default: LR(TT, KK, 10, 1, true); break; } \
  else if (p.waves == 1) switch (p.J) { case 1: LR(TT, KK, 1, 1, false); break; case 2: LR(TT, KK, 2, 1, false); break; \
                                        case 3: LR(TT, KK, 3, 1, false); break; default: LR(TT, KK, 4, 1, false); break; } \
  else if (p.waves == 2) { if (p.J == 3) LR(TT, KK, 3, 2, false); else LR(TT, KK, 4, 2, false); } \
  else if (p.waves == 4) { if (p.J == 3) LR(TT, KK, 3, 4, false); else LR(TT, KK, 4, 4, false); } \
  else { if (p.J == 3) LR(TT, KK, 3, 8, false); else LR(TT, KK, 4, 8, false); }
    if (dt == F32) { if (kind == 0) { LJ(float, 0) } else { LJ(float, 1) } }
    else if (dt == BF16) { if (kind == 0) { LJ(bf16, 0) } else { LJ(bf16, 1) } }
    else { if (kind == 0) { LJ(f16, 0) } else { LJ(f16, 1) } }
#undef LJ
#undef LR
    return hipGetLastError();
  }
  hipError_t e = colsum_partial(st, dt, T, H, dn, H, x, H, rstd, kind == 0 ? mean : nullptr, part_g, nblk);
  if (e == hipSuccess && kind == 0) e = colsum_partial(st, dt, T, H, dn, H, nullptr, H, nullptr, nullptr, part_b, nblk);
  if (e == hipSuccess) e = norm_bwd(st, dt, kind, T, H, dn, x, g, rstd, mean, dres, dx);
  return e;
}

// dst[c] += sum over the blocks.  A workgroup owns 64 columns: thread (row group q of 16, quad of 4 columns) adds blocks q,
// q + 16, ... eight loads at a time, and the 16 groups' sums are added in the order 0..15 through LDS: a fixed order.  One
// thread per column walking all 256 blocks was a chain of 64 loads on a few workgroups (22 us for the 20 vectors of width
// 256..1024 of a small GPT stage, 38 us at width 2048..8192; 5 and 20 us this way).
__global__ __launch_bounds__(256) void reduce_partials_kernel(const ReduceJob* __restrict__ jobs) {
  __shared__ f32x4 red[16][16];
  const ReduceJob j = jobs[blockIdx.x];
  const int qd = threadIdx.x & 15, q = threadIdx.x >> 4, c = (blockIdx.y * 16 + qd) * 4;
  if ((int)blockIdx.y * 64 >= j.width) return;
  const bool live = c < j.width;       // widths are multiples of 8
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  if (live) {
    const float* p = j.part + c;
#pragma unroll 8
    for (int b = q; b < j.nblk; b += 16) s += *reinterpret_cast<const f32x4*>(p + (int64_t)b * j.width);
  }
  red[q][qd] = s;
  __syncthreads();
  if (q == 0 && live) {
    f32x4* d = reinterpret_cast<f32x4*>(j.dst + c);
    for (int u = 1; u < 16; ++u) s += red[u][qd];
    *d = *d + s;
  }
}

hipError_t reduce_partials(hipStream_t st, const ReduceJob* jobs_dev, int njobs, int max_width) {
  if (njobs == 0) return hipSuccess;
  dim3 grid((unsigned)njobs, (unsigned)cdiv(max_width, 64)), blk(256);
  hipLaunchKernelGGL(reduce_partials_kernel, grid, blk, 0, st, jobs_dev);
  return hipGetLastError();
}

// ------------------------------------------------------------------ RoPE
__global__ void rope_table_kernel(int S, int d, double base, float2* table) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  const int half = d / 2;
  if (idx >= S * half) return;
  const int s = idx / half, i = idx % half;
  const double theta = (double)s * pow(base, -2.0 * (double)i / (double)d);
  table[idx] = make_float2((float)cos(theta), (float)sin(theta));
}
hipError_t rope_table(hipStream_t st, int S, int d, float base, float2* table) {
  const int n = S * (d / 2);
  hipLaunchKernelGGL(rope_table_kernel, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, st, S, d, (double)base, table);
  return hipGetLastError();
}

template <typename T>
__global__ __launch_bounds__(256) void rope_kernel(int Trows, int S, int ncols, int d, T* a, int64_t ld,
                                                   const float2* __restrict__ table, float sign) {
  constexpr int V = Vec<T>::N;
  const int vec_per_row = ncols / V;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (int64_t)Trows * vec_per_row) return;
  const int t = (int)(idx / vec_per_row);
  const int c = (int)(idx % vec_per_row) * V;
  const int pos = t % S;
  T* p = a + (int64_t)t * ld + c;
  float u[V], o[V];
  load_vec(p, u);
  const int i0 = (c % d) / 2;
#pragma unroll
  for (int i = 0; i < V / 2; ++i) {
    const float2 cs = table[pos * (d / 2) + i0 + i];
    const float sn = sign * cs.y;
    o[2 * i] = u[2 * i] * cs.x - u[2 * i + 1] * sn;
    o[2 * i + 1] = u[2 * i] * sn + u[2 * i + 1] * cs.x;
  }
  store_vec(p, o);
}
hipError_t rope_apply(hipStream_t st, DType dt, int T, int S, int ncols, int d, void* a, int64_t ld,
                      const float2* table, float sign) {
  const int V = dt == F32 ? 4 : 8;
  const int64_t n = (int64_t)T * (ncols / V);
  dim3 grid((unsigned)cdiv(n, 256)), blk(256);
  if (dt == F32) hipLaunchKernelGGL(rope_kernel<float>, grid, blk, 0, st, T, S, ncols, d, (float*)a, ld, table, sign);
  else if (dt == BF16) hipLaunchKernelGGL(rope_kernel<bf16>, grid, blk, 0, st, T, S, ncols, d, (bf16*)a, ld, table, sign);
  else hipLaunchKernelGGL(rope_kernel<f16>, grid, blk, 0, st, T, S, ncols, d, (f16*)a, ld, table, sign);
  return hipGetLastError();
}

// ------------------------------------------------------------------ activations
template <typename T, int MODE>  // 0: a = gelu(z); 1: dz = da * gelu'(z)
__global__ __launch_bounds__(256) void gelu_kernel(int64_t nvec, const T* __restrict__ z, const T* __restrict__ da,
                                                   T* __restrict__ out) {
  constexpr int V = Vec<T>::N;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= nvec) return;
  float zz[V], o[V], d[V];
  load_vec(z + i * V, zz);
  if (MODE == 1) load_vec(da + i * V, d);
#pragma unroll
  for (int k = 0; k < V; ++k) o[k] = MODE == 0 ? gelu_f(zz[k]) : d[k] * gelu_df(zz[k]);
  store_vec(out + i * V, o);
}
hipError_t gelu_fwd(hipStream_t st, DType dt, int64_t n, const void* z, void* a) {
  const int V = dt == F32 ? 4 : 8;
  dim3 grid((unsigned)cdiv(n / V, 256)), blk(256);
  if (dt == F32) hipLaunchKernelGGL((gelu_kernel<float, 0>), grid, blk, 0, st, n / V, (const float*)z, (const float*)nullptr, (float*)a);
  else if (dt == BF16) hipLaunchKernelGGL((gelu_kernel<bf16, 0>), grid, blk, 0, st, n / V, (const bf16*)z, (const bf16*)nullptr, (bf16*)a);
  else hipLaunchKernelGGL((gelu_kernel<f16, 0>), grid, blk, 0, st, n / V, (const f16*)z, (const f16*)nullptr, (f16*)a);
  return hipGetLastError();
}
hipError_t gelu_bwd(hipStream_t st, DType dt, int64_t n, const void* z, const void* da, void* dz) {
  const int V = dt == F32 ? 4 : 8;
  dim3 grid((unsigned)cdiv(n / V, 256)), blk(256);
  if (dt == F32) hipLaunchKernelGGL((gelu_kernel<float, 1>), grid, blk, 0, st, n / V, (const float*)z, (const float*)da, (float*)dz);
  else if (dt == BF16) hipLaunchKernelGGL((gelu_kernel<bf16, 1>), grid, blk, 0, st, n / V, (const bf16*)z, (const bf16*)da, (bf16*)dz);
  else hipLaunchKernelGGL((gelu_kernel<f16, 1>), grid, blk, 0, st, n / V, (const f16*)z, (const f16*)da, (f16*)dz);
  return hipGetLastError();
}

template <typename T, int MODE>  // 0: a = silu(g)*u ; 1: (dg, du) from da
__global__ __launch_bounds__(256) void swiglu_kernel(int Trows, int F, const T* gu, const T* __restrict__ da, T* out) {
  constexpr int V = Vec<T>::N;
  const int vec_per_row = F / V;
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (int64_t)Trows * vec_per_row) return;
  const int t = (int)(idx / vec_per_row);
  const int c = (int)(idx % vec_per_row) * V;
  float g[V], u[V];
  load_vec(gu + (int64_t)t * 2 * F + c, g);
  load_vec(gu + (int64_t)t * 2 * F + F + c, u);
  if (MODE == 0) {
    float o[V];
#pragma unroll
    for (int k = 0; k < V; ++k) o[k] = glu_f(g[k], u[k]);
    store_vec(out + (int64_t)t * F + c, o);
  } else {
    float d[V], dg[V], du[V];
    load_vec(da + (int64_t)t * F + c, d);
#pragma unroll
    for (int k = 0; k < V; ++k) glu_df(d[k], g[k], u[k], dg[k], du[k]);
    store_vec(out + (int64_t)t * 2 * F + c, dg);
    store_vec(out + (int64_t)t * 2 * F + F + c, du);
  }
}
hipError_t swiglu_fwd(hipStream_t st, DType dt, int T, int F, const void* gu, void* a) {
  const int V = dt == F32 ? 4 : 8;
  dim3 grid((unsigned)cdiv((int64_t)T * (F / V), 256)), blk(256);
  if (dt == F32) hipLaunchKernelGGL((swiglu_kernel<float, 0>), grid, blk, 0, st, T, F, (const float*)gu, (const float*)nullptr, (float*)a);
  else if (dt == BF16) hipLaunchKernelGGL((swiglu_kernel<bf16, 0>), grid, blk, 0, st, T, F, (const bf16*)gu, (const bf16*)nullptr, (bf16*)a);
  else hipLaunchKernelGGL((swiglu_kernel<f16, 0>), grid, blk, 0, st, T, F, (const f16*)gu, (const f16*)nullptr, (f16*)a);
  return hipGetLastError();
}
hipError_t swiglu_bwd(hipStream_t st, DType dt, int T, int F, const void* gu, const void* da, void* dgu) {
  const int V = dt == F32 ? 4 : 8;
  dim3 grid((unsigned)cdiv((int64_t)T * (F / V), 256)), blk(256);
  if (dt == F32) hipLaunchKernelGGL((swiglu_kernel<float, 1>), grid, blk, 0, st, T, F, (const float*)gu, (const float*)da, (float*)dgu);
  else if (dt == BF16) hipLaunchKernelGGL((swiglu_kernel<bf16, 1>), grid, blk, 0, st, T, F, (const bf16*)gu, (const bf16*)da, (bf16*)dgu);
  else hipLaunchKernelGGL((swiglu_kernel<f16, 1>), grid, blk, 0, st, T, F, (const f16*)gu, (const f16*)da, (f16*)dgu);
  return hipGetLastError();
}

// ------------------------------------------------------------------ embedding
template <typename T>
__global__ __launch_bounds__(256) void embed_fwd_kernel(int H, int V, const int32_t* __restrict__ ids,
                                                        const T* __restrict__ E, T* __restrict__ x, int32_t* __restrict__ keep) {
  constexpr int VN = Vec<T>::N;
  typedef typename Vec<T>::type vec_t;
  const int t = blockIdx.x;
  const int id = ids[t];
  if (keep && threadIdx.x == 0) keep[t] = id;
  const bool ok = id >= 0 && id < V;
  for (int c = threadIdx.x * VN; c < H; c += 256 * VN) {
    vec_t v;
    if (ok) v = *reinterpret_cast<const vec_t*>(E + (int64_t)id * H + c);   // bit-exact row copy
    else {
#pragma unroll
      for (int i = 0; i < VN; ++i) v[i] = from_f<T>(0.f);
    }
    *reinterpret_cast<vec_t*>(x + (int64_t)t * H + c) = v;
  }
}
hipError_t embed_fwd(hipStream_t st, DType dt, int T, int H, int V, const int32_t* ids, const void* E, void* x, int32_t* keep) {
  if (dt == F32) hipLaunchKernelGGL(embed_fwd_kernel<float>, dim3(T), dim3(256), 0, st, H, V, ids, (const float*)E, (float*)x, keep);
  else if (dt == BF16) hipLaunchKernelGGL(embed_fwd_kernel<bf16>, dim3(T), dim3(256), 0, st, H, V, ids, (const bf16*)E, (bf16*)x, keep);
  else hipLaunchKernelGGL(embed_fwd_kernel<f16>, dim3(T), dim3(256), 0, st, H, V, ids, (const f16*)E, (f16*)x, keep);
  return hipGetLastError();
}

// One workgroup per token.  The workgroup of the FIRST token carrying an id adds the rows of
// every token with that id, in increasing token order, to dE[id]; the others exit.  A row of dE
// has one owner workgroup and a column one owner thread, so no atomics are needed and the
// result does not depend on scheduling.  Tokens are looked over 256 at a time, each wave leaving its matches as one
// 64-bit mask, so only the set bits are visited (testing 256 flags one by one in every workgroup took 19 us for 256 tokens,
// 4 us this way), and rows move 16 bytes of dx per thread.
template <typename T>
__global__ __launch_bounds__(256) void embed_bwd_kernel(int Trows, int H, int V, const int32_t* __restrict__ ids,
                                                        const T* __restrict__ dx, float* __restrict__ dE) {
  constexpr int VN = Vec<T>::N;
  __shared__ unsigned long long masks[4];
  const int t = blockIdx.x;
  const int id = ids[t];
  if (id < 0 || id >= V) return;
  int earlier = 0;
  for (int u = threadIdx.x; u < t; u += 256) earlier |= (ids[u] == id);
  if (__syncthreads_or(earlier)) return;
  for (int base = t; base < Trows; base += 256) {
    const int u = base + threadIdx.x;
    const unsigned long long mine = __ballot(u < Trows && ids[u] == id);
    if ((threadIdx.x & 63) == 0) masks[threadIdx.x >> 6] = mine;
    __syncthreads();
    if (masks[0] | masks[1] | masks[2] | masks[3]) {
      for (int c = threadIdx.x * VN; c < H; c += 256 * VN) {   // H is a multiple of the vector width
        float* e = dE + (int64_t)id * H + c;
        float s[VN];
#pragma unroll
        for (int i = 0; i < VN; ++i) s[i] = e[i];
        for (int w = 0; w < 4; ++w)
          for (unsigned long long m = masks[w]; m; m &= m - 1) {
            float d[VN];
            load_vec(dx + (int64_t)(base + 64 * w + __ffsll(m) - 1) * H + c, d);
#pragma unroll
            for (int i = 0; i < VN; ++i) s[i] += d[i];
          }
#pragma unroll
        for (int i = 0; i < VN; ++i) e[i] = s[i];
      }
    }
    __syncthreads();
  }
}
hipError_t embed_bwd(hipStream_t st, DType dt, int T, int H, int V, const int32_t* ids, const void* dx, float* dE) {
  if (dt == F32) hipLaunchKernelGGL(embed_bwd_kernel<float>, dim3(T), dim3(256), 0, st, T, H, V, ids, (const float*)dx, dE);
  else if (dt == BF16) hipLaunchKernelGGL(embed_bwd_kernel<bf16>, dim3(T), dim3(256), 0, st, T, H, V, ids, (const bf16*)dx, dE);
  else hipLaunchKernelGGL(embed_bwd_kernel<f16>, dim3(T), dim3(256), 0, st, T, H, V, ids, (const f16*)dx, dE);
  return hipGetLastError();
}

// ------------------------------------------------------------------ cross entropy
// One workgroup per row, two passes over the row (maximum, then sum of exponentials; the second pass hits in L2).
// VEC: 16-byte accesses (V and ldz multiples of the vector width, z 16-byte aligned), else element by element.
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void ce_fwd_kernel(int V, const T* __restrict__ z, int64_t ldz,
                                                     const int32_t* __restrict__ targets, float* __restrict__ lse,
                                                     float* __restrict__ rowloss, int32_t* __restrict__ keep) {
  constexpr int VN = Vec<T>::N;
  __shared__ float red[4];
  const int t = blockIdx.x;
  const T* zr = z + (int64_t)t * ldz;
  float mx = -INFINITY;
  if (VEC) {
    for (int c = threadIdx.x * VN; c < V; c += 256 * VN) {
      float a[VN];
      load_vec(zr + c, a);
#pragma unroll
      for (int i = 0; i < VN; ++i) mx = fmaxf(mx, a[i]);
    }
  } else {
    for (int c = threadIdx.x; c < V; c += 256) mx = fmaxf(mx, to_f(zr[c]));
  }
  mx = wave_max(mx);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  float s = 0.f;
  if (VEC) {
    for (int c = threadIdx.x * VN; c < V; c += 256 * VN) {
      float a[VN];
      load_vec(zr + c, a);
#pragma unroll
      for (int i = 0; i < VN; ++i) s += expf(a[i] - mx);
    }
  } else {
    for (int c = threadIdx.x; c < V; c += 256) s += expf(to_f(zr[c]) - mx);
  }
  s = block_sum<4>(s, red);
  if (threadIdx.x == 0) {
    const float l = mx + logf(s);
    const int tg = targets[t];
    if (keep) keep[t] = tg;
    lse[t] = l;
    rowloss[t] = (tg >= 0 && tg < V) ? l - to_f(zr[tg]) : 0.f;
  }
}
__global__ __launch_bounds__(256) void mean_kernel(int n, const float* __restrict__ v, float* __restrict__ out) {
  __shared__ float red[4];
  float s = 0.f;
  for (int i = threadIdx.x; i < n; i += 256) s += v[i];
  s = block_sum<4>(s, red);
  if (threadIdx.x == 0) *out = s / (float)n;
}
hipError_t ce_fwd(hipStream_t st, DType dt, int T, int V, const void* z, int64_t ldz, const int32_t* targets,
                  float* lse, float* rowloss, float* loss, int32_t* keep) {
  const int VN = dt == F32 ? 4 : 8;
  const bool vec = V % VN == 0 && ldz % VN == 0 && ((uintptr_t)z & 15) == 0;
#define CE_FWD(TT) \
  if (vec) hipLaunchKernelGGL((ce_fwd_kernel<TT, true>), dim3(T), dim3(256), 0, st, V, (const TT*)z, ldz, targets, lse, rowloss, keep); \
  else hipLaunchKernelGGL((ce_fwd_kernel<TT, false>), dim3(T), dim3(256), 0, st, V, (const TT*)z, ldz, targets, lse, rowloss, keep)
  if (dt == F32) { CE_FWD(float); } else if (dt == BF16) { CE_FWD(bf16); } else { CE_FWD(f16); }
#undef CE_FWD
  hipLaunchKernelGGL(mean_kernel, dim3(1), dim3(256), 0, st, T, rowloss, loss);
  return hipGetLastError();
}
// Rows on grid.x (no 65535 limit on the number of tokens), column blocks on grid.y.  VEC as for the forward kernel:
// a thread then owns one 16-byte vector of its row.  A row without a valid target has no loss term (ce_fwd gives it
// 0), hence no gradient.
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void ce_bwd_kernel(int V, T* z, int64_t ldz, const int32_t* __restrict__ targets,
                                                     const float* __restrict__ lse, float scale) {
  constexpr int VN = VEC ? Vec<T>::N : 1;
  const int t = blockIdx.x;
  const int c = (blockIdx.y * 256 + threadIdx.x) * VN;
  if (c >= V) return;
  T* p = z + (int64_t)t * ldz + c;
  const int tg = targets[t];
  const bool ok = tg >= 0 && tg < V;
  const float l = lse[t];
  if (VEC) {
    float a[Vec<T>::N], o[Vec<T>::N];
    load_vec(p, a);
#pragma unroll
    for (int i = 0; i < Vec<T>::N; ++i) o[i] = ok ? scale * (expf(a[i] - l) - (c + i == tg ? 1.f : 0.f)) : 0.f;
    store_vec(p, o);
  } else {
    *p = from_f<T>(ok ? scale * (expf(to_f(*p) - l) - (c == tg ? 1.f : 0.f)) : 0.f);
  }
}
hipError_t ce_bwd(hipStream_t st, DType dt, int T, int V, void* z, int64_t ldz, const int32_t* targets,
                  const float* lse, float scale) {
  const int VN = dt == F32 ? 4 : 8;
  const bool vec = V % VN == 0 && ldz % VN == 0 && ((uintptr_t)z & 15) == 0;
  dim3 grid((unsigned)T, (unsigned)cdiv(V, 256 * (vec ? VN : 1))), blk(256);
#define CE_BWD(TT) \
  if (vec) hipLaunchKernelGGL((ce_bwd_kernel<TT, true>), grid, blk, 0, st, V, (TT*)z, ldz, targets, lse, scale); \
  else hipLaunchKernelGGL((ce_bwd_kernel<TT, false>), grid, blk, 0, st, V, (TT*)z, ldz, targets, lse, scale)
  if (dt == F32) { CE_BWD(float); } else if (dt == BF16) { CE_BWD(bf16); } else { CE_BWD(f16); }
#undef CE_BWD
  return hipGetLastError();
}

// ------------------------------------------------------------------ AdamW
__device__ __forceinline__ float adamw_one(float p, float g, float& m, float& v, const AdamW& h) {
  g *= h.grad_scale;
  m = h.beta1 * m + (1.0f - h.beta1) * g;
  v = h.beta2 * v + (1.0f - h.beta2) * g * g;
  const float mhat = m * h.inv_bc1;
  const float vhat = v * h.inv_bc2;
  return p - h.lr * (mhat / (sqrtf(vhat) + h.eps) + h.wd * p);
}

// One float4 of p, g, m, v per lane; reads 16 B/element, writes 12 B (+2 B 16-bit copy; +4 B zeroed grad with h.zero_grad).
// VEC=false is the scalar variant for ranges that are not 16-byte aligned and for the tail.
// W is the element type of the working copy (float: params itself is the master).  With h.skip set and *h.skip
// non-zero (a non-finite gradient was found, loss-scaled fp16 training) nothing but the zeroing of grad happens.
template <typename W, bool VEC>
__global__ __launch_bounds__(256) void adamw_kernel(int64_t n, int64_t begin, void* params, float* master,
                                                    float* grad, float* m, float* v, AdamW h) {
  constexpr bool LOW = sizeof(W) == 2;
  typedef W W4 __attribute__((ext_vector_type(4)));
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * (VEC ? 4 : 1);
  if (i >= n) return;
  const bool skip = h.skip != nullptr && *h.skip != 0;
  float* pm = LOW ? master + i : (float*)params + begin + i;
  if (VEC) {
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    if (skip) {
      if (h.zero_grad) __builtin_nontemporal_store(zero, (f32x4*)(grad + begin + i));
      return;
    }
    // every byte is touched once per step: non-temporal accesses keep the streams out of the caches
    f32x4 p4 = __builtin_nontemporal_load((f32x4*)pm), g4 = __builtin_nontemporal_load((f32x4*)(grad + begin + i)),
          m4 = __builtin_nontemporal_load((f32x4*)(m + i)), v4 = __builtin_nontemporal_load((f32x4*)(v + i));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float mm = m4[k], vv = v4[k];
      p4[k] = adamw_one(p4[k], g4[k], mm, vv, h);
      m4[k] = mm;
      v4[k] = vv;
    }
    __builtin_nontemporal_store(p4, (f32x4*)pm);
    __builtin_nontemporal_store(m4, (f32x4*)(m + i));
    __builtin_nontemporal_store(v4, (f32x4*)(v + i));
    if (h.zero_grad) __builtin_nontemporal_store(zero, (f32x4*)(grad + begin + i));
    if (LOW) {
      // The working copy is the rounding of the STORED fp32 value.  Without the barrier the compiler folds the
      // update's last fused multiply-add and the conversion into one mixed-precision instruction that rounds the
      // exact result once, which differs from half(master) whenever the fp32 value lands on a tie.
      W4 b;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float q = p4[k];
        asm volatile("" : "+v"(q));
        b[k] = (W)q;
      }
      __builtin_nontemporal_store(b, (W4*)((W*)params + begin + i));
    }
  } else {
    if (skip) {
      if (h.zero_grad) grad[begin + i] = 0.f;
      return;
    }
    float mm = m[i], vv = v[i];
    const float pn = adamw_one(*pm, grad[begin + i], mm, vv, h);
    *pm = pn;
    m[i] = mm;
    v[i] = vv;
    if (h.zero_grad) grad[begin + i] = 0.f;
    if (LOW) {
      float q = pn;
      asm volatile("" : "+v"(q));   // as above: round the stored value
      ((W*)params)[begin + i] = (W)q;
    }
  }
}

hipError_t adamw(hipStream_t st, DType dt, int64_t n, int64_t begin, void* params, float* master, float* grad,
                 float* m, float* v, const AdamW& h) {
  if (n <= 0) return hipSuccess;
  const bool aligned = (begin % 4) == 0;   // then grad+begin, params+begin share the alignment of the shard arrays
  const int64_t nv = aligned ? (n / 4) * 4 : 0;
  if (nv > 0) {
    dim3 grid((unsigned)cdiv(nv / 4, 256)), blk(256);
    if (dt == BF16) hipLaunchKernelGGL((adamw_kernel<bf16, true>), grid, blk, 0, st, nv, begin, params, master, grad, m, v, h);
    else if (dt == F16) hipLaunchKernelGGL((adamw_kernel<f16, true>), grid, blk, 0, st, nv, begin, params, master, grad, m, v, h);
    else hipLaunchKernelGGL((adamw_kernel<float, true>), grid, blk, 0, st, nv, begin, params, master, grad, m, v, h);
  }
  if (n > nv) {
    const int64_t r = n - nv;
    dim3 grid((unsigned)cdiv(r, 256)), blk(256);
    if (dt == BF16)
      hipLaunchKernelGGL((adamw_kernel<bf16, false>), grid, blk, 0, st, r, begin + nv, params, master + nv, grad, m + nv, v + nv, h);
    else if (dt == F16)
      hipLaunchKernelGGL((adamw_kernel<f16, false>), grid, blk, 0, st, r, begin + nv, params, master + nv, grad, m + nv, v + nv, h);
    else
      hipLaunchKernelGGL((adamw_kernel<float, false>), grid, blk, 0, st, r, begin + nv, params, (float*)nullptr, grad, m + nv, v + nv, h);
  }
  return hipGetLastError();
}

// Sets *flag to 1 when any of g[0..n) is not finite (never clears it): the overflow test of loss-scaled training.
__global__ __launch_bounds__(256) void nonfinite_kernel(const float* __restrict__ g, int64_t n, int* __restrict__ flag) {
  bool bad = false;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const float x = g[i];
    bad |= !(fabsf(x) <= 3.402823466e38f);   // false for inf and for nan
  }
  if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(flag, 1);
}
hipError_t nonfinite_check(hipStream_t st, const float* g, int64_t n, int* flag) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = cdiv(n, 256 * 8);
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(nonfinite_kernel, dim3((unsigned)blocks), dim3(256), 0, st, g, n, flag);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void fill_zero_kernel(float* p, int64_t n) {
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i + 4 <= n) {
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    *(f32x4*)(p + i) = zero;
  } else {
    for (int64_t k = i; k < n; ++k) p[k] = 0.f;
  }
}
hipError_t fill_zero(hipStream_t st, float* p, int64_t n) {
  if (n <= 0) return hipSuccess;
  // peel so that the vector stores are 16-byte aligned
  int64_t head = ((16 - ((uintptr_t)p & 15)) & 15) / 4;
  if (head > n) head = n;
  if (head) hipLaunchKernelGGL(fill_zero_kernel, dim3(1), dim3(256), 0, st, p, head < 4 ? head : 3);
  p += head;
  n -= head;
  if (n > 0) hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)cdiv(cdiv(n, 4), 256)), dim3(256), 0, st, p, n);
  return hipGetLastError();
}

hipError_t copy_bytes(hipStream_t st, void* dst, const void* src, int64_t bytes) {
  return hipMemcpyAsync(dst, src, (size_t)bytes, hipMemcpyDeviceToDevice, st);
}

}  // namespace zs

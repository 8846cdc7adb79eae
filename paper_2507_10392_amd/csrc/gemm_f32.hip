// fp32 GEMM on the fp32 matrix cores (v_mfma_f32_16x16x4_f32: fp32 operands, fp32 accumulation), for the fp32 configuration.
//
// What bounds it: the fp32 products of this library are small (a microbatch of a small model), so the time is the latency of
// one pass over K on too few workgroups, not arithmetic.  Hence no LDS staging shared by waves and no barrier in the K loop: a wave
// loads its own operands from L2, 16 bytes per lane, and small outputs have their K range divided over the waves of a
// workgroup, whose partial tiles are added through LDS in a fixed order.
//
// How the operands fit without a transpose.  A 16x16x4 step takes from lane l one value of row l%16 at k = l/16.  Which
// memory row stands behind "row l%16" and which k behind "k = l/16" of step e is free as long as both operands agree on k:
//   k-contiguous operand (A [M,K], B [N,K]): lane l reads 4 consecutive k of its row; value e goes to step e, so step e of
//     a 16-wide slab multiplies k = 4 (l/16) + e.
//   row-contiguous operand (A [K,M], B [K,N]): lane l reads NV consecutive columns of row k = 4 (l/16) + e for e = 0..3;
//     value j goes to block j, so block j holds the columns NV (l%16) + j.
// The matrix instruction gets B as its first operand, so a lane ends up with 4 consecutive columns of one row of C.
//
// Measured on the GEMMs of a [256 tokens] x 256..1024 GPT stage: 47-86 us per launch with the plain LDS-tiled kernel,
// 3.4-6.5 us here.
#include "kernels.h"
#include "rows_lds.h"

namespace zs {
namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
constexpr unsigned OUT = 0x80000000u;   // pushes a lane's offset past every descriptor (extents are below 2^30 bytes): reads 0

template <int N> struct FV;
template <> struct FV<1> { typedef float type; };
template <> struct FV<2> { typedef f32x2 type; };
template <> struct FV<4> { typedef f32x4 type; };

__device__ __forceinline__ f32x4 load4(__amdgpu_buffer_rsrc_t rs, unsigned voff, unsigned soff) {
  union { u32x4 u; f32x4 f; } c;
  c.u = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)voff, (int)soff, 0);
  return c.f;
}
__device__ __forceinline__ f32x2 load2(__amdgpu_buffer_rsrc_t rs, unsigned voff, unsigned soff) {
  union { u32x2 u; f32x2 f; } c;
  c.u = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)voff, (int)soff, 0);
  return c.f;
}
template <int N> __device__ __forceinline__ typename FV<N>::type loadn(__amdgpu_buffer_rsrc_t rs, unsigned voff, unsigned soff) {
  if constexpr (N == 4) return load4(rs, voff, soff);
  else if constexpr (N == 2) return load2(rs, voff, soff);
  else return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)voff, (int)soff, 0));
}

// Fragments of one operand for one slab of 16 k: NB blocks of 16 rows.
template <int ROWC, int NB> struct Frag;
template <int NB> struct Frag<0, NB> {   // k-contiguous
  f32x4 v[NB];
  __device__ __forceinline__ float at(int b, int e) const { return v[b][e]; }
};
template <int NB> struct Frag<1, NB> {   // row-contiguous
  typename FV<NB>::type v[4];
  __device__ __forceinline__ float at(int b, int e) const {
    if constexpr (NB == 1) return v[e]; else return v[e][b];
  }
};

// Forms that share out K bring k-contiguous operands in through LDS, two slabs at a time (rows_lds.h), where through_lds says so: of the
// 5.9 us of 256 x 256, K = 1024 on 16x16 tiles direct loads of A alone were 1.7.  Two pairs of slabs are in flight on 64x64 and 32x32
// tiles, where more leave no second workgroup per CU (32x32: 369 x 1232, K = 176, 468 tiles 6.4 us with three, 5.2 with two; 64x64: two
// gain 8 to 15 % over one where CUs have one workgroup), three or four on smaller ones.  The sums and their order are those of the
// direct loads.  us, direct : through LDS: 256 x 512, K = 1536 (dx) 10.9 : 7.3; 256 x 256, K = 1024 6.1 : 4.4; 1024 x 1024, K = 1024 26.9 :
// 22.5; 0.88 on the geometric mean of 645 products.  128x128 tiles reach the matrix cores' rate without.
// A workgroup owns a (16 MI WM) x (16 NI WN) tile of C (MI, NI = 1, 2 or 4): WM x WN waves side by side, times KW waves
// that share out K.
// ACT: see Gemm::act; kernels of their own, because the branch alone costs the small products 0.5 %.
template <int TA, int TB, int MI, int NI, int WM, int WN, int KW, int SEG, int ACT = 0, bool LINES = (KW > 1)>
__device__ __forceinline__ void f32_tile(const Gemm& g, int tiles_m, int tiles_n, int pid, int z) {
  constexpr int NQ = MI * NI;   // quads of 4 consecutive columns a lane holds
  constexpr bool STAGED = LINES && (TA == 0 || TB == 1);   // k-contiguous operands through LDS
  constexpr int RED = KW > 1 ? (KW - 1) * WM * WN * NQ * 64 : 1, SA = STAGED && TA == 0 ? MI * 128 : 0, SB = STAGED && TB == 1 ? NI * 128 : 0;
  constexpr int STAGE = KW * WM * WN * (SA + SB);
  constexpr bool SHARED = (RED + STAGE) * 16 > 65536;       // partial tiles take the place of the slabs
  __shared__ f32x4 lds[SHARED ? (RED > STAGE ? RED : STAGE) : RED + STAGE];
  f32x4* red = lds + (SHARED ? 0 : STAGE);
  const int lane = threadIdx.x & 63, wave = STAGED ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : threadIdx.x >> 6;
  const int lm = lane & 15, lg = lane >> 4;
  const int kw = wave / (WM * WN), wt = wave % (WM * WN);
  int tm, tn;
  gemm_tile_of(pid, tiles_m, tiles_n, tm, tn);
  const int m0 = (tm * WM + wt / WN) * 16 * MI, n0 = (tn * WN + wt % WN) * 16 * NI;
  const float* A = (const float*)g.A + (int64_t)z * g.sA;
  const float* B = (const float*)g.B + (int64_t)z * g.sB;
  const unsigned lda = (unsigned)g.lda, ldb = (unsigned)g.ldb;
  const int nseg = SEG ? g.K / g.kseg : 1, kb = SEG ? g.kseg : g.K;
  const __amdgpu_buffer_rsrc_t ra =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(A), 0, (int)((TA ? (g.K - 1) * lda + g.M : (g.M - 1) * lda + g.K) * 4), 0x00020000);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(B), 0, (int)((TB ? (unsigned)((nseg - 1) * g.segB) + (g.N - 1) * ldb + kb : (g.K - 1) * ldb + g.N) * 4), 0x00020000);

  // per-lane byte offsets of the slab at k = 0
  unsigned ao[TA ? 4 : MI], bo[TB ? NI : 4];
  if constexpr (TA == 0) {
#pragma unroll
    for (int i = 0; i < MI; ++i) ao[i] = ((m0 + 16 * i + lm) * lda + 4 * lg) * 4;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) ao[e] = m0 + MI * lm < g.M ? ((4 * lg + e) * lda + m0 + MI * lm) * 4 : OUT;
  }
  if constexpr (TB == 1) {
#pragma unroll
    for (int j = 0; j < NI; ++j) bo[j] = ((n0 + 16 * j + lm) * ldb + (SEG ? 0 : 4 * lg)) * 4;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) bo[e] = n0 + NI * lm < g.N ? ((4 * lg + e) * ldb + n0 + NI * lm) * 4 : OUT;
  }

  Frag<TA, MI> fa[2];                                        // unless STAGED
  Frag<1 - TB, NI> fb[2];
  auto load = [&](Frag<TA, MI>& a, Frag<1 - TB, NI>& b, int k) {
    const unsigned past = k + 4 * lg < g.K ? 0u : OUT;   // K is a multiple of 4 where an operand is k-contiguous
    if constexpr (TA == 0) {
#pragma unroll
      for (int i = 0; i < MI; ++i) a.v[i] = load4(ra, ao[i] | past, k * 4);
    } else {   // rows past K lie behind the descriptor
#pragma unroll
      for (int e = 0; e < 4; ++e) a.v[e] = loadn<MI>(ra, ao[e], k * lda * 4);
    }
    if constexpr (TB == 1) {
      if constexpr (SEG) {
        const int kl = k + 4 * lg, seg = kl / g.kseg;
        const unsigned so = (unsigned)(seg * g.segB + (kl - seg * g.kseg)) * 4;
#pragma unroll
        for (int j = 0; j < NI; ++j) b.v[j] = load4(rb, past ? OUT : bo[j] + so, 0);
      } else {
#pragma unroll
        for (int j = 0; j < NI; ++j) b.v[j] = load4(rb, bo[j] | past, k * 4);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) b.v[e] = loadn<NI>(rb, bo[e], k * ldb * 4);
    }
  };
  f32x4 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](const Frag<TA, MI>& a, const Frag<1 - TB, NI>& b) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b.at(j, e), a.at(i, e), acc[i][j], 0, 0, 0);
  };

  const int slabs = (g.K + 15) / 16, per = (slabs + KW - 1) / KW;
  const int s0 = kw * per, s1 = min(slabs, s0 + per);        // this wave's slabs
  if constexpr (STAGED) {
    constexpr int DEPTH = MI * NI >= 4 ? 2 : MI * NI == 1 ? 4 : 3;
    u32x4* la = reinterpret_cast<u32x4*>(lds) + wave * (SA + SB);
    u32x4* lb = la + SA;
    struct Pair { Rows<SA ? MI : 1> a; Rows<SB ? NI : 1> b; Frag<1, TA ? MI : 1> ra[2]; Frag<1, TB ? 1 : NI> rb[2]; } buf[DEPTH];
    const unsigned ra0 = ((m0 + (lane >> 3)) * lda + 4 * (lane & 7)) * 4, rb0 = ((n0 + (lane >> 3)) * ldb + (SEG ? 0 : 4 * (lane & 7))) * 4;
    auto load_pair = [&](Pair& f, int s) {
      const int k = s * 16, kl = k + 4 * (lane & 7);
      const unsigned past = kl < min(g.K, s1 * 16) ? 0u : OUT; // K is a multiple of 4 where an operand is k-contiguous
      if constexpr (SA > 0) load_rows<MI>(f.a, ra, ra0 | past, lda * 4, k * 4);
      else {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) f.ra[h].v[e] = loadn<MI>(ra, ao[e], (k + 16 * h) * lda * 4);
      }
      if constexpr (SB > 0) {
        if constexpr (SEG) {
          const int seg = kl / g.kseg;
          load_rows<NI>(f.b, rb, past ? OUT : rb0 + (unsigned)(seg * g.segB + (kl - seg * g.kseg)) * 4, ldb * 4, 0);
        } else load_rows<NI>(f.b, rb, rb0 | past, ldb * 4, k * 4);
      } else {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) f.rb[h].v[e] = loadn<NI>(rb, bo[e], (k + 16 * h) * ldb * 4);
      }
    };
    auto multiply_pair = [&](Pair& f, int s) {
      constexpr bool TURN = MI * NI < 16;                    // 64x64: no registers for the fragments of both slabs, see turn_rows
      f32x4 a[2][TURN && SA ? MI : 1], b[2][TURN && SB ? NI : 1];
      if constexpr (TURN) {
        if constexpr (SB > 0) turn_rows<NI, 2>(b, f.b, lb, lane);
        if constexpr (SA > 0) turn_rows<MI, 2>(a, f.a, la, lane);
      } else {
        wave_lds_order();
        if constexpr (SA > 0) put_rows<MI>(f.a, la, lane);
        if constexpr (SB > 0) put_rows<NI>(f.b, lb, lane);
        wave_lds_order();
      }
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (s + h < s1) {
          Frag<TA, MI> fa;
          Frag<1 - TB, NI> fb;
          if constexpr (SA == 0) fa = f.ra[h];
          else if constexpr (TURN) __builtin_memcpy(fa.v, a[h], sizeof fa.v);
          else get_rows<MI>(fa.v, la, h, lane);
          if constexpr (SB == 0) fb = f.rb[h];
          else if constexpr (TURN) __builtin_memcpy(fb.v, b[h], sizeof fb.v);
          else get_rows<NI>(fb.v, lb, h, lane);
          multiply(fa, fb);
        }
    };
#pragma unroll
    for (int i = 0; i < DEPTH; ++i)
      if (s0 + 2 * i < s1) load_pair(buf[i], s0 + 2 * i);
    for (int s = s0; s < s1; s += 2 * DEPTH)
#pragma unroll
      for (int i = 0; i < DEPTH; ++i)
        if (s + 2 * i < s1) {
          multiply_pair(buf[i], s + 2 * i);
          if (s + 2 * (i + DEPTH) < s1) load_pair(buf[i], s + 2 * (i + DEPTH));
        }
    if constexpr (SHARED) __syncthreads();
  } else if (s0 < s1) {   // two slabs in flight; loads behind s1 are issued and not used
    load(fa[0], fb[0], s0 * 16);
    for (int s = s0; s < s1; s += 2) {
      load(fa[1], fb[1], (s + 1) * 16);
      multiply(fa[0], fb[0]);
      if (s + 1 < s1) {
        load(fa[0], fb[0], (s + 2) * 16);
        multiply(fa[1], fb[1]);
      }
    }
  }

  // A lane's quads: quad (i, q) is row m(i), columns n(q) .. n(q)+3.
  auto row_of = [&](int i) { return m0 + (TA ? MI * lm + i : 16 * i + lm); };
  auto col_of = [&](int q) { return n0 + (TB ? 16 * q + 4 * lg : 4 * NI * lg + 4 * q); };
  auto quad = [&](int i, int q) {
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (TB) v[e] = acc[i][q][e];
      else v[e] = acc[i][(4 * q + e) % NI][(4 * q + e) / NI];   // column NI (4 lg + r) + j  <->  block j, register r
    }
    return v;
  };
  const float* bias = g.bias ? (const float*)g.bias + (int64_t)z * g.sBias : nullptr;
  const float* R = g.resid ? (const float*)g.resid + (int64_t)z * g.sC : nullptr;
  const bool rot = g.rope && z < g.rope_batches;
  float* C = (float*)g.C + (int64_t)z * g.sC;
  auto store = [&](f32x4 v, int m, int n) {
    if (m >= g.M || n >= g.N) return;   // N is a multiple of 4
    f32x4* pc = reinterpret_cast<f32x4*>(C + (int64_t)m * g.ldc + n);
    if (bias) v += *reinterpret_cast<const f32x4*>(bias + n);
    if (R) v += *reinterpret_cast<const f32x4*>(R + (int64_t)m * g.ldr + n);
    if (rot) {
      const f32x4 t = *reinterpret_cast<const f32x4*>(g.rope + (int64_t)(m % g.rope_S) * (g.rope_d / 2) + (n % g.rope_d) / 2);
      v = f32x4{v[0] * t[0] - v[1] * t[1], v[0] * t[1] + v[1] * t[0], v[2] * t[2] - v[3] * t[3], v[2] * t[3] + v[3] * t[2]};
    }
    if constexpr (ACT != 0) {
      f32x4* pz = reinterpret_cast<f32x4*>((float*)g.act_z + (int64_t)m * g.ldc + n);
      f32x4 a;
      if constexpr (ACT == 2) {
        const f32x4 zz = *pz;
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = v[e] * gelu_df(zz[e]);
      } else {
        *pc = v;
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = gelu_f(v[e]);
      }
      *pz = a;
      return;
    }
    *pc = g.c_f32_accum ? *pc + v : v;
  };
  if constexpr (KW == 1) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int q = 0; q < NI; ++q) store(quad(i, q), row_of(i), col_of(q));
  } else {
    // quad s of the tile is stored by the wave kw = s % KW; the others leave theirs in LDS, and it adds them in the order of kw
    constexpr int NW = WM * WN;
#pragma unroll
    for (int s = 0; s < NQ; ++s)
      if (s % KW != kw) red[(((kw < s % KW ? kw : kw - 1) * NW + wt) * NQ + s) * 64 + lane] = quad(s / NI, s % NI);
    __syncthreads();
#pragma unroll
    for (int s = 0; s < NQ; ++s)
      if (s % KW == kw) {
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int o = 0; o < KW; ++o)
          v += o == kw ? quad(s / NI, s % NI) : red[(((o < kw ? o : o - 1) * NW + wt) * NQ + s) * 64 + lane];
        store(v, row_of(s / NI), col_of(s % NI));
      }
  }
}

template <int TA, int TB, int MI, int NI, int WM, int WN, int KW, int SEG, int ACT, bool LINES>
__global__ __launch_bounds__(64 * WM * WN * KW) void gemm_f32_kernel(Gemm g, int tiles_m, int tiles_n) {
  f32_tile<TA, TB, MI, NI, WM, WN, KW, SEG, ACT, LINES>(g, tiles_m, tiles_n, blockIdx.x, blockIdx.y);
}
// Weight gradients of a layer in one launch (see gemm_group).
template <int MI, int NI, int WM, int WN, int KW> __global__ __launch_bounds__(64 * WM * WN * KW) void gemm_f32_group_kernel(GemmGroup q) {
  int tiles_m, tiles_n, pid, z;
  const Gemm g = q.product_of(blockIdx.x, tiles_m, tiles_n, pid, z);
  f32_tile<1, 0, MI, NI, WM, WN, KW, 0>(g, tiles_m, tiles_n, pid, z);
}

template <int MI, int NI, int WM, int WN, int KW> hipError_t launch_group(hipStream_t st, const Gemm* g, int n) {
  GemmGroup q(g, n, 16 * MI * WM, 16 * NI * WN);
  hipLaunchKernelGGL((gemm_f32_group_kernel<MI, NI, WM, WN, KW>), dim3((unsigned)q.total), dim3(64 * WM * WN * KW), 0, st, q);
  return hipGetLastError();
}

template <int MI, int NI, int WM, int WN, int KW, bool LINES> hipError_t launch_kernel(hipStream_t st, const Gemm& g) {
  const int tm = (int)cdiv(g.M, 16 * MI * WM), tn = (int)cdiv(g.N, 16 * NI * WN);
  dim3 grid((unsigned)(tm * tn), (unsigned)g.batch), blk(64 * WM * WN * KW);
  if (g.act == 1) hipLaunchKernelGGL((gemm_f32_kernel<0, 0, MI, NI, WM, WN, KW, 0, 1, LINES>), grid, blk, 0, st, g, tm, tn);
  else if (g.act) hipLaunchKernelGGL((gemm_f32_kernel<0, 1, MI, NI, WM, WN, KW, 0, 2, LINES>), grid, blk, 0, st, g, tm, tn);
  else if (g.kseg) hipLaunchKernelGGL((gemm_f32_kernel<0, 1, MI, NI, WM, WN, KW, 1, 0, LINES>), grid, blk, 0, st, g, tm, tn);
  else if (!g.transA && !g.transB) hipLaunchKernelGGL((gemm_f32_kernel<0, 0, MI, NI, WM, WN, KW, 0, 0, LINES>), grid, blk, 0, st, g, tm, tn);
  else if (!g.transA) hipLaunchKernelGGL((gemm_f32_kernel<0, 1, MI, NI, WM, WN, KW, 0, 0, LINES>), grid, blk, 0, st, g, tm, tn);
  else if (!g.transB) hipLaunchKernelGGL((gemm_f32_kernel<1, 0, MI, NI, WM, WN, KW, 0, 0, false>), grid, blk, 0, st, g, tm, tn);
  else hipLaunchKernelGGL((gemm_f32_kernel<1, 1, MI, NI, WM, WN, KW, 0, 0, LINES>), grid, blk, 0, st, g, tm, tn);
  return hipGetLastError();
}
// Through LDS or direct.  A short K has nothing to run beside the way round.  Where rows are not whole lines, so that a piece of 128 bytes lies in
// two, forward products on 16x32 tiles gain nothing once W no longer fits an XCD's L2, and input gradients on 32x32 tiles lose if their
// waves' shares end in half a pair of slabs and are short.  us, through LDS : direct: 66 x 208, K = 56 (dx) 2.56 : 2.35; 256 x 128, K = 128
// 2.83 : 2.70; 128 x 1024, K = 2768 17.7 : 16.3, but 221 x 304, K = 1224 6.4 : 7.5; 512 x 512, K = 1384 (dx, 11 slabs a wave) 11.7 : 10.9,
// but 266 x 888, K = 216 (dx, 2 slabs) 4.0 : 4.4 and 269 x 624, K = 3728 (30 slabs) 23.8 : 25.8.
template <int MI, int NI, int KW> bool through_lds(const Gemm& g) {
  if (g.K <= (MI * NI == 1 ? 128 : 64)) return false;
  if ((g.transA || g.lda % 32 == 0) && (!g.transB || g.ldb % 32 == 0)) return true;
  const int64_t share = cdiv(cdiv(g.K, 16), KW);
  if (g.transB) return MI * NI != 4 || share % 2 == 0 || share > 12;
  return MI * NI != 2 || (int64_t)g.K * g.N * 4 < (4 << 20);
}
template <int MI, int NI, int WM, int WN, int KW> hipError_t launch(hipStream_t st, const Gemm& g) {
  if constexpr (KW > 1)
    if (through_lds<MI, NI, KW>(g)) return launch_kernel<MI, NI, WM, WN, KW, true>(st, g);
  return launch_kernel<MI, NI, WM, WN, KW, false>(st, g);
}

}  // namespace

// 16-byte loads and stores: aligned bases, strides and extents that are multiples of 4 (K only where an operand is
// k-contiguous), and 32-bit byte offsets with room for a tile's overhang and the out-of-range push.
bool gemm_f32_supported(const Gemm& g) {
  auto al = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  if (g.M < 1 || g.N < 1 || g.K < 1 || g.batch < 1 || g.batch > 65535 || g.nx || g.glu) return false;
  if (!al(g.A) || !al(g.B) || !al(g.C) || g.lda % 4 || g.ldb % 4 || g.ldc % 4 || g.sA % 4 || g.sB % 4 || g.sC % 4) return false;
  if (g.N % 4 || (g.transA && g.M % 4) || ((!g.transA || g.transB) && g.K % 4)) return false;
  if (g.lda < (g.transA ? g.M : g.K) || g.ldc < g.N) return false;
  if (g.bias && (!al(g.bias) || g.sBias % 4)) return false;
  if (g.resid && (!al(g.resid) || g.ldr % 4)) return false;
  if (g.rope && (!al(g.rope) || g.rope_d % 4 || g.rope_S < 1 || g.c_f32_accum)) return false;
  if (g.kseg && (g.transA || !g.transB || g.kseg < 4 || g.kseg % 4 || g.segB % 4 || g.segB < 0 || g.K % g.kseg)) return false;
  if (g.ldb < (!g.transB ? g.N : g.kseg ? g.kseg : g.K)) return false;
  const int64_t rowsA = (g.transA ? g.K : g.M) + 160, rowsB = (g.transB ? g.N : g.K) + 160;   // a tile and two slabs over the end
  const int64_t segs = g.kseg ? (g.K / g.kseg - 1) * g.segB : 0;
  if (g.act && (g.batch != 1 || g.transA || g.kseg || g.rope || g.c_f32_accum || g.act != 1 + g.transB || ((uintptr_t)g.act_z & 15))) return false;
  return rowsA * g.lda * 4 < (1ll << 30) && (rowsB * g.ldb + segs) * 4 < (1ll << 30);
}

// Which tile: 128x128 (4 waves of 64x64), 64x64 with K over 4 waves, or 32x32, 16x32 or 16x16 with K over 8 waves.  The smaller
// ones exist for outputs that give the 256 CUs too few workgroups; the fewer outputs a wave has the more bytes it loads per
// flop.  The estimate: cycles of the busiest CU, at the 256 flops per cycle of its four matrix cores times what each form was
// measured to reach of it, plus a fixed part per workgroup.  With direct loads throughout, 256 x 256, K = 1024: 9.6 us on 32x32, 7.0 on 16x32, 5.9 on
// 16x16; 256 x 512, K = 2752 in two segments 25.1, 19.3 and 24.2; 256 x 1024, K = 256 4.9, 5.5 and 6.1; 64x64 9.4.
namespace {
const struct { int m, n; double share; } FORMS[5] = {{128, 128, 0.8}, {64, 64, 0.7}, {32, 32, 0.45}, {16, 32, 0.4}, {16, 16, 0.3}};

int pick_form(const Gemm& g, double& cycles) {
  int best = 0;
  for (int i = 0; i < 5; ++i) {
    const int64_t wgs = cdiv(g.M, FORMS[i].m) * cdiv(g.N, FORMS[i].n) * g.batch;
    const double t = (double)cdiv(wgs, 256) * (2.0 * FORMS[i].m * FORMS[i].n * (double)g.K / (256.0 * FORMS[i].share) + 1500.0);
    if (i == 0 || t < cycles) { best = i; cycles = t; }
  }
  return best;
}
}  // namespace

hipError_t gemm_f32(hipStream_t st, const Gemm& g) {
  double cycles;
  switch (pick_form(g, cycles)) {
    case 0: return launch<4, 4, 2, 2, 1>(st, g);
    case 1: return launch<4, 4, 1, 1, 4>(st, g);
    case 2: return launch<2, 2, 1, 1, 8>(st, g);
    case 3: return launch<1, 2, 1, 1, 8>(st, g);
    default: return launch<1, 1, 1, 1, 8>(st, g);
  }
}

// Whether a layer's weight gradients are faster together.  On their own they leave CUs idle in the last round of each and pay a fixed part per
// workgroup: what that costs is the estimate above over the same products at the big tile's rate without remainders.  Together
// they run on small tiles, which load three times the big tile's bytes per flop, and that weighs the more the larger the work is.
// The line is fitted to 121 layers of hidden 128 to 5056 and 16 to 4096 tokens that ran both ways, of which it loses 1.1 % at most.
// us per microbatch of one layer, forward and backward, one after the other : grouped: GPT, hidden 4096, 256 tokens 3506 : 3597, 1024
// tokens 11734 : 12451; Llama, hidden 4928, 1170 tokens 12612 : 13193; GPT, hidden 2048, 2048 tokens 6492 : 6573, 512 tokens 1828 : 1807; Llama,
// hidden 2048, 2048 tokens 7003 : 6820.
bool gemm_f32_group_pays(const Gemm* g, int n) {
  double own = 0.0, macs = 0.0;
  for (int i = 0; i < n; ++i) {
    double cycles;
    pick_form(g[i], cycles);
    own += cycles;
    macs += (double)g[i].M * g[i].N * g[i].K * g[i].batch;
  }
  return own > 2.0 * macs / (256.0 * 256.0 * FORMS[0].share) * (1.01 + macs / 1.6e12);
}

// 32x64 tiles: together the products fill the chip, and several workgroups on a CU cover one another's loads, merges and stores.
// K over 8 waves keeps the chains of additions, and the error against 64 bits, as short as the products' own tiles do; from about
// eight workgroups per CU on, where those take fewer waves as well, over 4.  us per microbatch of one layer, forward and backward,
// one after the other, and grouped with 8 waves and with 4: GPT, 256 tokens, hidden 256 116 -> 100, 100; Llama, 256 tokens, hidden 512
// 206 -> 189, 186; GPT, 256 tokens, hidden 1024 391 -> 370, 357; hidden 2048 1131 -> 1138, 1083.  64x64 tiles take 103, 191 and 362, 32x32
// tiles 98, 186 and 359 for the first three.
hipError_t gemm_f32_group(hipStream_t st, const Gemm* g, int n) {
  int64_t blocks = 0;
  for (int i = 0; i < n; ++i) blocks += cdiv(g[i].M, 32) * cdiv(g[i].N, 64) * g[i].batch;
  return blocks <= 2048 ? launch_group<2, 4, 1, 1, 8>(st, g, n) : launch_group<2, 4, 1, 1, 4>(st, g, n);
}

}  // namespace zs

// 16-bit GEMM for outputs too small to fill the chip with 128x128 tiles (bf16 / IEEE half operands, fp32 accumulation).
//
// What bounds such a product is the walk over K on few workgroups: with 128x128 tiles a 256 x 512 output has 8 of them, and
// 248 CUs watch.  Here a workgroup owns 32x32 or 64x64 outputs, its waves share out K and add their partial tiles through LDS
// in a fixed order, and every wave loads its own operands from L2: no barrier in the K loop, several slabs of 32 k in flight.
// The price is L2 traffic (a wave re-reads what a neighbour has read), so outputs that fill the chip stay with the staged
// kernels.  The rule stands with gemm_small_tile.
//
// How the operands fit without an LDS transpose.  A 16x16x32 step takes from lane l eight values of row l%16; which k stand
// behind them is free as long as both operands agree: k = 8 (l/16) + 0..7 of the slab.
//   k-contiguous operand (A [M,K], B [N,K]): 16 bytes per lane and block of 16 rows.  Input gradients, where both operands are, get
//     them through LDS of the wave's own (rows_lds.h): with one direct load per fragment the address unit was the limit.  us,
//     direct : through LDS, 64 x 768, K = 3072 12.8 : 6.9; 384 x 1024, K = 4096 30.3 : 15.8; 512 x 512, K = 512 4.2 : 3.7; 0.76 on the
//     geometric mean of 96 products with 64 to 1000 rows, K = 256 .. 4096.
//   row-contiguous operand (A [K,M], B [K,N]): lane l loads NV consecutive columns of each of its eight k-lines; pairs of
//     k-lines are then interleaved by one v_perm_b32 per register, which leaves in NV fragments the columns NV (l%16) + j.
// The matrix instruction gets B as its first operand, so a lane ends up with 4 consecutive columns of one row of C.
#include "kernels.h"
#include "rows_lds.h"

#include <algorithm>
#include <cmath>

namespace zs {
namespace {

constexpr unsigned OUT = 0x80000000u;   // pushes a lane's offset past every descriptor (extents are below 2^30 bytes): reads 0
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* p, int64_t elements) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)(elements * 2), 0x00020000);
}
template <typename E> __device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c);
template <> __device__ __forceinline__ f32x4 mfma<bf16>(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
template <> __device__ __forceinline__ f32x4 mfma<f16>(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// One operand's share of a slab of 32 k, NB blocks of 16 rows, as loaded.
template <int ROWC, int NB> struct Raw;
template <int NB> struct Raw<0, NB> {   // k-contiguous
  u32x4 v[NB];
  __device__ __forceinline__ u32x4 frag(int b) const { return v[b]; }
};
template <> struct Raw<1, 4> {          // row-contiguous, 4 columns of 8 k-lines
  u32x2 v[8];
  __device__ __forceinline__ u32x4 frag(int b) const {
    u32x4 f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      f[i] = __builtin_amdgcn_perm(v[2 * i + 1][b >> 1], v[2 * i][b >> 1], b & 1 ? 0x07060302u : 0x05040100u);
    return f;
  }
};
template <> struct Raw<1, 2> {          // row-contiguous, 2 columns of 8 k-lines
  unsigned v[8];
  __device__ __forceinline__ u32x4 frag(int b) const {
    u32x4 f;
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = __builtin_amdgcn_perm(v[2 * i + 1], v[2 * i], b & 1 ? 0x07060302u : 0x05040100u);
    return f;
  }
};
template <int NB> __device__ __forceinline__ void load_k(Raw<0, NB>& f, __amdgpu_buffer_rsrc_t rs, const unsigned (&at)[NB], unsigned add, unsigned soff) {
#pragma unroll
  for (int b = 0; b < NB; ++b) f.v[b] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(add == OUT ? OUT : at[b] + add), (int)soff, 0);
}
// at: byte offset of the lane's columns in its first k-line (OUT for columns past the end), ld2: bytes of a k-line
__device__ __forceinline__ void load_r(Raw<1, 4>& f, __amdgpu_buffer_rsrc_t rs, unsigned at, unsigned ld2, unsigned soff) {
#pragma unroll
  for (int i = 0; i < 8; ++i) f.v[i] = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)(at + i * ld2), (int)soff, 0);
}
__device__ __forceinline__ void load_r(Raw<1, 2>& f, __amdgpu_buffer_rsrc_t rs, unsigned at, unsigned ld2, unsigned soff) {
#pragma unroll
  for (int i = 0; i < 8; ++i) f.v[i] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(at + i * ld2), (int)soff, 0);
}

enum Form { NN, NT, NT_SEG, TN_ACC, TN_PARTS, NN_GLU, NT_GLU };

// T: blocks of 16 rows and columns a wave's tile has each way (2: 32x32, 4: 64x64), KW: waves that share out K, NBUF: slabs
// held (NBUF - 1 of them in flight).  NN_GLU: the tile has two blocks of 16 columns of each of the two projections.
template <typename E, int FORM, int T, int KW, int NBUF>
__device__ __forceinline__ void small_tile(const Gemm& g, int tiles_m, int tiles_n, int pid, int z) {
  constexpr int TA = FORM == TN_ACC || FORM == TN_PARTS, TB = FORM == NT || FORM == NT_SEG || FORM == NT_GLU;
  constexpr bool GLU1 = FORM == NN_GLU, ACC = TA;
  constexpr int NB = GLU1 ? 2 : T;                 // blocks of columns of one matrix B
  constexpr int NJ = GLU1 ? 2 * NB : NB;           // ... of the tile
  constexpr int NQ = T * NJ;                       // quads of 4 consecutive columns a lane holds
  constexpr bool STAGED = TB && KW > 1;            // both operands k-contiguous: through LDS
  constexpr int RED = KW > 1 ? (KW - 1) * NQ * 64 : 1, STAGE = STAGED ? KW * 2 * T * 128 : 0;
  __shared__ f32x4 red[RED > STAGE ? RED : STAGE]; // partial tiles take the place of the slabs
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lm = lane & 15, lg = lane >> 4;
  // ids are dealt round-robin to the 8 XCDs; each gets a contiguous run of the tile order
  const int ntiles = tiles_m * tiles_n;
  int tm, tn;
  if (pid < ntiles / 8 * 8) pid = (pid % 8) * (ntiles / 8) + pid / 8;
  gemm_tile_of(pid, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * 16 * T, n0 = tn * 16 * NB;
  const E* A = (const E*)g.A + (int64_t)z * g.sA;
  const E* B = (const E*)g.B + (int64_t)z * g.sB;
  const unsigned lda = (unsigned)g.lda, ldb = (unsigned)g.ldb;
  const int K1 = FORM == TN_PARTS ? g.kseg : g.K;   // rows of a part, or of the only one
  const int64_t recB = TB ? (FORM == NT_SEG ? (int64_t)(g.K / g.kseg - 1) * g.segB + (int64_t)(g.N - 1) * ldb + g.kseg : (int64_t)(g.N - 1) * ldb + g.K)
                          : (int64_t)(K1 - 1) * ldb + g.N + (GLU1 ? g.sB : 0);
  const __amdgpu_buffer_rsrc_t ra = rsrc(A, TA ? (int64_t)(K1 - 1) * lda + g.M : (int64_t)(g.M - 1) * lda + g.K), rb = rsrc(B, recB);

  unsigned ao[TA ? 1 : T], bo[TB ? NB : 1], bo2 = OUT;
  if constexpr (TA) ao[0] = m0 + T * lm < g.M ? (8 * lg * lda + m0 + T * lm) * 2 : OUT;
  else {
#pragma unroll
    for (int i = 0; i < T; ++i) ao[i] = ((m0 + 16 * i + lm) * lda + 8 * lg) * 2;
  }
  if constexpr (TB) {
#pragma unroll
    for (int j = 0; j < NB; ++j) bo[j] = ((n0 + 16 * j + lm) * ldb + (FORM == NT_SEG ? 0 : 8 * lg)) * 2;
  } else {
    bo[0] = n0 + NB * lm < g.N ? (8 * lg * ldb + n0 + NB * lm) * 2 : OUT;
    if (GLU1 && bo[0] != OUT) bo2 = bo[0] + (unsigned)g.sB * 2;
  }

  f32x4 acc[T][NJ];
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int slabs = (g.K + 31) / 32, per = (slabs + KW - 1) / KW;
  const int s0 = wave * per, s1 = min(slabs, s0 + per);   // this wave's slabs
  if constexpr (STAGED) {
    // Two pairs of slabs in flight, three on 32x32 tiles.  The fragments hold the same k as with direct loads.
    constexpr int DEPTH = T == 2 ? 3 : 2;
    u32x4* la = reinterpret_cast<u32x4*>(red) + wave * 2 * T * 128;
    u32x4* lb = la + T * 128;
    struct Pair { Rows<T> a, b; } pairs[DEPTH];
    const unsigned a0 = ((m0 + (lane >> 3)) * lda + 8 * (lane & 7)) * 2, b0 = ((n0 + (lane >> 3)) * ldb + (FORM == NT_SEG ? 0 : 8 * (lane & 7))) * 2;
    auto load = [&](Pair& f, int s) {
      const int k = s * 32, kl = k + 8 * (lane & 7);
      const bool past = kl >= min(g.K, s1 * 32);           // K is a multiple of 8 where an operand is k-contiguous
      load_rows<T>(f.a, ra, past ? OUT : a0, lda * 2, k * 2);
      if constexpr (FORM == NT_SEG) {
        const int seg = kl / g.kseg;
        load_rows<T>(f.b, rb, past ? OUT : b0 + (unsigned)(seg * g.segB + (kl - seg * g.kseg)) * 2, ldb * 2, 0);
      } else load_rows<T>(f.b, rb, past ? OUT : b0, ldb * 2, k * 2);
    };
#pragma unroll
    for (int i = 0; i < DEPTH; ++i)
      if (s0 + 2 * i < s1) load(pairs[i], s0 + 2 * i);
    for (int s = s0; s < s1; s += 2 * DEPTH)
#pragma unroll
      for (int i = 0; i < DEPTH; ++i)
        if (s + 2 * i < s1) {
          put_rows<T>(pairs[i].a, la, lane);
          put_rows<T>(pairs[i].b, lb, lane);
          if (s + 2 * (i + DEPTH) < s1) load(pairs[i], s + 2 * (i + DEPTH));
#pragma unroll
          for (int h = 0; h < 2; ++h)
            if (s + 2 * i + h < s1) {
              u32x4 a[T], b[T];
              get_rows<T>(a, la, h, lane);
              get_rows<T>(b, lb, h, lane);
#pragma unroll
              for (int j = 0; j < T; ++j)
#pragma unroll
                for (int q = 0; q < T; ++q) acc[q][j] = mfma<E>(b[j], a[q], acc[q][j]);
            }
        }
    __syncthreads();
  } else {
    struct Slab { Raw<TA, T> a; Raw<1 - TB, NB> b, b2; };
    Slab buf[NBUF];
    auto load = [&](Slab& s, int slab) {
      const int k = slab * 32;
      const unsigned past = k + 8 * lg < g.K ? 0u : OUT;   // K is a multiple of 8 where an operand is k-contiguous
      if constexpr (FORM == TN_PARTS) {   // slabs do not straddle parts: kseg is a multiple of 128
        const int p = min(k / g.kseg, g.nx), kin = k - p * g.kseg;
        const int rows = p < g.nx ? g.kseg : g.K - g.nx * g.kseg;
        const __amdgpu_buffer_rsrc_t pa = rsrc((p ? (const E*)g.Ax[p - 1] : (const E*)g.A) + (int64_t)z * g.sA, (int64_t)(rows - 1) * lda + g.M),
                                     pb = rsrc((p ? (const E*)g.Bx[p - 1] : (const E*)g.B) + (int64_t)z * g.sB, (int64_t)(rows - 1) * ldb + g.N);
        load_r(s.a, pa, ao[0], lda * 2, kin * lda * 2);
        load_r(s.b, pb, bo[0], ldb * 2, kin * ldb * 2);
        return;
      }
      if constexpr (TA) load_r(s.a, ra, ao[0], lda * 2, k * lda * 2);   // k-lines past K lie behind the descriptor
      else load_k<T>(s.a, ra, ao, past, k * 2);
      if constexpr (FORM == NT_SEG) {
        const int kl = k + 8 * lg, seg = kl / g.kseg;
        load_k<NB>(s.b, rb, bo, past ? OUT : (unsigned)(seg * g.segB + (kl - seg * g.kseg)) * 2, 0);
      } else if constexpr (TB) {
        load_k<NB>(s.b, rb, bo, past, k * 2);
      } else {
        load_r(s.b, rb, bo[0], ldb * 2, k * ldb * 2);
        if constexpr (GLU1) load_r(s.b2, rb, bo2, ldb * 2, k * ldb * 2);
      }
    };
    auto multiply = [&](const Slab& s) {
      u32x4 a[T];
#pragma unroll
      for (int i = 0; i < T; ++i) a[i] = s.a.frag(i);
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const u32x4 b = GLU1 && j >= NB ? s.b2.frag(j % NB) : s.b.frag(j % NB);
#pragma unroll
        for (int i = 0; i < T; ++i) acc[i][j] = mfma<E>(b, a[i], acc[i][j]);
      }
    };

#pragma unroll
    for (int i = 0; i < NBUF - 1; ++i)
      if (s0 + i < s1) load(buf[i], s0 + i);
    for (int s = s0; s < s1; s += NBUF)
#pragma unroll
      for (int i = 0; i < NBUF; ++i)
        if (s + i < s1) {
          if (s + i + NBUF - 1 < s1) load(buf[(i + NBUF - 1) % NBUF], s + i + NBUF - 1);
          multiply(buf[i]);
        }
  }

  // A lane's quads: quad (i, q) is row m(i), columns n(q) .. n(q)+3 (NN_GLU: quads NB.. are the up columns).
  auto quad = [&](int i, int q) {
    const int base = q / NB * NB, ql = q % NB;
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (TB) v[e] = acc[i][q][e];
      else v[e] = acc[i][base + (4 * ql + e) % NB][(4 * ql + e) / NB];   // column NB (4 lg + r) + j  <->  block j, register r
    }
    return v;
  };
  // quad s is finished by the wave s % KW; the others leave theirs in LDS, and it adds them in the order of the waves
#pragma unroll
  for (int s = 0; s < NQ; ++s)
    if (KW > 1 && s % KW != wave) red[((wave < s % KW ? wave : wave - 1) * NQ + s) * 64 + lane] = quad(s / NJ, s % NJ);
  if (KW > 1) __syncthreads();
  auto sum = [&](int s) {
    if (KW == 1) return quad(s / NJ, s % NJ);
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int o = 0; o < KW; ++o) v += o == s % KW ? quad(s / NJ, s % NJ) : red[((o < s % KW ? o : o - 1) * NQ + s) * 64 + lane];
    return v;
  };
  typedef E E4 __attribute__((ext_vector_type(4)));
  auto row_of = [&](int i) { return m0 + (TA ? T * lm + i : 16 * i + lm); };
  auto col_of = [&](int q) { return n0 + (TB ? 16 * q + 4 * lg : 4 * NB * lg + 4 * q); };
  if constexpr (GLU1) {
    static_assert(KW == 1, "a lane holds the gate and the up quad of the same columns");
#pragma unroll
    for (int s = 0; s < NQ; ++s)
      if (s % NJ < NB) {
        const f32x4 gv = quad(s / NJ, s % NJ), uv = quad(s / NJ, s % NJ + NB);
        const int m = row_of(s / NJ), n = col_of(s % NJ);
        if (m >= g.M || n >= g.N) continue;
        E4 og, ou, oa;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          og[e] = (E)gv[e];
          ou[e] = (E)uv[e];
          oa[e] = (E)glu_f((float)og[e], (float)ou[e]);
        }
        E* pg = (E*)g.gu + (int64_t)m * g.gu_ld + n;
        *reinterpret_cast<E4*>(pg) = og;
        *reinterpret_cast<E4*>(pg + g.gu_up) = ou;
        *reinterpret_cast<E4*>((E*)g.C + (int64_t)m * g.ldc + n) = oa;
      }
    return;
  }
  const E* bias = g.bias ? (const E*)g.bias + (int64_t)z * g.sBias : nullptr;
  const E* R = g.resid ? (const E*)g.resid + (int64_t)z * g.sC : nullptr;
  const bool rot = g.rope && z < g.rope_batches;
#pragma unroll
  for (int s = 0; s < NQ; ++s)
    if (s % KW == wave) {
      const int m = row_of(s / NJ), n = col_of(s % NJ);
      if (m >= g.M || n >= g.N) continue;              // N is a multiple of 4
      f32x4 v = sum(s);
      if constexpr (ACC) {
        f32x4* pc = reinterpret_cast<f32x4*>((float*)g.C + (int64_t)z * g.sC + (int64_t)m * g.ldc + n);
        *pc = *pc + v;
        continue;
      }
      E4 o;
      if constexpr (FORM == NT_GLU) {                  // v is da: (gate, up) of these columns become (dgate, dup) in place
        E* pg = (E*)g.gu + (int64_t)m * g.gu_ld + n;
        const E4 gg = *reinterpret_cast<const E4*>(pg), uu = *reinterpret_cast<const E4*>(pg + g.gu_up);
        E4 ou;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float dg, du;
          glu_df(v[e], (float)gg[e], (float)uu[e], dg, du);
          o[e] = (E)dg;
          ou[e] = (E)du;
        }
        *reinterpret_cast<E4*>(pg) = o;
        *reinterpret_cast<E4*>(pg + g.gu_up) = ou;
        continue;
      }
      if (bias) {
        const E4 bb = *reinterpret_cast<const E4*>(bias + n);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] += (float)bb[e];
      }
      if (R) {
        const E4 rr = *reinterpret_cast<const E4*>(R + (int64_t)m * g.ldr + n);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] += (float)rr[e];
      }
      if (rot) {
        const f32x4 t = *reinterpret_cast<const f32x4*>(g.rope + (int64_t)(m % g.rope_S) * (g.rope_d / 2) + (n % g.rope_d) / 2);
        v = f32x4{v[0] * t[0] - v[1] * t[1], v[0] * t[1] + v[1] * t[0], v[2] * t[2] - v[3] * t[3], v[2] * t[3] + v[3] * t[2]};
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (E)v[e];
      *reinterpret_cast<E4*>((E*)g.C + (int64_t)z * g.sC + (int64_t)m * g.ldc + n) = o;
    }
}

template <typename E, int FORM, int T, int KW, int NBUF>
__global__ __launch_bounds__(64 * KW) void gemm_small_kernel(Gemm g, int tiles_m, int tiles_n) {
  small_tile<E, FORM, T, KW, NBUF>(g, tiles_m, tiles_n, blockIdx.x, blockIdx.y);
}
// Weight gradients of a layer in one launch (see gemm_group).
template <typename E, int T, int KW, int NBUF> __global__ __launch_bounds__(64 * KW) void gemm_small_group_kernel(GemmGroup q) {
  int tiles_m, tiles_n, pid, z;
  const Gemm g = q.product_of(blockIdx.x, tiles_m, tiles_n, pid, z);
  small_tile<E, TN_ACC, T, KW, NBUF>(g, tiles_m, tiles_n, pid, z);
}
template <typename E, int T, int KW, int NBUF> hipError_t launch_group(hipStream_t st, const Gemm* g, int n) {
  GemmGroup q(g, n, 16 * T, 16 * T);
  hipLaunchKernelGGL((gemm_small_group_kernel<E, T, KW, NBUF>), dim3((unsigned)q.total), dim3(64 * KW), 0, st, q);
  return hipGetLastError();
}

template <typename E, int FORM, int T, int KW, int NBUF> hipError_t launch(hipStream_t st, const Gemm& g) {
  const int tm = (int)cdiv(g.M, 16 * T), tn = (int)cdiv(g.N, 16 * (FORM == NN_GLU ? 2 : T));
  hipLaunchKernelGGL((gemm_small_kernel<E, FORM, T, KW, NBUF>), dim3((unsigned)(tm * tn), (unsigned)g.batch), dim3(64 * KW), 0, st, g, tm, tn);
  return hipGetLastError();
}
// Forward products walk K with one wave, in the order of the staged kernels, and give their bits (with eight slabs in flight
// that costs little: 256 x 512, K = 512 4.5 us against 3.9 us with K shared out); 64x64 tiles gain nothing there.  The
// gradients' products share K out over 8 waves with either tile.
template <typename E, int FORM> hipError_t launch_form(hipStream_t st, const Gemm& g, int tile) {
  if constexpr (FORM == NN || FORM == NN_GLU) return launch<E, FORM, 2, 1, 8>(st, g);
  else return tile == 32 ? launch<E, FORM, 2, 8, 4>(st, g) : launch<E, FORM, 4, 8, 3>(st, g);
}
template <typename E> hipError_t launch_type(hipStream_t st, const Gemm& g, int tile) {
  if (g.glu == 1) return launch_form<E, NN_GLU>(st, g, tile);
  if (g.glu == 2) return launch_form<E, NT_GLU>(st, g, tile);
  if (g.transA) return g.nx ? launch_form<E, TN_PARTS>(st, g, tile) : launch_form<E, TN_ACC>(st, g, tile);
  if (g.transB) return g.kseg ? launch_form<E, NT_SEG>(st, g, tile) : launch_form<E, NT>(st, g, tile);
  return launch_form<E, NN>(st, g, tile);
}

}  // namespace

bool gemm_small_takes(const Gemm& g) {
  if (g.N % 4 || g.batch > 65535 || g.transA != g.c_f32_accum || (g.transA && g.transB)) return false;   // the forms of the stage's products
  // The k-lines of a row-contiguous operand that fill up the last slab lie behind its descriptor, unless their 32-bit offsets
  // wrap around: few rows, more than 2^32 / 64 bytes apart.
  const int64_t lines = cdiv(g.nx ? (int64_t)g.K - (int64_t)g.nx * g.kseg : g.K, 32) * 32;
  return !(g.transA && lines * g.lda * 2 >= (1ll << 32)) && !(!g.transB && lines * g.ldb * 2 >= (1ll << 32));
}

// Tile of the small kernel (32 or 64) when it is the faster way, else 0.  Times in us, fitted to single products of bf16 with
// M, N = 8 .. 6000, K = 8 .. 24000 and one to three batches.  Forward: a fixed part, and per k the latency of a walk or the
// loads of the workgroups that share a CU, whichever is longer.  Gradients: a round of workgroups on the 256 CUs costs a fixed
// time (a workgroup's launch, merge and store) plus the walk over K.  A k-contiguous B costs more per k (see above).  On the
// geometric mean of 1400 products the choice is within 0.4 % of the fastest of 32, 64 and 128x128 with one slab in flight, one part
// of K and no oblong tile beside it, which is what `staged` prices: gemm_mfma has become faster since, above all for input gradients
// with scratch, and the line has not been drawn again.  Measured against those staged tiles, us: 256 x 512, K = 512 4.5 : 8.9, input gradient with K = 2752 in two
// segments 10.9 : 27.1; 512 x 512, K = 256, accumulating 3.3 : 5.8; 1024 x 1024, K = 1024, accumulating 9.6 : 13.0.  At 1024 x
// 2048, K = 1024 it loses (16.3 : 14.1), at 512 x 4096, K = 4096 (47 : 37), and accumulating over few tokens, where the rounds'
// fixed time is all there is (1528 x 2624, K = 8: 16.6 : 7.8; 2376 x 1632, K = 16, two batches 30.4 : 11.7).
int gemm_small_tile(const Gemm& g, double* us) {
  if (!gemm_small_takes(g)) return 0;
  const double per_cu = (g.glu == 1 ? 2.0 : g.batch) / 256.0, k = (double)g.K;   // gate and up count like a batch of two
  const double n32 = cdiv(g.M, 32) * cdiv(g.N, 32) * per_cu, n64 = cdiv(g.M, 64) * cdiv(g.N, 64) * per_cu,
               n128 = cdiv(g.M, 128) * cdiv(g.N, 128) * per_cu;
  const double staged = 4.5 + 7.8e-3 * k * (n128 <= 1.0 ? 1.0 : n128 <= 2.0 ? 2.0 : n128 * 0.9);
  if (!g.transA && !g.transB) return 2.4 + k * std::max(4.5e-3, 2.6e-3 * n32) < 0.9 * staged ? 32 : 0;
  const double t32 = g.transB ? 2.0 + (2.6e-3 * k + 0.55) * std::ceil(n32) : 2.1 + (2.3e-3 * k + 0.83) * std::ceil(n32);
  const double t64 = g.transB ? 0.9 + (5.3e-3 * k + 2.4) * std::ceil(n64) : 0.4 + (4.0e-3 * k + 3.8) * std::ceil(n64);
  if (us) *us = std::min(t32, t64);
  if (t32 < 0.9 * staged && t32 <= t64) return 32;
  return t64 < 0.9 * staged ? 64 : 0;
}

hipError_t gemm_small(hipStream_t st, DType dt, const Gemm& g, int tile) {
  return dt == F16 ? launch_type<f16>(st, g, tile) : launch_type<bf16>(st, g, tile);
}

// Grouped weight gradients: 64x64 tiles whose two waves share K, so that four workgroups fit a CU and a layer of hidden 512 is one
// round.  The time in us, fitted to 13 layers (hidden 256 .. 2048, 64 .. 2048 tokens) that ran both ways, against the sum of the
// products' own times.  us per microbatch, forward and backward, one after the other : grouped: Llama, hidden 512, 256 tokens 143.8 :
// 133.6; GPT, hidden 512, 1024 tokens 229 : 216; Llama, hidden 768, 512 tokens 236 : 226; it loses for Llama, hidden 1024, 1024 tokens
// (341 : 349) and hidden 2048, 64 tokens (340 : 370).
double gemm_small_group_us(const Gemm* g, int n) {
  double tiles = 0.0;
  for (int i = 0; i < n; ++i) tiles += (double)cdiv(g[i].M, 64) * cdiv(g[i].N, 64) * g[i].batch / 256.0;
  return 4.35 + std::max(tiles, 1.0) * (1.37 + 3.98e-3 * g[0].K);
}
hipError_t gemm_small_group(hipStream_t st, DType dt, const Gemm* g, int n) {
  return dt == F16 ? launch_group<f16, 4, 2, 3>(st, g, n) : launch_group<bf16, 4, 2, 3>(st, g, n);
}

}  // namespace zs

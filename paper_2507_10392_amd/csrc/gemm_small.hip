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
//     them through LDS of the wave's own (rows_lds.h) unless K is short (launch_form): with one direct load per fragment the address
//     unit was the limit.  us, direct : through LDS, 64 x 768, K = 3072 12.7 : 6.4; 384 x 1024, K = 3072 23.6 : 11.3; 512 x 512, K = 512
//     4.4 : 3.5.
//   row-contiguous operand (A [K,M], B [K,N]): lane l loads NV consecutive columns of each of its eight k-lines; pairs of
//     k-lines are then interleaved by one v_perm_b32 per register, which leaves in NV fragments the columns NV (l%16) + j.
// The matrix instruction gets B as its first operand, so a lane ends up with 4 consecutive columns of one row of C.
#include "kernels.h"
#include "rows_lds.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace zs {
namespace {

constexpr unsigned OUT = 0x80000000u;   // pushes a lane's offset past every descriptor (extents are below 2^30 bytes): reads 0
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

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

// A row-contiguous operand's share of a slab of 32 k, NB blocks of 16 rows, as loaded.
template <int NB> struct Raw;
template <> struct Raw<4> {          // 4 columns of 8 k-lines
  u32x2 v[8];
  __device__ __forceinline__ u32x4 frag(int b) const {
    u32x4 f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      f[i] = __builtin_amdgcn_perm(v[2 * i + 1][b >> 1], v[2 * i][b >> 1], b & 1 ? 0x07060302u : 0x05040100u);
    return f;
  }
};
template <> struct Raw<2> {          // 2 columns of 8 k-lines
  unsigned v[8];
  __device__ __forceinline__ u32x4 frag(int b) const {
    u32x4 f;
#pragma unroll
    for (int i = 0; i < 4; ++i) f[i] = __builtin_amdgcn_perm(v[2 * i + 1], v[2 * i], b & 1 ? 0x07060302u : 0x05040100u);
    return f;
  }
};
// at: byte offset of the lane's columns in its first k-line (OUT for columns past the end), ld2: bytes of a k-line
__device__ __forceinline__ void load_r(Raw<4>& f, __amdgpu_buffer_rsrc_t rs, unsigned at, unsigned ld2, unsigned soff) {
#pragma unroll
  for (int i = 0; i < 8; ++i) f.v[i] = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)(at + i * ld2), (int)soff, 0);
}
__device__ __forceinline__ void load_r(Raw<2>& f, __amdgpu_buffer_rsrc_t rs, unsigned at, unsigned ld2, unsigned soff) {
#pragma unroll
  for (int i = 0; i < 8; ++i) f.v[i] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(at + i * ld2), (int)soff, 0);
}

// A k-contiguous operand's share of a slab, read straight into fragments: 8 k of rows 16 apart.
template <int NB> struct RawK {
  u32x4 v[NB];
  __device__ __forceinline__ u32x4 frag(int b) const { return v[b]; }
};
template <int NB> __device__ __forceinline__ void load_k(RawK<NB>& f, __amdgpu_buffer_rsrc_t rs, unsigned at, unsigned ld2, unsigned soff) {
#pragma unroll
  for (int b = 0; b < NB; ++b) f.v[b] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(at + 16 * b * ld2), (int)soff, 0);
}

enum Form { NT, NT_SEG, TN_ACC, TN_PARTS, NT_GLU };

__device__ __forceinline__ void tile_of(int pid, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int ntiles = tiles_m * tiles_n;   // ids are dealt round-robin to the 8 XCDs; each gets a contiguous run of the tile order
  if (pid < ntiles / 8 * 8) pid = (pid % 8) * (ntiles / 8) + pid / 8;
  gemm_tile_of(pid, tiles_m, tiles_n, tm, tn);
}

// T: blocks of 16 rows and columns a wave's tile has each way (2: 32x32, 4: 64x64), KW: waves that share out K, LINES: k-contiguous operands
// come in through LDS, NBUF: slabs held otherwise (NBUF - 1 of them in flight).
template <typename E, int FORM, int T, int KW, int NBUF, bool LINES>
__device__ __forceinline__ void small_tile(const Gemm& g, int tiles_m, int tiles_n, int pid, int z) {
  constexpr bool TA = FORM == TN_ACC || FORM == TN_PARTS, TB = !TA, ACC = TA;
  constexpr int NQ = T * T;                        // quads of 4 consecutive columns a lane holds
  constexpr int RED = (KW - 1) * NQ * 64, STAGE = LINES ? KW * 2 * T * 128 : 0;
  __shared__ f32x4 red[RED > STAGE ? RED : STAGE]; // partial tiles take the place of the slabs
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lm = lane & 15, lg = lane >> 4;
  int tm, tn;
  tile_of(pid, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * 16 * T, n0 = tn * 16 * T;
  const E* A = (const E*)g.A + (int64_t)z * g.sA;
  const E* B = (const E*)g.B + (int64_t)z * g.sB;
  const unsigned lda = (unsigned)g.lda, ldb = (unsigned)g.ldb;
  const int K1 = FORM == TN_PARTS ? g.kseg : g.K;   // rows of a part, or of the only one
  const int64_t recB = TB ? (FORM == NT_SEG ? (int64_t)(g.K / g.kseg - 1) * g.segB + (int64_t)(g.N - 1) * ldb + g.kseg : (int64_t)(g.N - 1) * ldb + g.K)
                          : (int64_t)(K1 - 1) * ldb + g.N;
  const __amdgpu_buffer_rsrc_t ra = rsrc(A, TA ? (int64_t)(K1 - 1) * lda + g.M : (int64_t)(g.M - 1) * lda + g.K), rb = rsrc(B, recB);

  f32x4 acc[T][T];
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int slabs = (g.K + 31) / 32, per = (slabs + KW - 1) / KW;
  const int s0 = wave * per, s1 = min(slabs, s0 + per);   // this wave's slabs
  if constexpr (LINES) {
    // Two pairs of slabs in flight: on 32x32 tiles a third takes the registers of a CU's second workgroup (512 x 768, K = 256 4.8 us, 4.2 with
    // two).
    // The fragments hold the same k as with direct loads.
    constexpr int DEPTH = 2;
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
          wave_lds_order();   // the pair before has been read
          put_rows<T>(pairs[i].a, la, lane);
          put_rows<T>(pairs[i].b, lb, lane);
          wave_lds_order();
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
    const unsigned ao = TB ? ((m0 + lm) * lda + 8 * lg) * 2 : m0 + T * lm < g.M ? (8 * lg * lda + m0 + T * lm) * 2 : OUT,
                   bo = TB ? ((n0 + lm) * ldb + (FORM == NT_SEG ? 0 : 8 * lg)) * 2 : n0 + T * lm < g.N ? (8 * lg * ldb + n0 + T * lm) * 2 : OUT;
    struct Slab { std::conditional_t<TB, RawK<T>, Raw<T>> a, b; } buf[NBUF];
    auto load = [&](Slab& s, int slab) {                   // k-lines past K lie behind the descriptors
      const int k = slab * 32;
      if constexpr (TB) {
        const int kl = k + 8 * lg;
        const bool past = kl >= g.K;                       // K is a multiple of 8
        load_k<T>(s.a, ra, past ? OUT : ao, lda * 2, k * 2);
        if constexpr (FORM == NT_SEG) {
          const int seg = kl / g.kseg;
          load_k<T>(s.b, rb, past ? OUT : bo + (unsigned)(seg * g.segB + (kl - seg * g.kseg)) * 2, ldb * 2, 0);
        } else load_k<T>(s.b, rb, past ? OUT : bo, ldb * 2, k * 2);
      } else if constexpr (FORM == TN_PARTS) {   // slabs do not straddle parts: kseg is a multiple of 128
        const int p = min(k / g.kseg, g.nx), kin = k - p * g.kseg;
        const int rows = p < g.nx ? g.kseg : g.K - g.nx * g.kseg;
        const __amdgpu_buffer_rsrc_t pa = rsrc((p ? (const E*)g.Ax[p - 1] : (const E*)g.A) + (int64_t)z * g.sA, (int64_t)(rows - 1) * lda + g.M),
                                     pb = rsrc((p ? (const E*)g.Bx[p - 1] : (const E*)g.B) + (int64_t)z * g.sB, (int64_t)(rows - 1) * ldb + g.N);
        load_r(s.a, pa, ao, lda * 2, kin * lda * 2);
        load_r(s.b, pb, bo, ldb * 2, kin * ldb * 2);
      } else {
        load_r(s.a, ra, ao, lda * 2, k * lda * 2);
        load_r(s.b, rb, bo, ldb * 2, k * ldb * 2);
      }
    };
    auto multiply = [&](const Slab& s) {
      u32x4 a[T];
#pragma unroll
      for (int i = 0; i < T; ++i) a[i] = s.a.frag(i);
#pragma unroll
      for (int j = 0; j < T; ++j) {
        const u32x4 b = s.b.frag(j);
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

  // A lane's quads: quad (i, q) is row m(i), columns n(q) .. n(q)+3.
  auto quad = [&](int i, int q) {
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (TB) v[e] = acc[i][q][e];
      else v[e] = acc[i][(4 * q + e) % T][(4 * q + e) / T];   // column T (4 lg + r) + j  <->  block j, register r
    }
    return v;
  };
  // quad s is finished by the wave s % KW; the others leave theirs in LDS, and it adds them in the order of the waves
#pragma unroll
  for (int s = 0; s < NQ; ++s)
    if (s % KW != wave) red[((wave < s % KW ? wave : wave - 1) * NQ + s) * 64 + lane] = quad(s / T, s % T);
  __syncthreads();
  auto sum = [&](int s) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int o = 0; o < KW; ++o) v += o == s % KW ? quad(s / T, s % T) : red[((o < s % KW ? o : o - 1) * NQ + s) * 64 + lane];
    return v;
  };
  typedef E E4 __attribute__((ext_vector_type(4)));
  auto row_of = [&](int i) { return m0 + (TA ? T * lm + i : 16 * i + lm); };
  auto col_of = [&](int q) { return n0 + (TB ? 16 * q + 4 * lg : 4 * T * lg + 4 * q); };
  const E* bias = g.bias ? (const E*)g.bias + (int64_t)z * g.sBias : nullptr;
  const E* R = g.resid ? (const E*)g.resid + (int64_t)z * g.sC : nullptr;
  const bool rot = g.rope && z < g.rope_batches;
#pragma unroll
  for (int s = 0; s < NQ; ++s)
    if (s % KW == wave) {
      const int m = row_of(s / T), n = col_of(s % T);
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

// y = x W (GLU: gate and up projection of the same columns, and the gated unit of the rounded values).  A workgroup of 4 waves owns 32x32
// outputs, every wave one 16x16 block of them (GLU: of each projection), which walks K in the order of the staged kernels and so
// gives their bits.  The waves share the loads: stages of 128 k, whole lines of x and the tile's 64 bytes of every line of W, go
// to one of two LDS buffers, with four stages in flight (eight are 3 % slower).  x's 16-byte pieces are stored at position
// p ^ row % 16; W stays [k][column], lines 96 bytes apart, and is read transposed.  A stage costs 0.33 us, its LDS round trip and barrier.
// us against one wave per tile, whose address unit took the 64 pieces of every load of x one by one: 256 x 512, K = 512 4.5 : 3.9, K =
// 1384 8.1 : 6.2; 256 x 3072, K = 768 (768 tiles) 8.2 : 8.4; 0.88 on the geometric mean of 96 products with 64 to 1000 rows.
template <typename E, bool GLU>
__device__ __forceinline__ void forward_together(const Gemm& g, int tiles_m, int tiles_n, int pid, int z) {
  constexpr int SK = 128, DEPTH = 4, NM = GLU ? 2 : 1;     // k of a stage, stages in flight, matrices W
  constexpr int LINE = 6, SA = 32 * 16, SB = SK * LINE;    // 16-byte pieces: of a line of W, of a stage of x and of W
  __shared__ u32x4 lds[2][SA + NM * SB];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wi = wave >> 1, wj = wave & 1;
  const int lm = lane & 15, lg = lane >> 4;
  int tm, tn;
  tile_of(pid, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * 32, n0 = tn * 32;
  const E* B = (const E*)g.B + (int64_t)z * g.sB;
  const unsigned lda = (unsigned)g.lda, ldb = (unsigned)g.ldb;
  const __amdgpu_buffer_rsrc_t ra = rsrc((const E*)g.A + (int64_t)z * g.sA, (int64_t)(g.M - 1) * lda + g.K);
  const __amdgpu_buffer_rsrc_t rb[2] = {rsrc(B, (int64_t)(g.K - 1) * ldb + g.N), rsrc(B + (GLU ? g.sB : 0), (int64_t)(g.K - 1) * ldb + g.N)};

  struct Stage { u32x4 a[2], b[NM][2]; } st[DEPTH];
  const unsigned ao = ((m0 + (tid >> 4)) * lda + 8 * (tid & 15)) * 2, bo = n0 + 8 * (tid & 3) < g.N ? ((tid >> 2) * ldb + n0 + 8 * (tid & 3)) * 2 : OUT;
  auto load = [&](Stage& s, int k0) {
    const unsigned at = k0 + 8 * (tid & 15) < g.K ? ao : OUT;   // K is a multiple of 8
#pragma unroll
    for (int i = 0; i < 2; ++i) s.a[i] = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)at, (int)((16 * i * lda + k0) * 2), 0);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const unsigned line = k0 + 64 * i + (tid >> 2) < g.K ? bo : OUT;
#pragma unroll
      for (int w = 0; w < NM; ++w) s.b[w][i] = __builtin_amdgcn_raw_buffer_load_b128(rb[w], (int)line, (int)((k0 + 64 * i) * ldb * 2), 0);
    }
  };
  auto put = [&](const Stage& s, u32x4* to) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      to[((tid >> 4) + 16 * i) * 16 + ((tid & 15) ^ (tid >> 4))] = s.a[i];
#pragma unroll
      for (int w = 0; w < NM; ++w) to[SA + w * SB + ((tid >> 2) + 64 * i) * LINE + (tid & 3)] = s.b[w][i];
    }
  };
  f32x4 acc[NM];
#pragma unroll
  for (int w = 0; w < NM; ++w) acc[w] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto slabs = [&](auto count, const u32x4* from) {            // fragments of all slabs first: one LDS latency
    constexpr int NS = decltype(count)::value;
    u32x4 a[NS], b[NS][NM];
#pragma unroll
    for (int h = 0; h < NS; ++h) {
      a[h] = from[(16 * wi + lm) * 16 + ((4 * h + lg) ^ lm)];
#pragma unroll
      for (int w = 0; w < NM; ++w) {
        const short* p = reinterpret_cast<const short*>(from + SA + w * SB + (32 * h + 8 * lg + (lm >> 2)) * LINE) + 16 * wj + 4 * (lm & 3);
        union { struct { s16x4 lo, hi; } s; u32x4 v; } u;
        u.s.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
        u.s.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * LINE * 8));
        b[h][w] = u.v;
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int h = 0; h < NS; ++h)
#pragma unroll
      for (int w = 0; w < NM; ++w) acc[w] = mfma<E>(b[h][w], a[h], acc[w]);
  };
  auto multiply = [&](const u32x4* from, int k0) {
    const int left = (g.K - k0 + 31) / 32;                      // slabs; the last stage may have fewer than four
    if (left >= 4) slabs(std::integral_constant<int, 4>{}, from);
    else if (left == 3) slabs(std::integral_constant<int, 3>{}, from);
    else if (left == 2) slabs(std::integral_constant<int, 2>{}, from);
    else slabs(std::integral_constant<int, 1>{}, from);
  };

  typedef E E4 __attribute__((ext_vector_type(4)));
  const int m = m0 + 16 * wi + lm, n = n0 + 16 * wj + 4 * lg;   // the lane's row and first of its 4 columns
  const bool inside = m < g.M && n < g.N;                       // N is a multiple of 8
  const bool bias = !GLU && inside && g.bias, resid = !GLU && inside && g.resid, rot = !GLU && inside && g.rope && z < g.rope_batches;
  const int stages = (g.K + SK - 1) / SK;
#pragma unroll
  for (int i = 0; i < DEPTH; ++i)
    if (i < stages) load(st[i], i * SK);
  E4 bb = {}, rr = {};                                          // what the store adds comes in behind the first stages
  f32x4 t = {};
  if (bias) bb = *reinterpret_cast<const E4*>((const E*)g.bias + (int64_t)z * g.sBias + n);
  if (resid) rr = *reinterpret_cast<const E4*>((const E*)g.resid + (int64_t)z * g.sC + (int64_t)m * g.ldr + n);
  if (rot) t = *reinterpret_cast<const f32x4*>(g.rope + (int64_t)(m % g.rope_S) * (g.rope_d / 2) + (n % g.rope_d) / 2);
  for (int s = 0; s < stages; s += DEPTH)
#pragma unroll
    for (int i = 0; i < DEPTH; ++i)
      if (s + i < stages) {
        put(st[i], lds[i & 1]);                                 // last read before the previous stage's barrier
        if (s + i + DEPTH < stages) load(st[i], (s + i + DEPTH) * SK);
        __syncthreads();
        multiply(lds[i & 1], (s + i) * SK);
      }
  if (!inside) return;
  E4 o;
  if constexpr (GLU) {
    E4 ou, oa;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o[e] = (E)acc[0][e];
      ou[e] = (E)acc[1][e];
      oa[e] = (E)glu_f((float)o[e], (float)ou[e]);
    }
    E* pg = (E*)g.gu + (int64_t)m * g.gu_ld + n;
    *reinterpret_cast<E4*>(pg) = o;
    *reinterpret_cast<E4*>(pg + g.gu_up) = ou;
    *reinterpret_cast<E4*>((E*)g.C + (int64_t)m * g.ldc + n) = oa;
  } else {
    f32x4 v = acc[0];
    if (bias) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += (float)bb[e];
    }
    if (resid) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += (float)rr[e];
    }
    if (rot) v = f32x4{v[0] * t[0] - v[1] * t[1], v[0] * t[1] + v[1] * t[0], v[2] * t[2] - v[3] * t[3], v[2] * t[3] + v[3] * t[2]};
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (E)v[e];
    *reinterpret_cast<E4*>((E*)g.C + (int64_t)z * g.sC + (int64_t)m * g.ldc + n) = o;
  }
}

// The same with one wave per tile, which reads its operands straight into fragments, seven slabs of 32 k ahead: see forward_shared.
template <typename E, bool GLU>
__device__ __forceinline__ void forward_alone(const Gemm& g, int tiles_m, int tiles_n, int pid, int z) {
  constexpr int T = 2, NB = 2, NJ = GLU ? 2 * NB : NB, NBUF = 8;   // blocks of rows, of columns of one matrix and of the tile; slabs held
  const int lane = threadIdx.x & 63, lm = lane & 15, lg = lane >> 4;
  int tm, tn;
  tile_of(pid, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * 16 * T, n0 = tn * 16 * NB;
  const E* A = (const E*)g.A + (int64_t)z * g.sA;
  const E* B = (const E*)g.B + (int64_t)z * g.sB;
  const unsigned lda = (unsigned)g.lda, ldb = (unsigned)g.ldb;
  const __amdgpu_buffer_rsrc_t ra = rsrc(A, (int64_t)(g.M - 1) * lda + g.K), rb = rsrc(B, (int64_t)(g.K - 1) * ldb + g.N);
  const __amdgpu_buffer_rsrc_t rb2 = rsrc(B + (GLU ? g.sB : 0), (int64_t)(g.K - 1) * ldb + g.N);
  unsigned ao[T];
#pragma unroll
  for (int i = 0; i < T; ++i) ao[i] = ((m0 + 16 * i + lm) * lda + 8 * lg) * 2;
  const unsigned bo = n0 + NB * lm < g.N ? (8 * lg * ldb + n0 + NB * lm) * 2 : OUT;
  struct Slab { RawK<T> a; Raw<NB> b, b2; };
  Slab buf[NBUF];
  auto load = [&](Slab& s, int slab) {   // k-lines past K lie behind the descriptors
    const int k = slab * 32;
    const bool past = k + 8 * lg >= g.K;
#pragma unroll
    for (int i = 0; i < T; ++i) s.a.v[i] = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)(past ? OUT : ao[i]), k * 2, 0);
    load_r(s.b, rb, bo, ldb * 2, k * ldb * 2);
    if constexpr (GLU) load_r(s.b2, rb2, bo, ldb * 2, k * ldb * 2);
  };
  f32x4 acc[T][NJ];
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](const Slab& s) {
    u32x4 a[T];
#pragma unroll
    for (int i = 0; i < T; ++i) a[i] = s.a.frag(i);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const u32x4 b = GLU && j >= NB ? s.b2.frag(j % NB) : s.b.frag(j % NB);
#pragma unroll
      for (int i = 0; i < T; ++i) acc[i][j] = mfma<E>(b, a[i], acc[i][j]);
    }
  };
  // s0 is the only wave's first slab, 0, which the compiler cannot see: where it can, it peels the loop and then waits for all loads in
  // flight at every slab (512 x 768, K = 2080 16.2 us instead of 11.4).
  const int slabs = (g.K + 31) / 32, s0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * slabs, s1 = min(slabs, s0 + slabs);
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

  // column NB (4 lg + r) + j  <->  block j, register r
  auto quad = [&](int i, int q) {
    const int base = q / NB * NB, ql = q % NB;
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = acc[i][base + (4 * ql + e) % NB][(4 * ql + e) / NB];
    return v;
  };
  typedef E E4 __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const int m = m0 + 16 * i + lm, n = n0 + 4 * NB * lg + 4 * q;
      if (m >= g.M || n >= g.N) continue;
      f32x4 v = quad(i, q);
      E* out = (E*)g.C + (int64_t)z * g.sC + (int64_t)m * g.ldc + n;
      E4 o;
      if constexpr (GLU) {
        const f32x4 u = quad(i, q + NB);
        E4 ou, oa;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          o[e] = (E)v[e];
          ou[e] = (E)u[e];
          oa[e] = (E)glu_f((float)o[e], (float)ou[e]);
        }
        E* pg = (E*)g.gu + (int64_t)m * g.gu_ld + n;
        *reinterpret_cast<E4*>(pg) = o;
        *reinterpret_cast<E4*>(pg + g.gu_up) = ou;
        *reinterpret_cast<E4*>(out) = oa;
      } else {
        if (g.bias) {
          const E4 bb = *reinterpret_cast<const E4*>((const E*)g.bias + (int64_t)z * g.sBias + n);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] += (float)bb[e];
        }
        if (g.resid) {
          const E4 rr = *reinterpret_cast<const E4*>((const E*)g.resid + (int64_t)z * g.sC + (int64_t)m * g.ldr + n);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] += (float)rr[e];
        }
        if (g.rope && z < g.rope_batches) {
          const f32x4 t = *reinterpret_cast<const f32x4*>(g.rope + (int64_t)(m % g.rope_S) * (g.rope_d / 2) + (n % g.rope_d) / 2);
          v = f32x4{v[0] * t[0] - v[1] * t[1], v[0] * t[1] + v[1] * t[0], v[2] * t[2] - v[3] * t[3], v[2] * t[3] + v[3] * t[2]};
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (E)v[e];
        *reinterpret_cast<E4*>(out) = o;
      }
    }
}

template <typename E, bool GLU> __global__ __launch_bounds__(64) void gemm_small_forward_alone_kernel(Gemm g, int tiles_m, int tiles_n) {
  forward_alone<E, GLU>(g, tiles_m, tiles_n, blockIdx.x, blockIdx.y);
}
template <typename E, bool GLU> __global__ __launch_bounds__(256, GLU ? 2 : 4) void gemm_small_forward_kernel(Gemm g, int tiles_m, int tiles_n) {
  forward_together<E, GLU>(g, tiles_m, tiles_n, blockIdx.x, blockIdx.y);
}

template <typename E, int FORM, int T, int KW, int NBUF, bool LINES>
__global__ __launch_bounds__(64 * KW) void gemm_small_kernel(Gemm g, int tiles_m, int tiles_n) {
  small_tile<E, FORM, T, KW, NBUF, LINES>(g, tiles_m, tiles_n, blockIdx.x, blockIdx.y);
}
// Weight gradients of a layer in one launch (see gemm_group).
template <typename E, int T, int KW, int NBUF> __global__ __launch_bounds__(64 * KW) void gemm_small_group_kernel(GemmGroup q) {
  int tiles_m, tiles_n, pid, z;
  const Gemm g = q.product_of(blockIdx.x, tiles_m, tiles_n, pid, z);
  small_tile<E, TN_ACC, T, KW, NBUF, false>(g, tiles_m, tiles_n, pid, z);
}
template <typename E, int T, int KW, int NBUF> hipError_t launch_group(hipStream_t st, const Gemm* g, int n) {
  GemmGroup q(g, n, 16 * T, 16 * T);
  hipLaunchKernelGGL((gemm_small_group_kernel<E, T, KW, NBUF>), dim3((unsigned)q.total), dim3(64 * KW), 0, st, q);
  return hipGetLastError();
}

template <typename E, int FORM, int T, int KW, int NBUF, bool LINES> hipError_t launch(hipStream_t st, const Gemm& g) {
  const int tm = (int)cdiv(g.M, 16 * T), tn = (int)cdiv(g.N, 16 * T);
  hipLaunchKernelGGL((gemm_small_kernel<E, FORM, T, KW, NBUF, LINES>), dim3((unsigned)(tm * tn), (unsigned)g.batch), dim3(64 * KW), 0, st, g, tm, tn);
  return hipGetLastError();
}
// Four waves to a tile that share its loads, or one wave.  With more than a tile per CU other tiles cover a lone wave's waits, and it is the faster
// way over a short K, where the shared form still fills its stages; where rows of x are not whole lines, unless K is long; and for gate and
// up together, whose LDS leaves a CU two workgroups, until every CU has them.  us, shared : alone: 829 x 2424, K = 48 5.8 : 4.0; 548 x 1376, K =
// 912 11.0 : 8.3; 700 x 1024, K = 2768 21.3 : 22.7; gate and up: 128 x 2088, K = 776 9.9 : 8.6 (264 tiles), 256 x 1376, K = 512 7.2 : 6.8 (344),
// 400 x 1024, K = 256 4.9 : 5.3 (416).  It loses up to 7 % at 512 to 768 tiles (512 x 1024, K = 2768 15.5 : 14.5).
bool forward_shared(const Gemm& g) {
  const int64_t tiles = cdiv(g.M, 32) * cdiv(g.N, 32) * g.batch;
  if (tiles <= 256 || g.K <= 96) return tiles <= 256;
  return g.K <= 256 || (g.glu ? tiles > 400 : g.lda % 64 == 0 || g.K > 2600);
}
template <typename E, bool GLU> hipError_t launch_forward(hipStream_t st, const Gemm& g) {
  const int tm = (int)cdiv(g.M, 32), tn = (int)cdiv(g.N, 32);
  const dim3 grid((unsigned)(tm * tn), (unsigned)g.batch);
  if (forward_shared(g)) hipLaunchKernelGGL((gemm_small_forward_kernel<E, GLU>), grid, dim3(256), 0, st, g, tm, tn);
  else hipLaunchKernelGGL((gemm_small_forward_alone_kernel<E, GLU>), grid, dim3(64), 0, st, g, tm, tn);
  return hipGetLastError();
}
// The gradients' products share K out over 8 waves with either tile.  Input gradients of one slab per wave have nothing to run beside the way
// through LDS, and up to three where a piece of 128 bytes lies in two lines: us, through LDS : direct: 334 x 1016, K = 232 3.9 : 3.6; 1024 x 512, K =
// 128 4.5 : 3.5; 232 x 680, K = 648 4.1 : 3.8; 678 x 624, K = 280 3.9 : 3.6.
template <typename E, int FORM> hipError_t launch_form(hipStream_t st, const Gemm& g, int tile) {
  if constexpr (FORM == NT || FORM == NT_SEG || FORM == NT_GLU)
    if (g.K > 768 || (g.K >= 256 && g.lda % 64 == 0 && g.ldb % 64 == 0))
      return tile == 32 ? launch<E, FORM, 2, 8, 4, true>(st, g) : launch<E, FORM, 4, 8, 3, true>(st, g);
  return tile == 32 ? launch<E, FORM, 2, 8, 4, false>(st, g) : launch<E, FORM, 4, 8, 3, false>(st, g);
}
template <typename E> hipError_t launch_type(hipStream_t st, const Gemm& g, int tile) {
  if (g.glu == 1) return launch_forward<E, true>(st, g);
  if (g.glu == 2) return launch_form<E, NT_GLU>(st, g, tile);
  if (g.transA) return g.nx ? launch_form<E, TN_PARTS>(st, g, tile) : launch_form<E, TN_ACC>(st, g, tile);
  if (g.transB) return g.kseg ? launch_form<E, NT_SEG>(st, g, tile) : launch_form<E, NT>(st, g, tile);
  return launch_forward<E, false>(st, g);
}

}  // namespace

bool gemm_small_takes(const Gemm& g) {
  if (g.N % 4 || g.batch > 65535 || g.transA != g.c_f32_accum || (g.transA && g.transB)) return false;   // the forms of the stage's products
  // k-lines of a row-contiguous operand that fill up the last slab (forward: stage) must not wrap around in 32 bits: few rows, far
  // apart.  They lie behind the descriptor; the forward's lanes are pushed there by 2^31.
  const int64_t lines = cdiv(g.nx ? (int64_t)g.K - (int64_t)g.nx * g.kseg : g.K, 32) * 32;
  if (g.transA) return lines * g.lda * 2 < (1ll << 32) && lines * g.ldb * 2 < (1ll << 32);
  return g.transB || cdiv(g.K, 128) * 128 * g.ldb * 2 < (1ll << 31);
}

// Tile of the small kernel (32 or 64) when it is the faster way, else 0.  Times in us, fitted to single products of bf16 with
// M, N = 8 .. 6000, K = 8 .. 24000 and one to three batches.  Forward: a fixed part, and per k the latency of a walk or the
// loads of the workgroups that share a CU, whichever is longer.  Gradients: a round of workgroups on the 256 CUs costs a fixed
// time (a workgroup's launch, merge and store) plus the walk over K.  A k-contiguous B costs more per k (see above).  On the
// geometric mean of 1400 products the choice is within 0.4 % of the fastest of 32, 64 and 128x128 with one slab in flight, one part
// of K and no oblong tile beside it, which is what `staged` prices: gemm_mfma has become faster since, above all for input gradients
// with scratch, and so have the small kernels' forward products and input gradients; the line still takes the fastest of 32, 64 and
// the staged tiles within 0.3 % on the geometric mean of 150 more products of 32 to 2500 rows (15 % at worst), and has not been
// drawn again.  Measured against those staged tiles, us: 256 x 512, K = 512 4.5 : 8.9, input gradient with K = 2752 in two
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

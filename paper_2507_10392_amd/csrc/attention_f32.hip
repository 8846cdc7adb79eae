// Causal softmax attention of the fp32 configuration on the fp32 matrix cores (v_mfma_f32_16x16x4_f32), forward and backward,
// without atomics and without the S x S matrix.
//
// What bounds it: the models that run in fp32 are small, so a launch has few rows and its time is a wave's walk over the keys.
// A workgroup therefore owns only 16 queries (or keys), and its four waves share out the other side's tiles of 32 rows and
// merge at the end through LDS, in a fixed order.  Every wave loads its own operands from L2: "k" fragments (4 consecutive
// elements along the head dim per lane; whole lines that change places in LDS, see load_lines) for the products over d, "r" fragments
// (4 consecutive head-dim columns of rows 4 (l/16) + e, which are whole lines as they are) for the products over keys or queries.
// All products are transposed (S^T = K Q^T, O^T = V^T P^T): a lane then owns query l%16 and holds the scores of keys 4 (l/16) + r
// in register r, which is the operand layout that step e = r of the second product wants, so P never moves between lanes.
// The loads of a tile run one tile-quarter (or more, registers permitting) ahead of their use.
//
// Measured, forward + backward in three launches with direct loads of "k" fragments (now through LDS, see load_lines), against the
// wave-per-row kernel: 8 heads of 64, S = 128: 91 -> 30 us; 4 heads of 128, S = 256: 273 -> 51 us; 16 heads of 64, S = 1000:
// 2080 -> 188 us; the errors against float64 are smaller (dk 8.1e-7 -> 4.8e-7).
#include "kernels.h"
#include "attention_rows.h"

namespace zs {
namespace {

constexpr unsigned OUT = 0x80000000u;   // past every descriptor: reads 0
constexpr int KW = 4;                   // waves of a workgroup
constexpr int TK = 32;                  // rows of a tile of the other side

// Rows of one head: [S, dd] with row stride ld, read as zero outside.
struct Head { __amdgpu_buffer_rsrc_t rs; unsigned ld; };
__device__ __forceinline__ Head head_of(const float* p, int64_t ld, int S, int dd) {
  return Head{__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, (int)((((int64_t)S - 1) * ld + dd) * 4), 0x00020000), (unsigned)ld};
}
__device__ __forceinline__ f32x4 load4(const Head& h, unsigned voff, unsigned soff) {
  union { u32x4 u; f32x4 f; } c;
  c.u = __builtin_amdgcn_raw_buffer_load_b128(h.rs, (int)voff, (int)soff, 0);
  return c.f;
}
// 16 rows x 16 DS columns from row `row0`: k[s] = columns 16 s + 4 (l/16) .. +3 of row l%16.  They come as whole lines (load_lines; read as
// fragments, the lanes of a load would lie in 16 rows, and the address unit takes four times as long for their pieces) and change
// places in LDS of the wave's own (to_k; wave_lds_order, no barrier), the 16-byte piece p of row r at p ^ r.
// us, fragments : lines: S = 256, 4 heads of 128 forward 13.0 : 10.8, backward 26.0 : 19.7; S = 128, 8 of 64 10.9 : 7.9 (backward); S = 1000, 16
// of 64 40 : 30 and 138 : 105; 64 of 128 325 : 201 and 932 : 842.
template <int DS> struct Lines { f32x4 v[16 * 4 * DS]; };
template <int DS> __device__ __forceinline__ void load_lines(f32x4 (&f)[DS], const Head& h, int row0, int lane, int dd) {
  constexpr int P = 4 * DS, R = 64 / P;   // pieces of a row, rows of a load
  const unsigned at = 4 * (lane % P) < dd ? lane / P * h.ld * 4 + lane % P * 16 : OUT;
#pragma unroll
  for (int s = 0; s < DS; ++s) f[s] = load4(h, at, (row0 + R * s) * h.ld * 4);
}
template <int DS> __device__ __forceinline__ void to_k(f32x4 (&f)[DS], Lines<DS>& lines, int lane) {
  constexpr int P = 4 * DS, R = 64 / P;
  wave_lds_order();   // the rows before have been read
#pragma unroll
  for (int s = 0; s < DS; ++s) {
    const int row = R * s + lane / P;
    lines.v[row * P + ((lane % P) ^ row)] = f[s];
  }
  wave_lds_order();
#pragma unroll
  for (int s = 0; s < DS; ++s) f[s] = lines.v[(lane & 15) * P + ((4 * s + (lane >> 4)) ^ (lane & 15))];
}
// The same 16 rows by columns: r[4 g + e] = columns 64 g + 4 (l%16) .. +3 of row 4 (l/16) + e.
template <int DS> __device__ __forceinline__ void load_r(f32x4 (&f)[DS], const Head& h, int row0, int lane, int dd) {
#pragma unroll
  for (int g = 0; g < DS / 4; ++g) {
    const unsigned col = 64 * g + 4 * (lane & 15);
#pragma unroll
    for (int e = 0; e < 4; ++e) f[4 * g + e] = load4(h, (int)col < dd ? ((4 * (lane >> 4) + e) * h.ld + col) * 4 : OUT, row0 * h.ld * 4);
  }
}
__device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
// 16x16 block over the head dim: register r of lane l = sum_c rows[4 (l/16) + r][c] * mine[l%16][c].
template <int DS> __device__ __forceinline__ f32x4 dot(const f32x4 (&rows)[DS], const f32x4 (&mine)[DS]) {
  f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;   // two chains: half the depth and half the rounding
#pragma unroll
  for (int s = 0; s < DS; ++s)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (s & 1) b = mfma(rows[s][e], mine[s][e], b);
      else a = mfma(rows[s][e], mine[s][e], a);
    }
  return a + b;
}
// acc += rows^T w: w[r] belongs to row 4 (l/16) + r.  acc[4 g + j] holds, in register r of lane l, column
// 64 g + 16 (l/16) + 4 r + j of lane l's own row l%16.
template <int DS> __device__ __forceinline__ void add_weighted(f32x4 (&acc)[DS], const f32x4 (&rows)[DS], const f32x4& w) {
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int g = 0; g < DS / 4; ++g)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[4 * g + j] = mfma(rows[4 * g + e][j], w[e], acc[4 * g + j]);
}
// quad q = 4 g + r of an accumulator: columns quad_col(q) .. +3 of the lane's row
template <int DS> __device__ __forceinline__ f32x4 quad(const f32x4 (&acc)[DS], int q) {
  const int g = q >> 2, r = q & 3;
  return f32x4{acc[4 * g][r], acc[4 * g + 1][r], acc[4 * g + 2][r], acc[4 * g + 3][r]};
}
__device__ __forceinline__ int quad_col(int q, int lane) { return 64 * (q >> 2) + 16 * (lane >> 4) + 4 * (q & 3); }
__device__ __forceinline__ float over_groups_max(float v) {
  v = fmaxf(v, __shfl_xor(v, 16, 64));
  return fmaxf(v, __shfl_xor(v, 32, 64));
}
__device__ __forceinline__ float over_groups_sum(float v) {
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}
// Rotates back the two pairs of a quad: (u, w) -> (u c + w s, w c - u s).
__device__ __forceinline__ f32x4 unrotate(const f32x4& x, const float2* rope, int pos, int col, int dd) {
  const float2 t0 = rope[(int64_t)pos * (dd / 2) + col / 2], t1 = rope[(int64_t)pos * (dd / 2) + col / 2 + 1];
  return f32x4{x[0] * t0.x + x[1] * t0.y, x[1] * t0.x - x[0] * t0.y, x[2] * t1.x + x[3] * t1.y, x[3] * t1.x - x[2] * t1.y};
}
// Blocks with the most work first, over all heads (a causal block's work grows with its distance from the start or the end).
struct Block { int rank, h, b; };
__device__ __forceinline__ Block block_of(int id, int nh, int mb) {
  const int nhb = nh * mb, hb = id % nhb;
  return Block{id / nhb, hb % nh, hb / nh};
}

// Sum of the waves' accumulators, quad by quad: wave w gets the sums of the quads q with q % KW == w, quad q as mine[q / KW].
template <int DS> __device__ __forceinline__ void merge(f32x4 (&mine)[DS / KW], f32x4* red, const f32x4 (&acc)[DS], int wave, int lane) {
#pragma unroll
  for (int q = 0; q < DS; ++q)
    if (q % KW != wave) red[((wave < q % KW ? wave : wave - 1) * DS + q) * 64 + lane] = quad<DS>(acc, q);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < DS; ++q)
    if (q % KW == wave) {
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int o = 0; o < KW; ++o) v += o == wave ? quad<DS>(acc, q) : red[((o < wave ? o : o - 1) * DS + q) * 64 + lane];
      mine[q / KW] = v;
    }
}

// Rows of the block that hold a non-finite value in any wave's quads, as bits 0..15.
__device__ __forceinline__ unsigned rows_of(unsigned* masks, float mark, int wave) {
  const unsigned long long m = __ballot(!(mark == 0.f));
  masks[wave] = (unsigned)((m | m >> 16 | m >> 32 | m >> 48) & 0xffffu);
  __syncthreads();
  unsigned rows = 0;
#pragma unroll
  for (int w = 0; w < KW; ++w) rows |= masks[w];
  return rows;
}
template <int DS> __device__ __forceinline__ float mark_of(const f32x4 (&x)[DS / KW]) {
  float mark = 0.f;
#pragma unroll
  for (int i = 0; i < DS / KW; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) mark = mark_non_finite(mark, x[i][e]);
  return mark;
}

// The rows `redo` of the block are dealt out over the waves.  Calls of their own, not inlined, so that the kernels' code stays
// what it is without them.
template <int DS>
__device__ __attribute__((noinline)) void redo_fwd_rows(float* rowbuf, unsigned redo, int q0, int dd, const float* q,
                                                        const float* k, const float* v, int64_t ld, float* o, int64_t ldo, float scale) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for_dealt_rows(&redo, 1, KW, wave, [&](int, int r) {
    float* row = o + (int64_t)(q0 + r) * ldo;
    attn_fwd_row<DS / 4>(rowbuf, q0 + r, dd, q, k, v, ld, scale, lane, [&](int c, float x) { row[c] = x; });
  });
}
template <int DS>
__device__ __attribute__((noinline)) void redo_dq_rows(float* rowbuf, unsigned redo, int q0, int dd, const float* q,
                                                       const float* k, const float* v, int64_t ld, const float* dout, int64_t ldo,
                                                       float li, float dlt, float scale, const float2* rope, float* dq, int64_t ldd) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for_dealt_rows(&redo, 1, KW, wave, [&](int, int r) {
    const int i = q0 + r;
    float* row = dq + (int64_t)i * ldd;
    attn_dq_row<DS / 4>(rowbuf, i, dd, q, k, v, ld, dout, ldo, __shfl(li, r, 64), __shfl(dlt, r, 64), scale, lane,
                        [&](int c, float x) { row[c] = rope ? unrotate_column(x, rope, i, c, dd) : x; });
  });
}
template <int DS>
__device__ __attribute__((noinline)) void redo_dkv_rows(float* rowbuf, unsigned redo, int k0, int S, int dd, const float* q,
                                                        const float* k, const float* v, int64_t ld, const float* dout, int64_t ldo,
                                                        const float* lse_h, const float* dlt_h, const float* o, float scale,
                                                        const float2* rope, float* dk, float* dv, int64_t ldd) {
  auto delta = [&](int i) {   // dlt_h = NULL: from the rows of O
    if (dlt_h) return dlt_h[i];
    float x = 0.f;
    for (int c = 0; c < dd; ++c) x = fmaf(dout[(int64_t)i * ldo + c], o[(int64_t)i * ldo + c], x);
    return x;
  };
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for_dealt_rows(&redo, 1, KW, wave, [&](int, int r) {
    const int j = k0 + r;
    const int64_t to = (int64_t)j * ldd;
    if (dkv_row_is_nan(j, S, lse_h, lane)) {
      for (int c = lane; c < dd; c += 64) dk[to + c] = dv[to + c] = NAN;
      return;
    }
    attn_dkv_row<DS / 4>(rowbuf, j, S, dd, q, k, v, ld, dout, ldo, lse_h, delta, scale, lane, [&](int c, float xk, float xv) {
      dk[to + c] = rope ? unrotate_column(xk, rope, j, c, dd) : xk;
      dv[to + c] = xv;
    });
  });
}

// ------------------------------------------------------------------------------------------ forward
// Two waves per SIMD are asked for, here and in the dK/dV kernel of 64 columns: left alone, the compiler takes more registers than two waves
// have (us, one : two waves: forward of 2 x 32 heads of 128, S = 512 90 : 63; backward of as many of 64 138 : 114).
template <int DS, int NBUF>
__global__ __attribute__((amdgpu_waves_per_eu(2))) __launch_bounds__(64 * KW) void attn_fwd_f32_kernel(int S, int dd, const float* __restrict__ q, const float* __restrict__ k,
                                                              const float* __restrict__ v, int64_t ld, float* __restrict__ o,
                                                              int64_t ldo, float* __restrict__ lse, float scale, int nh, int mb) {
  __shared__ f32x4 red[(KW - 1) * DS * 64];
  __shared__ float rowbuf[KW][32 * DS];   // rows that are redone
  __shared__ unsigned masks[KW];
  __shared__ float ms[KW][16], ls[KW][16];
  __shared__ Lines<DS> lines[KW];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Block blk = block_of(blockIdx.x, nh, mb);
  const int q0 = ((S + 15) / 16 - 1 - blk.rank) * 16, my_q = q0 + (lane & 15);
  const int64_t tok0 = (int64_t)blk.b * S;
  const Head hq = head_of(q + tok0 * ld + blk.h * dd, ld, S, dd), hk = head_of(k + tok0 * ld + blk.h * dd, ld, S, dd),
             hv = head_of(v + tok0 * ld + blk.h * dd, ld, S, dd);
  f32x4 qf[DS], acc[DS], buf[NBUF][DS];
  load_lines<DS>(qf, hq, q0, lane, dd);
#pragma unroll
  for (int s = 0; s < DS; ++s) acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  // fragments of a tile in the order of their use: K rows 0-15, K rows 16-31, V rows 0-15, V rows 16-31
  auto load = [&](f32x4 (&f)[DS], int step, int tile) {
    const int row0 = tile * TK + 16 * (step & 1);
    if (step < 2) load_lines<DS>(f, hk, row0, lane, dd); else load_r<DS>(f, hv, row0, lane, dd);
  };
  const int tiles = (min(q0 + 15, S - 1)) / TK + 1;
  if (wave < tiles) {
#pragma unroll
    for (int s = 0; s < NBUF - 1; ++s) load(buf[s], s, wave);
    to_k<DS>(qf, lines[wave], lane);
    for (int t = wave; t < tiles; t += KW) {
      f32x4 p[2];
#pragma unroll
      for (int step = 0; step < 4; ++step) {
        const int ahead = step + NBUF - 1;   // loads behind the last tile are issued and not used
        load(buf[ahead % NBUF], ahead % 4, ahead < 4 ? t : t + KW);
        if (step < 2) {
          to_k<DS>(buf[step % NBUF], lines[wave], lane);
          p[step] = dot<DS>(buf[step % NBUF], qf);
          if (step == 1) {
            const int key0 = t * TK + 4 * (lane >> 4);
            float mx = -INFINITY;
#pragma unroll
            for (int jb = 0; jb < 2; ++jb)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                // rounded before the maximum is taken off, so that the largest weight is exactly 1
                p[jb][r] = key0 + 16 * jb + r > my_q ? -INFINITY : __fmul_rn(p[jb][r], scale);
                mx = fmaxf(mx, p[jb][r]);
              }
            // the maximum of scale * score: key 0 is visible to every query, so it is finite from the first tile on for
            // wave 0; another wave may see nothing of a row yet and then keeps m = -inf and weights of zero
            const float mn = fmaxf(m, over_groups_max(mx));
            const float ref = mn == -INFINITY ? 0.f : mn, alpha = expf(m - ref);
            float sum = 0.f;
#pragma unroll
            for (int jb = 0; jb < 2; ++jb)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                p[jb][r] = expf(p[jb][r] - ref);
                sum += p[jb][r];
              }
            l = l * alpha + over_groups_sum(sum);
            m = mn;
#pragma unroll
            for (int s = 0; s < DS; ++s) acc[s] *= alpha;
          }
        } else {
          add_weighted<DS>(acc, buf[step % NBUF], p[step - 2]);
        }
      }
    }
  }
  if (lane < 16) { ms[wave][lane] = m; ls[wave][lane] = l; }
  __syncthreads();
  float mt = -INFINITY, lt = 0.f;
#pragma unroll
  for (int w = 0; w < KW; ++w) mt = fmaxf(mt, ms[w][lane & 15]);
#pragma unroll
  for (int w = 0; w < KW; ++w) lt += ls[w][lane & 15] * expf(ms[w][lane & 15] - mt);
  const float mine = expf(m - mt) / lt;   // a wave that saw no key: exp(-inf) = 0
#pragma unroll
  for (int s = 0; s < DS; ++s) acc[s] *= mine;
  f32x4 out[DS / KW];
  merge<DS>(out, red, acc, wave, lane);
  const unsigned redo = rows_of(masks, my_q < S && lt == lt ? mark_of<DS>(out) : 0.f, wave);
#pragma unroll
  for (int i = 0; i < DS / KW; ++i) {
    const int col = quad_col(KW * i + wave, lane);
    if (my_q < S && col < dd && !(redo >> (lane & 15) & 1)) *reinterpret_cast<f32x4*>(o + (tok0 + my_q) * ldo + blk.h * dd + col) = out[i];
  }
  if (__builtin_expect(redo != 0, 0)) {
    const int64_t at = tok0 * ld + blk.h * dd;
    redo_fwd_rows<DS>(rowbuf[wave], redo, q0, dd, q + at, k + at, v + at, ld, o + tok0 * ldo + blk.h * dd, ldo, scale);
  }
  if (wave == 0 && lane < 16 && my_q < S) lse[((int64_t)blk.b * nh + blk.h) * S + my_q] = mt + logf(lt);
}

// ------------------------------------------------------------------------------------------ dQ (and delta = dO . O)
template <int DS> struct BwdLds {
  f32x4 red[(KW - 1) * DS * 64];
  float rowbuf[KW][32 * DS];   // rows that are redone
  unsigned masks[KW];
  Lines<DS> lines[KW];
};
template <int DS, int NBUF>
__device__ __forceinline__ void dq_block(BwdLds<DS>& lds, int block, int S, int dd, const float* __restrict__ q, const float* __restrict__ k,
                                         const float* __restrict__ v, int64_t ld, const float* __restrict__ o, const float* __restrict__ dout,
                                         int64_t ldo, const float* __restrict__ lse, float* __restrict__ delta, float* __restrict__ dq,
                                         int64_t ldd, float scale, int nh, int mb, const float2* __restrict__ rope) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Block blk = block_of(block, nh, mb);
  const int q0 = ((S + 15) / 16 - 1 - blk.rank) * 16, my_q = q0 + (lane & 15);
  const int64_t tok0 = (int64_t)blk.b * S;
  const Head hq = head_of(q + tok0 * ld + blk.h * dd, ld, S, dd), hk = head_of(k + tok0 * ld + blk.h * dd, ld, S, dd),
             hv = head_of(v + tok0 * ld + blk.h * dd, ld, S, dd), ho = head_of(o + tok0 * ldo + blk.h * dd, ldo, S, dd),
             hdo = head_of(dout + tok0 * ldo + blk.h * dd, ldo, S, dd);
  f32x4 qf[DS], dof[DS], acc[DS], buf[NBUF][DS];
  load_lines<DS>(qf, hq, q0, lane, dd);
  load_lines<DS>(dof, hdo, q0, lane, dd);
  float dlt = 0.f;
  load_lines<DS>(acc, ho, q0, lane, dd);
  to_k<DS>(qf, lds.lines[wave], lane);
  to_k<DS>(dof, lds.lines[wave], lane);
  to_k<DS>(acc, lds.lines[wave], lane);
#pragma unroll
  for (int s = 0; s < DS; ++s)
#pragma unroll
    for (int e = 0; e < 4; ++e) dlt = fmaf(dof[s][e], acc[s][e], dlt);
  dlt = over_groups_sum(dlt);
  const int64_t stat = ((int64_t)blk.b * nh + blk.h) * S + min(my_q, S - 1);
  if (wave == 0 && lane < 16 && my_q < S) delta[stat] = dlt;
  const float li = lse[stat];
#pragma unroll
  for (int s = 0; s < DS; ++s) acc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
  // order of use: K, V of rows 0-15 by k, K, V of rows 16-31 by k, K of rows 0-15 and 16-31 by columns
  auto load = [&](f32x4 (&f)[DS], int step, int tile) {
    const int row0 = tile * TK;
    if (step < 4) load_lines<DS>(f, step & 1 ? hv : hk, row0 + 16 * (step >> 1), lane, dd);
    else load_r<DS>(f, hk, row0 + 16 * (step - 4), lane, dd);
  };
  const int tiles = min(q0 + 15, S - 1) / TK + 1;
  if (wave < tiles) {
#pragma unroll
    for (int s = 0; s < NBUF - 1; ++s) load(buf[s], s, wave);
    for (int t = wave; t < tiles; t += KW) {
      f32x4 sc, ds[2];
#pragma unroll
      for (int step = 0; step < 6; ++step) {
        const int ahead = step + NBUF - 1;
        load(buf[ahead % NBUF], ahead % 6, ahead < 6 ? t : t + KW);
        if (step < 4) {
          to_k<DS>(buf[step % NBUF], lds.lines[wave], lane);
          if (!(step & 1)) { sc = dot<DS>(buf[step % NBUF], qf); continue; }
          const f32x4 dp = dot<DS>(buf[step % NBUF], dof);
          const int key0 = t * TK + 16 * (step >> 1) + 4 * (lane >> 4);
#pragma unroll
          for (int r = 0; r < 4; ++r) ds[step >> 1][r] = key0 + r > my_q ? 0.f : expf(fmaf(sc[r], scale, -li)) * (dp[r] - dlt);
        } else {
          add_weighted<DS>(acc, buf[step % NBUF], ds[step - 4]);
        }
      }
    }
  }
  f32x4 out[DS / KW];
  merge<DS>(out, lds.red, acc, wave, lane);
  const unsigned redo = rows_of(lds.masks, my_q < S && li == li && dlt == dlt ? mark_of<DS>(out) : 0.f, wave);
#pragma unroll
  for (int i = 0; i < DS / KW; ++i) {
    const int col = quad_col(KW * i + wave, lane);
    if (my_q >= S || col >= dd || (redo >> (lane & 15) & 1)) continue;
    f32x4 x = out[i] * scale;
    if (rope) x = unrotate(x, rope, my_q, col, dd);
    *reinterpret_cast<f32x4*>(dq + (tok0 + my_q) * ldd + blk.h * dd + col) = x;
  }
  if (__builtin_expect(redo != 0, 0)) {
    const int64_t at = tok0 * ld + blk.h * dd;
    redo_dq_rows<DS>(lds.rowbuf[wave], redo, q0, dd, q + at, k + at, v + at, ld, dout + tok0 * ldo + blk.h * dd, ldo, li, dlt, scale,
                     rope, dq + tok0 * ldd + blk.h * dd, ldd);
  }
}

template <int DS, int NBUF>
__global__ __launch_bounds__(64 * KW) void attn_bwd_dq_f32_kernel(int S, int dd, const float* __restrict__ q, const float* __restrict__ k,
                                                                 const float* __restrict__ v, int64_t ld, const float* __restrict__ o,
                                                                 const float* __restrict__ dout, int64_t ldo,
                                                                 const float* __restrict__ lse, float* __restrict__ delta,
                                                                 float* __restrict__ dq, int64_t ldd, float scale, int nh, int mb,
                                                                 const float2* __restrict__ rope) {
  __shared__ BwdLds<DS> lds;
  dq_block<DS, NBUF>(lds, blockIdx.x, S, dd, q, k, v, ld, o, dout, ldo, lse, delta, dq, ldd, scale, nh, mb, rope);
}

// ------------------------------------------------------------------------------------------ dK, dV
// QBUF > 0: dQ (with QBUF buffers) and dK/dV in one launch, for grids that leave CUs idle when they run one after the other: the
// blocks from dkv_blocks on are dQ's.  No block reads what another one writes: delta of a tile's rows is formed here from dO and
// the same rows of O, in dQ's order of additions, instead of read.
template <int DS, int NBUF, int QBUF>
__global__ __attribute__((amdgpu_waves_per_eu(DS == 4 && !QBUF ? 2 : 1))) __launch_bounds__(64 * KW) void attn_bwd_dkv_f32_kernel(int S, int dd, const float* __restrict__ q, const float* __restrict__ k,
                                                                  const float* __restrict__ v, int64_t ld,
                                                                  const float* __restrict__ dout, int64_t ldo,
                                                                  const float* __restrict__ lse, const float* __restrict__ delta,
                                                                  float* __restrict__ dk, float* __restrict__ dv, int64_t ldd, float scale,
                                                                  int nh, int mb, const float2* __restrict__ rope, int dkv_blocks,
                                                                  const float* __restrict__ o, float* __restrict__ delta_out, float* __restrict__ dq) {
  constexpr bool BOTH = QBUF > 0;
  constexpr int R = BOTH ? 3 : 2, KSTEPS = 2 * R, STEPS = KSTEPS + 4;   // steps by k of 16 rows, of a tile, and all of a tile
  static_assert(STEPS % NBUF == 0, "a tile ends with the buffer before the one it began with");
  __shared__ BwdLds<DS> lds;
  if constexpr (BOTH)
    if ((int)blockIdx.x >= dkv_blocks) {
      dq_block<DS, QBUF>(lds, blockIdx.x - dkv_blocks, S, dd, q, k, v, ld, o, dout, ldo, lse, delta_out, dq, ldd, scale, nh, mb, rope);
      return;
    }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Block blk = block_of(blockIdx.x, nh, mb);
  const int k0 = blk.rank * 16, my_k = k0 + (lane & 15);
  const int64_t tok0 = (int64_t)blk.b * S;
  const Head hq = head_of(q + tok0 * ld + blk.h * dd, ld, S, dd), hk = head_of(k + tok0 * ld + blk.h * dd, ld, S, dd),
             hv = head_of(v + tok0 * ld + blk.h * dd, ld, S, dd), hdo = head_of(dout + tok0 * ldo + blk.h * dd, ldo, S, dd),
             ho = BOTH ? head_of(o + tok0 * ldo + blk.h * dd, ldo, S, dd) : hdo;
  const float* lse_h = lse + ((int64_t)blk.b * nh + blk.h) * S;
  const float* dlt_h = BOTH ? nullptr : delta + ((int64_t)blk.b * nh + blk.h) * S;
  f32x4 kf[DS], vf[DS], dka[DS], dva[DS], buf[NBUF][DS];
  load_lines<DS>(kf, hk, k0, lane, dd);
  load_lines<DS>(vf, hv, k0, lane, dd);
#pragma unroll
  for (int s = 0; s < DS; ++s) dka[s] = dva[s] = f32x4{0.f, 0.f, 0.f, 0.f};
  // order of use: Q, dO (BOTH: and O) of rows 0-15 by k, the same of rows 16-31, then by columns dO, Q of rows 0-15 and of rows 16-31
  auto load = [&](f32x4 (&f)[DS], int step, int tile) {
    if (step < KSTEPS) load_lines<DS>(f, step % R == 0 ? hq : step % R == 1 ? hdo : ho, tile * TK + 16 * (step / R), lane, dd);
    else load_r<DS>(f, (step - KSTEPS) & 1 ? hq : hdo, tile * TK + 16 * ((step - KSTEPS) >> 1), lane, dd);
  };
  const int first = k0 / TK + wave, tiles = (S + TK - 1) / TK;
  if (first < tiles) {
#pragma unroll
    for (int s = 0; s < NBUF - 1; ++s) load(buf[s], s, first);
    to_k<DS>(kf, lds.lines[wave], lane);
    to_k<DS>(vf, lds.lines[wave], lane);
    for (int t = first; t < tiles; t += KW) {
      f32x4 p[2], ds[2];
      float li[2][4], di[2][4];
#pragma unroll
      for (int ib = 0; ib < 2; ++ib)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = min(t * TK + 16 * ib + 4 * (lane >> 4) + r, S - 1);
          li[ib][r] = lse_h[i];
          if (!BOTH) di[ib][r] = dlt_h[i];
        }
      f32x4 dp;
#pragma unroll
      for (int step = 0; step < STEPS; ++step) {
        const int ib = step / R;
        if (step < KSTEPS) to_k<DS>(buf[step % NBUF], lds.lines[wave], lane);
        if (BOTH && step < KSTEPS && step % R == 2) {   // before the load into the buffer of dO
          float x = 0.f;
#pragma unroll
          for (int s = 0; s < DS; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) x = fmaf(buf[(step - 1) % NBUF][s][e], buf[step % NBUF][s][e], x);
          x = over_groups_sum(x);                        // row l%16
#pragma unroll
          for (int r = 0; r < 4; ++r) di[ib][r] = __shfl(x, 4 * (lane >> 4) + r, 64);
        }
        const int ahead = step + NBUF - 1;
        load(buf[ahead % NBUF], ahead % STEPS, ahead < STEPS ? t : t + KW);
        if (step < KSTEPS) {
          if (step % R == 0) { p[ib] = dot<DS>(buf[step % NBUF], kf); continue; }
          if (step % R == 1) dp = dot<DS>(buf[step % NBUF], vf);
          if (step % R != R - 1) continue;
          const int i0 = t * TK + 16 * ib + 4 * (lane >> 4);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            p[ib][r] = i0 + r < my_k || i0 + r >= S ? 0.f : expf(fmaf(p[ib][r], scale, -li[ib][r]));
            ds[ib][r] = i0 + r < my_k || i0 + r >= S ? 0.f : p[ib][r] * (dp[r] - di[ib][r]);
          }
        } else if (!((step - KSTEPS) & 1)) {
          add_weighted<DS>(dva, buf[step % NBUF], p[(step - KSTEPS) >> 1]);
        } else {
          add_weighted<DS>(dka, buf[step % NBUF], ds[(step - KSTEPS) >> 1]);
        }
      }
    }
  }
  f32x4 outv[DS / KW], outk[DS / KW];
  merge<DS>(outv, lds.red, dva, wave, lane);
  __syncthreads();   // the second merge reuses the buffer
  merge<DS>(outk, lds.red, dka, wave, lane);
  const unsigned redo = rows_of(lds.masks, my_k < S ? mark_of<DS>(outv) + mark_of<DS>(outk) : 0.f, wave);
#pragma unroll
  for (int i = 0; i < DS / KW; ++i) {
    const int col = quad_col(KW * i + wave, lane);
    if (my_k >= S || col >= dd || (redo >> (lane & 15) & 1)) continue;
    const int64_t to = (tok0 + my_k) * ldd + blk.h * dd + col;
    f32x4 x = outk[i] * scale;
    if (rope) x = unrotate(x, rope, my_k, col, dd);
    *reinterpret_cast<f32x4*>(dv + to) = outv[i];
    *reinterpret_cast<f32x4*>(dk + to) = x;
  }
  if (__builtin_expect(redo != 0, 0)) {
    const int64_t at = tok0 * ld + blk.h * dd;
    redo_dkv_rows<DS>(lds.rowbuf[wave], redo, k0, S, dd, q + at, k + at, v + at, ld, dout + tok0 * ldo + blk.h * dd, ldo, lse_h, dlt_h,
                      BOTH ? o + tok0 * ldo + blk.h * dd : nullptr, scale, rope, dk + tok0 * ldd + blk.h * dd, dv + tok0 * ldd + blk.h * dd, ldd);
  }
}

}  // namespace

// Aligned 16-byte pieces of rows through 32-bit offsets (with room for the tiles issued ahead), head dims up to 128.
bool attn_f32_supported(int mb, int S, int nh, int d, int64_t ld_max, uintptr_t pointers, int64_t strides) {
  return d <= 128 && (pointers & 15) == 0 && strides % 4 == 0 && ((int64_t)S + 16 * TK) * ld_max * 4 < (1ll << 30) &&
         cdiv(S, 16) * nh * mb < (1ll << 31);
}

hipError_t attn_fwd_f32(hipStream_t st, int mb, int S, int nh, int d, const void* q, const void* k, const void* v, int64_t ld, void* o,
                        int64_t ldo, float* lse) {
  dim3 grid((unsigned)(cdiv(S, 16) * nh * mb)), blk(64 * KW);
  const float scale = 1.0f / sqrtf((float)d);
  if (d <= 64)
    hipLaunchKernelGGL((attn_fwd_f32_kernel<4, 4>), grid, blk, 0, st, S, d, (const float*)q, (const float*)k, (const float*)v, ld,
                       (float*)o, ldo, lse, scale, nh, mb);
  else
    hipLaunchKernelGGL((attn_fwd_f32_kernel<8, 4>), grid, blk, 0, st, S, d, (const float*)q, (const float*)k, (const float*)v, ld,
                       (float*)o, ldo, lse, scale, nh, mb);
  return hipGetLastError();
}

hipError_t attn_bwd_f32(hipStream_t st, int mb, int S, int nh, int d, const void* q, const void* k, const void* v, int64_t ld,
                        const void* o, const void* dout, int64_t ldo, const float* lse, float* delta, void* dq, void* dk, void* dv,
                        int64_t ldd, const float2* rope) {
  const int64_t blocks = cdiv(S, 16) * nh * mb;
  const float scale = 1.0f / sqrtf((float)d);
  const float *qp = (const float*)q, *kp = (const float*)k, *vp = (const float*)v, *op = (const float*)o, *dop = (const float*)dout;
  float *dqp = (float*)dq, *dkp = (float*)dk, *dvp = (float*)dv;
  const dim3 blk(64 * KW);
  // Together up to 256 blocks, a CU each for every kernel's: the time is that of dK/dV and what dQ finds free beside it.  Separate :
  // together, us: S = 256, 4 heads of 128 (64 blocks) 38 : 26; S = 512, 8 of 128 (256) 61 : 52, 8 of 64 36 : 31; S = 1024, 4 of 128 (256) 105 : 81; S = 128, 30
  // of 64 (240) 18.0 : 17.2; S = 512, 2 x 6 of 128 (384) 77 : 75, 2 x 8 (512) 86 : 95.
  if (blocks <= 256 && attn_bwd_apart((int64_t)mb * S, 4ll * nh * d, k, v, 4 * ld, o, 4 * ldo, dq, dk, dv, 4 * ldd)) {
    auto kern = d <= 64 ? attn_bwd_dkv_f32_kernel<4, 10, 6> : attn_bwd_dkv_f32_kernel<8, 5, 3>;
    hipLaunchKernelGGL(kern, dim3((unsigned)(2 * blocks)), blk, 0, st, S, d, qp, kp, vp, ld, dop, ldo, lse, nullptr, dkp, dvp, ldd, scale, nh, mb,
                       rope, (int)blocks, op, delta, dqp);
    return hipGetLastError();
  }
  const dim3 grid((unsigned)blocks);
  auto kern_dq = d <= 64 ? attn_bwd_dq_f32_kernel<4, 6> : attn_bwd_dq_f32_kernel<8, 3>;
  auto kern_dkv = d <= 64 ? attn_bwd_dkv_f32_kernel<4, 8, 0> : attn_bwd_dkv_f32_kernel<8, 4, 0>;
  hipLaunchKernelGGL(kern_dq, grid, blk, 0, st, S, d, qp, kp, vp, ld, op, dop, ldo, lse, delta, dqp, ldd, scale, nh, mb, rope);
  hipLaunchKernelGGL(kern_dkv, grid, blk, 0, st, S, d, qp, kp, vp, ld, dop, ldo, lse, delta, dkp, dvp, ldd, scale, nh, mb, rope, 0, nullptr, nullptr,
                     nullptr);
  return hipGetLastError();
}

}  // namespace zs

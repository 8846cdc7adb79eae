// Flash-style causal attention on the CDNA4 matrix cores, 16-bit in, fp32 softmax: head dim 128, and (SPLIT) head dims below
// it, padded with zeros to D = 64, 96 or 128.
//
// The S x S score matrix is never stored: K/V (forward, dQ) or Q/dO (dK/dV) tiles of 64 rows are
// staged in LDS and every wavefront keeps its own 32 rows' operands and accumulators in
// registers.  All products are computed TRANSPOSED (S^T = K Q^T, O^T = V^T P^T, ...): with
// v_mfma_f32_32x32x16_bf16 a lane then owns one query (or key) column, so the softmax row
// maximum and sum are reductions over the lane's own registers plus one exchange with lane^32,
// and the fp32 accumulator registers of one product are, converted to bf16, already laid out
// as the B operand of the next one.  The A operands that need the transposed tile (V^T, K^T,
// dO^T, Q^T) are read with ds_read_b64_tr_b16, which hands a lane 4 values that are consecutive
// along the tile's ROW index, so tiles sit in LDS exactly as they sit in memory.
//
// Backward is two kernels without atomics (fixed summation order): one owns 128 queries and
// produces dQ, one owns 128 keys and produces dK and dV; both recompute P from the saved
// log-sum-exp.  delta_i = dO_i . O_i is formed by the dQ kernel for its own rows and stored for the other, or by both where they share a launch.
//
// SPLIT: probabilities and dS, fp32 in the wave-per-row kernel that served these head dims, go into the second product as a
// high and a low 16-bit part (two matrix instructions on the same A fragment), which together keep 16 (bf16) or 22 (half) of
// their 24 bits.  In half the low part is scaled by 2^11, and where small values matter absolutely (P and dS in the backward) it
// has accumulators of its own, so that it stays out of the subnormal range.  The errors against float64 are those of the
// wave-per-row kernel (S = 64 .. 4096, d = 64, 80, 96: 1.6e-3 to 1.9e-3 in bf16 and 2.0e-4 to 2.5e-4 in half, both the outputs'
// rounding, equal within 0.2 %; lse 2.3e-8 against 4.3e-8; 4 x 16 heads of 64, S = 1000: 4490 -> 100 us forward + backward in
// bf16).  The scores' factor and the row sums are kept a
// little better than one fp32 operation would (scale_lo, four partial sums), for the sake of lse, which is returned in fp32.
// A row whose sums are not finite is computed again in fp32, one wave per row: masked rows enter a product with weight zero,
// which does not hold off inf and NaN (attention_rows.h).
#include "kernels.h"
#include "attention_rows.h"

#include <cmath>

// This file is compiled four times: as it stands for bf16 and heads of 128, and through attention_mfma_f16.hip,
// attention_split.hip and attention_split_f16.hip, which define ZS_ATTN_F16 (IEEE half) and ZS_ATTN_SPLIT (narrower heads) and
// include it.  e16 is the 16-bit element type of the build; the builds differ in the conversions to and from float, the
// matrix-core instruction, the head dims and the names they export.  The two head-dim builds are apart because the dK/dV kernel
// of 128 uses all 256 registers: in one unit with the other kernels the compiler shares facts about common helpers, and a change
// there made it spill 6 of them inside its loop.
#ifdef ZS_ATTN_F16
#define ZS_ATTN_MFMA __builtin_amdgcn_mfma_f32_32x32x16_f16
#define ZS_ATTN_NAME(x) x##_f16
namespace zs { typedef f16 e16; typedef f16x8 e16x8; typedef f16x4 e16x4; }
#else
#define ZS_ATTN_MFMA __builtin_amdgcn_mfma_f32_32x32x16_bf16
#define ZS_ATTN_NAME(x) x
namespace zs { typedef bf16 e16; typedef bf16x8 e16x8; typedef bf16x4 e16x4; }
#endif


namespace zs {

namespace {

constexpr int TR = 64;             // rows of a staged tile
// Padded LDS row length in elements for (padded) head dim D: for D = 128, 304 bytes = 76 banks = 12 (mod 64).  The 16 rows
// that one cycle of a row-fragment read touches then start in 16 different 4-bank groups (no conflicts); the 4 rows x 64 bytes
// of a transposing read overlap in 4 of their 16 banks, the least any padding allows next to that.  D = 64 and 96 (44 and 60
// banks) spread the 16 rows as well.
template <int D> constexpr int LDT = D + 24;
template <int D> constexpr int TILE = TR * LDT<D>;     // elements of one staged tile
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

__device__ __forceinline__ e16x8 zero8() {
  e16x8 z;
#pragma unroll
  for (int i = 0; i < 8; ++i) z[i] = (e16)0.f;
  return z;
}

// A-operand fragment of a row-major LDS tile: lane (row = lane%32, g = lane/32) gets 8 consecutive columns.
template <int D> __device__ __forceinline__ e16x8 lds_frag(const e16* tile, int row0, int col0, int lane) {
  return *reinterpret_cast<const e16x8*>(tile + (row0 + (lane & 31)) * LDT<D> + col0 + 8 * (lane >> 5));
}

// A-operand fragment of the TRANSPOSE of a row-major LDS tile M[k][n]: lane (i = lane%32, g = lane/32)
// gets M[k][n0+i] for the 8 contraction slots  k = k0 + 4g + {0,1,2,3, 8,9,10,11}.  This slot order is
// the order in which a lane's accumulator registers 8s..8s+7 of a 32-row MFMA block hold rows, so the
// matching B operand is just those registers.
template <int D> __device__ __forceinline__ e16x8 lds_frag_tr(const e16* tile, int k0, int n0, int lane) {
  const int r = lane & 15, gi = lane >> 4;
  const e16* p = tile + (k0 + 4 * (gi >> 1) + (r >> 2)) * LDT<D> + n0 + 16 * (gi & 1) + 4 * (r & 3);
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 8 * LDT<D>));
  union { struct { s16x4 a, b; } s; e16x8 v; } u;
  u.s.a = lo;
  u.s.b = hi;
  return u.v;
}

__device__ __forceinline__ e16x8 pack8(const f32x16& a, int s) {
  e16x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = (e16)a[8 * s + e];
  return o;
}

// pack8 as a high and a low part: a = hi + lo * LO_UNIT up to 2^-17 (bf16) or 2^-22 (half) of it.
#ifdef ZS_ATTN_F16
constexpr float LO_SCALE = 2048.0f;   // the low half part is stored times 2^11
constexpr bool LO_ACC = true;         // and needs accumulators of its own
#else
constexpr float LO_SCALE = 1.0f;
constexpr bool LO_ACC = false;
#endif
constexpr float LO_UNIT = 1.0f / LO_SCALE;
// dS goes in times 2^-4 in half, which leaves 2^20 of range on top; its low part still resolves 2^-32.  Above that the high part
// is inf and the sums of the row are not finite, so the row is redone in fp32 and keeps the fp32 kernel's range.
constexpr float DS_SCALE = LO_ACC ? 0.0625f : 1.0f;
__device__ __forceinline__ e16x8 pack8_lo(const f32x16& a, int s, const e16x8& hi, float lo_scale) {
  e16x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = (e16)((a[8 * s + e] - (float)hi[e]) * lo_scale);
  return o;
}

// A 64 x D tile moves HBM -> registers (fetch, issued before the MFMAs of the current tile so the
// latency hides behind them) -> LDS (put, after them).  For D = 128 thread t carries 4 vectors of 16 bytes:
// vector v = t + 256 i is row v/16, columns 8*(v%16)...
template <int NT, int D> struct TileRegs { e16x8 v[(8 * D + NT - 1) / NT]; };   // NT threads share the 64 D/8 vectors of a tile
// Rows of one (batch, head) are read through a raw buffer descriptor over [first row, last row's dd columns]:
// the per-lane offset is one register (D = 96: three), the tile's row offset a scalar, and rows at or past nrows fall
// beyond num_records and read as zero without a branch, as do the columns dd..D-1 of a padded head, whose offset is pushed
// there.  Offsets are 32-bit: nrows * ld * 2 < 2^31.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t head_rsrc(const e16* base, int64_t ld, int nrows, int dd) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<e16*>(base), 0, (int)((((int64_t)nrows - 1) * ld + dd) * 2), 0x00020000);
}
template <int NT, int D>
__device__ __forceinline__ void fetch_tile(TileRegs<NT, D>& x, __amdgpu_buffer_rsrc_t rs, int ld, int row0, unsigned tid, int dd) {
  constexpr unsigned RV = D / 8;   // vectors per row
#pragma unroll
  for (int i = 0; i < (8 * D + NT - 1) / NT; ++i) {
    union { u32x4 u; e16x8 h; } c;
    if constexpr (NT % RV == 0) {
      const int col = (int)(tid % RV) * 8;
      const int voff = col < dd ? ((int)(tid / RV) * ld + col) * 2 : (int)0x80000000;
      c.u = __builtin_amdgcn_raw_buffer_load_b128(rs, voff, (row0 + (int)(NT / RV) * i) * ld * 2, 0);
    } else {
      const unsigned v = tid + NT * i;
      const int col = (int)(v % RV) * 8;
      const int voff = col < dd ? ((int)(v / RV) * ld + col) * 2 : (int)0x80000000;
      c.u = __builtin_amdgcn_raw_buffer_load_b128(rs, voff, row0 * ld * 2, 0);
    }
    x.v[i] = c.h;
  }
}
template <int NT, int D> __device__ __forceinline__ void put_tile(const TileRegs<NT, D>& x, e16* tile, unsigned tid) {
#pragma unroll
  for (int i = 0; i < (8 * D + NT - 1) / NT; ++i) {
    const unsigned v = tid + NT * i;
    if (8 * D % NT != 0 && v >= 8 * D) break;   // D = 96 on 512 threads
    *reinterpret_cast<e16x8*>(tile + (v / (D / 8)) * LDT<D> + (v % (D / 8)) * 8) = x.v[i];
  }
}

// Row fragments kept in registers for a whole kernel: lane (row = row0 + lane%32, g) holds, for each of the D/16 contraction steps over
// d, 8 consecutive elements.  Rows >= nrows and columns >= dd read as zero.
template <int D>
__device__ __forceinline__ void load_row_frags(e16x8 (&f)[D / 16], const e16* __restrict__ src, int64_t ld, int row0,
                                               int nrows, int lane, int dd) {
  const int row = row0 + (lane & 31);
#pragma unroll
  for (int s = 0; s < D / 16; ++s) {
    const int c = 16 * s + 8 * (lane >> 5);
    f[s] = row < nrows && c < dd ? *reinterpret_cast<const e16x8*>(src + (int64_t)row * ld + c) : zero8();
  }
}
// The same by way of LDS: the wave's 32 rows come as whole lines (load_lines) and change places in its own part of the LDS (to_frags; 32
// rows of LDT).  Read as fragments, the lanes of a load lie in 32 rows, and the address unit takes four times as long for their
// pieces; the same holds for stores of accumulators (store_rows).  The backward kernels load up to three blocks of rows that way
// and store two; in the forward, whose only block is Q, the way round costs more than it saves (16 heads of 128, S = 2048: 46.3 us
// with direct loads, 49.4 without), and only the store goes through LDS.  us, fragments : lines, backward of 16 heads of 128, S =
// 2048 98.9 : 83.0; 32 heads, S = 4096 460 : 447; 4 heads, S = 256 19.8 : 16.3.  Where a CU has few waves at work on rows, as in short
// sequences, there is no queue before the address unit and the way round only adds its latencies: see lines_fwd.
template <int D>
__device__ __forceinline__ void load_lines(e16x8 (&f)[D / 16], const e16* __restrict__ src, int64_t ld, int row0, int nrows, int lane, int dd) {
  constexpr int P = D / 8;   // 16-byte pieces of a row
#pragma unroll
  for (int i = 0; i < D / 16; ++i) {
    const int v = lane + 64 * i, row = row0 + v / P, c = v % P * 8;
    f[i] = row < nrows && c < dd ? *reinterpret_cast<const e16x8*>(src + (int64_t)row * ld + c) : zero8();
  }
}
template <int D> __device__ __forceinline__ void to_frags(e16x8 (&f)[D / 16], e16* rows, int lane) {
  wave_lds_order();   // the rows before have been read
#pragma unroll
  for (int i = 0; i < D / 16; ++i) {
    const int v = lane + 64 * i;
    *reinterpret_cast<e16x8*>(rows + v / (D / 8) * LDT<D> + v % (D / 8) * 8) = f[i];
  }
  wave_lds_order();
#pragma unroll
  for (int s = 0; s < D / 16; ++s) f[s] = lds_frag<D>(rows, 0, 16 * s, lane);
}
// Rows row0 .. of dst, but those past nrows and those marked in `skip`, from a wave's accumulators.
template <int D>
__device__ __forceinline__ void store_rows(const f32x16 (&acc)[D / 32], float factor, e16* rows, e16* dst, int64_t ld, int row0, int nrows, int lane,
                                           int dd, unsigned skip) {
  wave_lds_order();
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      e16x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = (e16)(acc[db][4 * c + e] * factor);
      *reinterpret_cast<e16x4*>(rows + (lane & 31) * LDT<D> + db * 32 + 8 * c + 4 * (lane >> 5)) = w;
    }
  wave_lds_order();
  constexpr int P = D / 4;   // 8-byte pieces of a row, as aligned as a direct store's would be
#pragma unroll
  for (int i = 0; i < D / 8; ++i) {
    const int v = lane + 64 * i, r = v / P, c = v % P * 4;
    const e16x4 w = *reinterpret_cast<const e16x4*>(rows + r * LDT<D> + c);
    if (row0 + r < nrows && c < dd && !(skip >> r & 1)) *reinterpret_cast<e16x4*>(dst + (int64_t)(row0 + r) * ld + c) = w;
  }
}

// The same straight from the accumulators, every lane into the row that it holds.
template <int D, bool SPLIT>
__device__ __forceinline__ void store_direct(const f32x16 (&acc)[D / 32], float factor, e16* dst, int64_t ld, int row, int nrows, int lane, int dd,
                                             unsigned skip) {
  if (row >= nrows || skip >> (lane & 31) & 1) return;
  e16* to = dst + (int64_t)row * ld;
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int col = db * 32 + 8 * c + 4 * (lane >> 5);
      if (SPLIT && col >= dd) continue;
      e16x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = (e16)(acc[db][4 * c + e] * factor);
      *reinterpret_cast<e16x4*>(to + col) = w;
    }
}

// Row index (inside a 32-row MFMA block) held by accumulator register r of this lane.
__device__ __forceinline__ int acc_row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }

// Causal blocks differ in work by up to the number of tiles, so the launch order matters: workgroups are
// dispatched in increasing linear id, and id -> (rank, head) with the rank (0 = most work) in the slow
// position puts the heavy blocks of ALL heads first and leaves light blocks for the tail.  Consecutive
// ids go to different XCDs round-robin; with nh*mb a multiple of 8 a head keeps its XCD, whose L2 then
// holds the K/V (or Q/dO) rows its blocks stream.
struct BlockId { int rank, h, b; };
__device__ __forceinline__ BlockId block_id(int id, int nh, int mb) {
  const int nhb = nh * mb, hb = id % nhb;
  return BlockId{id / nhb, hb % nh, hb / nh};
}

// Inverse rotary rotation of a lane's columns of position pos, as the accumulators hold them (4 consecutive head-dim values, two
// adjacent pairs, per block and quad): (u, w) -> (u c + w s, -u s + w c).  All angles (LOADS blocks' worth) are read before the
// first is used, and before the caller's first store: a wait for a load behind a store waits for the store as well, and one
// load, wait and store after the other was 16 memory latencies at the end of the kernel (a small LLaMA step, 2 x 16 launches at
// S = 256: 2807 -> 2790 us).
typedef float f32x4v __attribute__((ext_vector_type(4)));
template <int D, int LOADS>
__device__ __forceinline__ void unrotate_row(f32x16 (&x)[D / 32], const float2* __restrict__ rope, int pos, int lane, int dd) {
  const float2* row = rope + (int64_t)pos * (dd / 2);
#pragma unroll
  for (int d0 = 0; d0 < D / 32; d0 += LOADS) {
    f32x4v t[LOADS][4];   // (cos, sin) x 2
#pragma unroll
    for (int i = 0; i < LOADS; ++i)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int col = (d0 + i) * 32 + 8 * c + 4 * (lane >> 5);
        if (d0 + i < D / 32) t[i][c] = *reinterpret_cast<const f32x4v*>(row + (col < dd ? col / 2 : 0));   // columns past dd are not stored
      }
#pragma unroll
    for (int i = 0; i < LOADS; ++i)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if (d0 + i >= D / 32) continue;
        f32x16& a = x[d0 + i < D / 32 ? d0 + i : 0];
        const float c = t[i][j / 2][2 * (j % 2)], sn = t[i][j / 2][2 * (j % 2) + 1], u = a[2 * j], w = a[2 * j + 1];
        a[2 * j] = u * c + w * sn;
        a[2 * j + 1] = w * c - u * sn;
      }
  }
}

// acc (+ its low part) of the second of two waves that share rows is added to the first one's through LDS: 16 KB per pair for
// D = 128.  LDS must be free; it is free again when the call returns.
template <int D, int NL>
__device__ __forceinline__ void merge_halves(f32x16 (&acc)[D / 32], f32x16 (&lo)[NL], f32x4* red, int half, int wave, int lane) {
  if constexpr (NL > 1) {
#pragma unroll
    for (int i = 0; i < D / 32; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][r] = fmaf(lo[i][r], LO_UNIT, acc[i][r]);
  }
  red += wave * (D / 32) * 4 * 64;
  if (half == 1) {
#pragma unroll
    for (int i = 0; i < D / 32; ++i)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        red[(i * 4 + c) * 64 + lane] = f32x4{acc[i][4 * c], acc[i][4 * c + 1], acc[i][4 * c + 2], acc[i][4 * c + 3]};
  }
  __syncthreads();
  if (half == 0) {
#pragma unroll
    for (int i = 0; i < D / 32; ++i)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const f32x4 o = red[(i * 4 + c) * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][4 * c + e] += o[e];
      }
  }
  __syncthreads();
}

// SPLIT: rows whose sums are not finite are redone, see attention_rows.h.  For that the LDS, free after the last tile, holds two
// rows per wave, then the rows' bits per group of 32 (lane and lane ^ 32 hold a row's columns), then (dQ) delta of the rows.
template <int N> __device__ __forceinline__ float mark_of(const f32x16 (&x)[N]) {
  float mark[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) mark[r % 4] = mark_non_finite(mark[r % 4], x[i][r]);
  return (mark[0] + mark[1]) + (mark[2] + mark[3]);
}
template <int NW> struct RedoLds { float rows[NW][256]; unsigned masks[NW]; float delta[NW * 32]; };
// A wave's 32 rows for store_rows: behind what redone rows need, at the start of the LDS where none are.
template <int NW, int D, bool SPLIT> __device__ __forceinline__ e16* rows_lds(char* smem, int wave) {
  return reinterpret_cast<e16*>(smem + (SPLIT ? (sizeof(RedoLds<NW>) + 15) / 16 * 16 : 0)) + wave * 32 * LDT<D>;
}
template <int NW> __device__ __forceinline__ RedoLds<NW>& redo_lds(char* smem) { return *reinterpret_cast<RedoLds<NW>*>(smem); }
// Publishes the rows of this wave's group; writer: one wave per group.
template <int NW> __device__ __forceinline__ unsigned rows_of(RedoLds<NW>& lds, int group, bool writer, bool live, float mark) {
  const unsigned long long m = __ballot(live && !(mark == 0.f));
  const unsigned rows = (unsigned)m | (unsigned)(m >> 32);
  if (writer) lds.masks[group] = rows;
  __syncthreads();
  return rows;
}

// Calls of their own, not inlined: with this code inside, the dQ and dK/dV kernels are scheduled for fewer registers and issue
// their LDS reads later (4 x 16 heads of 64, S = 1000: dQ 32.3 -> 33.9 us, 32.6 with the call).
template <int NW>
__device__ __attribute__((noinline)) void redo_fwd_rows(char* smem, int q0, int dd, const e16* qh, const e16* kh,
                                                        const e16* vh, int64_t ld, e16* oh, int64_t ldo) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  RedoLds<NW>& rl = redo_lds<NW>(smem);
  for_dealt_rows(rl.masks, NW, NW, wave, [&](int g, int r) {
    const int i = q0 + 32 * g + r;
    attn_fwd_row<2>(rl.rows[wave], i, dd, qh, kh, vh, ld, 1.0f / sqrtf((float)dd), lane, [&](int c, float x) { oh[(int64_t)i * ldo + c] = (e16)x; });
  });
}
template <int NW>
__device__ __attribute__((noinline)) void redo_dq_rows(char* smem, int groups, int q0, int dd, const e16* qh,
                                                       const e16* kh, const e16* vh, int64_t ld, const e16* doh, int64_t ldo,
                                                       const float* lse_h, float scale, const float2* rope, e16* dqh, int64_t ldd) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  RedoLds<NW>& rl = redo_lds<NW>(smem);
  for_dealt_rows(rl.masks, groups, NW, wave, [&](int g, int r) {
    const int i = q0 + 32 * g + r;
    attn_dq_row<2>(rl.rows[wave], i, dd, qh, kh, vh, ld, doh, ldo, lse_h[i], rl.delta[32 * g + r], scale, lane, [&](int c, float x) {
      dqh[(int64_t)i * ldd + c] = (e16)(rope ? unrotate_column(x, rope, i, c, dd) : x);
    });
  });
}
template <int NW>
__device__ __attribute__((noinline)) void redo_dkv_rows(char* smem, int groups, int k0, int S, int dd, const e16* qh,
                                                        const e16* kh, const e16* vh, int64_t ld, const e16* doh, int64_t ldo,
                                                        const float* lse_h, const float* dlt_h, float scale, const float2* rope,
                                                        e16* dkh, e16* dvh, int64_t ldd) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  RedoLds<NW>& rl = redo_lds<NW>(smem);
  for_dealt_rows(rl.masks, groups, NW, wave, [&](int g, int r) {
    const int j = k0 + 32 * g + r;
    const int64_t to = (int64_t)j * ldd;
    if (dkv_row_is_nan(j, S, lse_h, lane)) {
      for (int c = lane; c < dd; c += 64) dkh[to + c] = dvh[to + c] = (e16)NAN;
      return;
    }
    attn_dkv_row<2>(rl.rows[wave], j, S, dd, qh, kh, vh, ld, doh, ldo, lse_h, [&](int i) { return dlt_h[i]; }, scale, lane, [&](int c, float xk, float xv) {
      dkh[to + c] = (e16)(rope ? unrotate_column(xk, rope, j, c, dd) : xk);
      dvh[to + c] = (e16)xv;
    });
  });
}

// ------------------------------------------------------------------------------------------ forward
// grid ceil(S/(32 NW))*nh*mb, NW waves; wave w owns queries q0 + 32w .. +31; heavy (late) blocks are launched first.
// NW = 4: two workgroups per CU.  NW = 8: one workgroup per CU whose staged K/V tiles serve 256 queries, so a wave
// issues half as many tile loads and LDS stores per key tile (used when that still gives every CU a workgroup).
template <int NW, int D, bool SPLIT, bool LINES>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 2 : 1) void attn_fwd_kernel(int S, const e16* __restrict__ q, const e16* __restrict__ k,
                                                       const e16* __restrict__ v, int64_t ld, e16* __restrict__ o,
                                                       int64_t ldo, float* __restrict__ lse, float scale_log2, float scale_lo,
                                                       int nh, int mb, int head_dim) {
  const int dd = SPLIT ? head_dim : D;
  extern __shared__ __align__(16) char smem_raw[];
  e16* smem = reinterpret_cast<e16*>(smem_raw);            // [2][K tile | V tile]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const BlockId bid = block_id(blockIdx.x, nh, mb);
  const int qb = (S + 32 * NW - 1) / (32 * NW) - 1 - bid.rank, h = bid.h, b = bid.b;
  const int64_t tok0 = (int64_t)b * S;
  const e16* qh = q + tok0 * ld + h * dd;
  const e16* kh = k + tok0 * ld + h * dd;
  const e16* vh = v + tok0 * ld + h * dd;
  const __amdgpu_buffer_rsrc_t rsk = head_rsrc(kh, ld, S, dd), rsv = head_rsrc(vh, ld, S, dd);
  const int q0 = qb * 32 * NW, wq0 = q0 + wave * 32;
  const int my_q = wq0 + (lane & 31);

  e16x8 qf[D / 16];
  load_row_frags<D>(qf, qh, ld, wq0, S, lane, dd);
  f32x16 oacc[D / 32];
#pragma unroll
  for (int i = 0; i < D / 32; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[i][r] = 0.f;
  float m = -INFINITY, l = 0.f;

  const int last_q = min(q0 + 32 * NW - 1, S - 1);
  const int ntiles = last_q / TR + 1;
  TileRegs<64 * NW, D> kr, vr;
  fetch_tile(kr, rsk, (int)ld, 0, tid, dd);
  fetch_tile(vr, rsv, (int)ld, 0, tid, dd);
  put_tile(kr, smem, tid);
  put_tile(vr, smem + TILE<D>, tid);
  __syncthreads();
  for (int t = 0; t < ntiles; ++t) {
    const e16* Kt = smem + (t & 1) * 2 * TILE<D>;
    const e16* Vt = Kt + TILE<D>;
    if (t + 1 < ntiles) {
      fetch_tile(kr, rsk, (int)ld, (t + 1) * TR, tid, dd);
      fetch_tile(vr, rsv, (int)ld, (t + 1) * TR, tid, dd);
    }
    const int key0 = t * TR;
    if (key0 <= wq0 + 31) {   // otherwise every key of the tile is in this wave's future
      f32x16 sacc[2];
#pragma unroll
      for (int jb = 0; jb < 2; ++jb) {
#pragma unroll
        for (int r = 0; r < 16; ++r) sacc[jb][r] = 0.f;
#pragma unroll
        for (int s = 0; s < D / 16; ++s)
          sacc[jb] = ZS_ATTN_MFMA(lds_frag<D>(Kt, jb * 32, 16 * s, lane), qf[s], sacc[jb], 0, 0, 0);
      }
      if (key0 + TR - 1 > wq0) {   // tile touches the diagonal: mask keys in the future of this lane's query
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (key0 + jb * 32 + acc_row(r, lane) > my_q) sacc[jb][r] = -INFINITY;
      }
      float mx = -INFINITY;
#pragma unroll
      for (int jb = 0; jb < 2; ++jb)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[jb][r]);
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64)) * scale_log2;   // scale > 0, so the maximum commutes with it
      // Lazy rescaling: the reference maximum m only moves when some row's maximum grew by more than 2^8;
      // until then P is formed against the old reference (values up to 2^8, harmless in e16/fp32) and the
      // 64 accumulator registers are left alone.  m, l and O always refer to the same reference, so
      // O/l and m + log2(l) are exact whatever the schedule of updates.
      if (__any(mx > m + 8.0f)) {
        const float mn = fmaxf(m, mx);          // finite: key 0 is visible to every query in the first tile
        const float alpha = __builtin_amdgcn_exp2f(m - mn);
        l *= alpha;
        m = mn;
#pragma unroll
        for (int i = 0; i < D / 32; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[i][r] *= alpha;
      }
      float rs = 0.f, part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int jb = 0; jb < 2; ++jb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float x = fmaf(sacc[jb][r], scale_log2, -m);
          if constexpr (SPLIT) x = fmaf(sacc[jb][r], scale_lo, x);
          const float p = __builtin_amdgcn_exp2f(x);
          sacc[jb][r] = p;
          if constexpr (SPLIT) part[r & 3] += p;
          else rs += p;
        }
      if constexpr (SPLIT) rs = (part[0] + part[1]) + (part[2] + part[3]);
      rs += __shfl_xor(rs, 32, 64);
      l += rs;
#pragma unroll
      for (int jb = 0; jb < 2; ++jb)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          const e16x8 pf = pack8(sacc[jb], s2);
          e16x8 pl = pf;
          if constexpr (SPLIT) pl = pack8_lo(sacc[jb], s2, pf, 1.0f);   // P <= 2^8 of a sum l >= 1: no low accumulator needed
#pragma unroll
          for (int db = 0; db < D / 32; ++db) {
            const e16x8 vf = lds_frag_tr<D>(Vt, jb * 32 + 16 * s2, db * 32, lane);
            oacc[db] = ZS_ATTN_MFMA(vf, pf, oacc[db], 0, 0, 0);
            if constexpr (SPLIT) oacc[db] = ZS_ATTN_MFMA(vf, pl, oacc[db], 0, 0, 0);
          }
        }
    }
    if (t + 1 < ntiles) {   // the other buffer was last read before the barrier that ended the previous iteration
      put_tile(kr, smem + ((t + 1) & 1) * 2 * TILE<D>, tid);
      put_tile(vr, smem + ((t + 1) & 1) * 2 * TILE<D> + TILE<D>, tid);
    }
    __syncthreads();
  }
  unsigned redo = 0;
  if constexpr (SPLIT) redo = rows_of(redo_lds<NW>(smem_raw), wave, true, my_q < S && l == l, mark_of(oacc));
  if constexpr (LINES) store_rows<D>(oacc, 1.0f / l, rows_lds<NW, D, SPLIT>(smem_raw, wave), o + tok0 * ldo + h * dd, ldo, wq0, S, lane, dd, redo);
  else store_direct<D, SPLIT>(oacc, 1.0f / l, o + tok0 * ldo + h * dd, ldo, my_q, S, lane, dd, redo);
  if (my_q < S) {
    if (lane < 32)   // SPLIT: formed in double, once per row: m may lag the maximum by 8, so log l alone would round like lse does
      lse[((int64_t)b * nh + h) * S + my_q] =
          SPLIT ? (float)((double)m * 0.6931471805599453 + log((double)l)) : (m + log2f(l)) * LN2;
  }
  if constexpr (SPLIT) {
    if (__builtin_expect(any_row(redo_lds<NW>(smem_raw).masks, NW, lane), 0))
      redo_fwd_rows<NW>(smem_raw, q0, dd, qh, kh, vh, ld, o + tok0 * ldo + h * dd, ldo);
  }
}

// ------------------------------------------------------------------------------------------ dQ
// grid ceil(S/(32 NW))*nh*mb, NW waves (4 or 8 as in the forward kernel); wave w owns queries q0+32w..; loops over K/V
// tiles up to the diagonal.
// dQ^T[d][q] += K^T[d][key] dS^T[key][q],  dS^T = P^T o (dP^T - delta_q),  dP^T = V dO^T.
// QS = 2: two waves share 32 queries, each taking one half of every tile's keys; their sums meet in LDS at the end.
template <int NW, int QS, int D, bool SPLIT, bool LINES>
__device__ __forceinline__ void dq_block(int block, int S, const e16* __restrict__ q, const e16* __restrict__ k, const e16* __restrict__ v, int64_t ld,
                                         const e16* __restrict__ o, const e16* __restrict__ dout, int64_t ldo, const float* __restrict__ lse,
                                         float* __restrict__ delta, e16* __restrict__ dq, int64_t ldd, float scale, int nh, int mb,
                                         const float2* __restrict__ rope, int head_dim) {
  const int dd = SPLIT ? head_dim : D;
  extern __shared__ __align__(16) char smem_raw[];
  e16* smem = reinterpret_cast<e16*>(smem_raw);
  constexpr int QW = NW / QS;   // groups of 32 queries
  const int tid = threadIdx.x, lane = tid & 63, wave = QS == 1 ? tid >> 6 : (tid >> 6) % QW, half = QS == 1 ? 0 : (tid >> 6) / QW;
  const BlockId bid = block_id(block, nh, mb);
  const int qb = (S + 32 * QW - 1) / (32 * QW) - 1 - bid.rank, h = bid.h, b = bid.b;
  const int64_t tok0 = (int64_t)b * S;
  const e16* qh = q + tok0 * ld + h * dd;
  const e16* kh = k + tok0 * ld + h * dd;
  const e16* vh = v + tok0 * ld + h * dd;
  const e16* doh = dout + tok0 * ldo + h * dd;
  const __amdgpu_buffer_rsrc_t rsk = head_rsrc(kh, ld, S, dd), rsv = head_rsrc(vh, ld, S, dd);
  const int q0 = qb * 32 * QW, wq0 = q0 + wave * 32;
  const int my_q = wq0 + (lane & 31);
  const float scale_log2 = scale * LOG2E;

  TileRegs<64 * NW, D> kr, vr;   // the first tiles are in flight while delta is formed
  fetch_tile(kr, rsk, (int)ld, 0, tid, dd);
  fetch_tile(vr, rsv, (int)ld, 0, tid, dd);
  e16x8 qf[D / 16], dof[D / 16];
  e16x8 of[D / 16];
  if constexpr (LINES) {
    load_lines<D>(qf, qh, ld, wq0, S, lane, dd);
    load_lines<D>(dof, doh, ldo, wq0, S, lane, dd);
    load_lines<D>(of, o + tok0 * ldo + h * dd, ldo, wq0, S, lane, dd);
  } else {
    load_row_frags<D>(qf, qh, ld, wq0, S, lane, dd);
    load_row_frags<D>(dof, doh, ldo, wq0, S, lane, dd);
  }
  const int64_t stat = ((int64_t)b * nh + h) * S + min(my_q, S - 1);
  const float lse2 = lse[stat] * LOG2E;
  // delta_q = dO_q . O_q: each lane sums its 64 of the row's 128 products, lane^32 holds the others.
  // The value is also stored for the dK/dV kernel, which runs after this one.
  float dlt = 0.f;
  {
    if constexpr (LINES) {
      e16* rows = smem + (tid >> 6) * 32 * LDT<D>;
      to_frags<D>(qf, rows, lane);
      to_frags<D>(dof, rows, lane);
      to_frags<D>(of, rows, lane);
    } else load_row_frags<D>(of, o + tok0 * ldo + h * dd, ldo, wq0, S, lane, dd);
#pragma unroll
    for (int s = 0; s < D / 16; ++s)
#pragma unroll
      for (int e = 0; e < 8; ++e) dlt = fmaf((float)dof[s][e], (float)of[s][e], dlt);
    dlt += __shfl_xor(dlt, 32, 64);
    if (half == 0 && lane < 32 && my_q < S) delta[stat] = dlt;
  }
  f32x16 acc[D / 32], acclo[SPLIT && LO_ACC ? D / 32 : 1];
#pragma unroll
  for (int i = 0; i < D / 32; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) { acc[i][r] = 0.f; if (SPLIT && LO_ACC) acclo[SPLIT && LO_ACC ? i : 0][r] = 0.f; }

  const int last_q = min(q0 + 32 * QW - 1, S - 1);
  const int ntiles = last_q / TR + 1;
  if (LINES) __syncthreads();
  put_tile(kr, smem, tid);
  put_tile(vr, smem + TILE<D>, tid);
  __syncthreads();
  for (int t = 0; t < ntiles; ++t) {
    const e16* Kt = smem + (t & 1) * 2 * TILE<D>;
    const e16* Vt = Kt + TILE<D>;
    if (t + 1 < ntiles) {
      fetch_tile(kr, rsk, (int)ld, (t + 1) * TR, tid, dd);
      fetch_tile(vr, rsv, (int)ld, (t + 1) * TR, tid, dd);
    }
    const int key0 = t * TR;
    if (key0 <= wq0 + 31) {
      const bool diag = key0 + TR - 1 > wq0;
#pragma unroll
      for (int j = 0; j < 2 / QS; ++j) {
        const int jb = QS == 2 ? half : j;
        f32x16 sacc, pacc;
#pragma unroll
        for (int r = 0; r < 16; ++r) sacc[r] = pacc[r] = 0.f;
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
          sacc = ZS_ATTN_MFMA(lds_frag<D>(Kt, jb * 32, 16 * s, lane), qf[s], sacc, 0, 0, 0);
          pacc = ZS_ATTN_MFMA(lds_frag<D>(Vt, jb * 32, 16 * s, lane), dof[s], pacc, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) sacc[r] = __builtin_amdgcn_exp2f(fmaf(sacc[r], scale_log2, -lse2)) * (pacc[r] - dlt) * (SPLIT ? DS_SCALE : 1.0f);
        if (diag) {   // keys in the future of this lane's query contribute nothing
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (key0 + jb * 32 + acc_row(r, lane) > my_q) sacc[r] = 0.f;
        }
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          const e16x8 dsf = pack8(sacc, s2);
          e16x8 dsl = dsf;
          if constexpr (SPLIT) dsl = pack8_lo(sacc, s2, dsf, LO_SCALE);
#pragma unroll
          for (int db = 0; db < D / 32; ++db) {
            const e16x8 kt = lds_frag_tr<D>(Kt, jb * 32 + 16 * s2, db * 32, lane);
            acc[db] = ZS_ATTN_MFMA(kt, dsf, acc[db], 0, 0, 0);
            if constexpr (SPLIT) {
              f32x16& a = LO_ACC ? acclo[LO_ACC ? db : 0] : acc[db];
              a = ZS_ATTN_MFMA(kt, dsl, a, 0, 0, 0);
            }
          }
        }
      }
    }
    if (t + 1 < ntiles) {   // the other buffer was last read before the barrier that ended the previous iteration
      put_tile(kr, smem + ((t + 1) & 1) * 2 * TILE<D>, tid);
      put_tile(vr, smem + ((t + 1) & 1) * 2 * TILE<D> + TILE<D>, tid);
    }
    __syncthreads();
  }
  if constexpr (QS == 2) merge_halves<D>(acc, acclo, reinterpret_cast<f32x4*>(smem_raw), half, wave, lane);
  if constexpr (SPLIT && LO_ACC && QS == 1) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[db][r] = fmaf(acclo[db][r], LO_UNIT, acc[db][r]);
  }
  unsigned redo = 0;
  if constexpr (SPLIT) {
    RedoLds<NW>& rl = redo_lds<NW>(smem_raw);
    if (half == 0 && lane < 32) rl.delta[32 * wave + lane] = dlt;
    redo = rows_of(rl, wave, half == 0, my_q < S && lse2 == lse2 && dlt == dlt, mark_of(acc));
  }
  if (half == 0 && (LINES || my_q < S)) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[db][r] *= SPLIT ? scale / DS_SCALE : scale;
    if (rope) unrotate_row<D, D / 32>(acc, rope, min(my_q, S - 1), lane, dd);
    if constexpr (LINES) store_rows<D>(acc, 1.0f, rows_lds<NW, D, SPLIT>(smem_raw, wave), dq + tok0 * ldd + h * dd, ldd, wq0, S, lane, dd, redo);
    else store_direct<D, SPLIT>(acc, 1.0f, dq + tok0 * ldd + h * dd, ldd, my_q, S, lane, dd, redo);
  }
  if constexpr (SPLIT) {
    if (__builtin_expect(any_row(redo_lds<NW>(smem_raw).masks, QW, lane), 0))
      redo_dq_rows<NW>(smem_raw, QW, q0, dd, qh, kh, vh, ld, doh, ldo, lse + ((int64_t)b * nh + h) * S, scale, rope,
                       dq + tok0 * ldd + h * dd, ldd);
  }
}

template <int NW, int QS, int D, bool SPLIT, bool LINES>
__global__ __launch_bounds__(64 * NW, NW == 4 && !(SPLIT && LO_ACC && D > 64) ? 2 : 1) void attn_bwd_dq_kernel(int S, const e16* __restrict__ q, const e16* __restrict__ k,
                                                          const e16* __restrict__ v, int64_t ld,
                                                          const e16* __restrict__ o, const e16* __restrict__ dout,
                                                          int64_t ldo, const float* __restrict__ lse,
                                                          float* __restrict__ delta,
                                                          e16* __restrict__ dq, int64_t ldd, float scale, int nh,
                                                          int mb, const float2* __restrict__ rope, int head_dim) {
  dq_block<NW, QS, D, SPLIT, LINES>(blockIdx.x, S, q, k, v, ld, o, dout, ldo, lse, delta, dq, ldd, scale, nh, mb, rope, head_dim);
}

// ------------------------------------------------------------------------------------------ dK, dV
// grid ceil(S/(32 NW))*nh*mb, NW waves; wave w owns keys k0+32w..; loops over Q/dO tiles from the diagonal to the
// end.  With 8 waves the staged Q/dO tiles serve 256 keys and two waves share each SIMD, so one wave's
// softmax arithmetic overlaps the other's MFMAs.
// S[q][key] = Q K^T (lane = key, registers = queries), P = exp2(S c - lse_q), dP = dO V^T,
// dV^T[d][key] += dO^T[d][q] P[q][key],  dK^T[d][key] += Q^T[d][q] dS[q][key].
// QS = 2: two waves share 32 keys, each taking one half of every tile's queries; their sums meet in LDS at the end.
// The waves per SIMD are stated because the scheduler otherwise aims for more than the registers allow and issues LDS reads later
// (heads of 64 at S = 1000: 46 -> 48 us).
// BOTH: dQ and dK/dV in one launch, for grids that leave CUs idle when they run one after the other: the blocks from dkv_blocks on are
// dQ's.  No block reads what another one writes: delta of a tile's rows is formed here from dO and the same rows of O, 16 lanes to a
// row, instead of read.
template <int NW, int QS, int D, bool SPLIT, bool BOTH, bool LINES>
__global__ __attribute__((amdgpu_waves_per_eu(SPLIT && LO_ACC && D > 64 ? 1 : 2, 2))) __launch_bounds__(64 * NW) void attn_bwd_dkv_kernel(int S, const e16* __restrict__ q, const e16* __restrict__ k,
                                                           const e16* __restrict__ v, int64_t ld,
                                                           const e16* __restrict__ dout, int64_t ldo,
                                                           const float* __restrict__ lse, const float* __restrict__ delta,
                                                           e16* __restrict__ dk, e16* __restrict__ dv, int64_t ldd,
                                                           float scale, int nh, int mb, const float2* __restrict__ rope, int head_dim,
                                                           int dkv_blocks, const e16* __restrict__ o, float* __restrict__ delta_out, e16* __restrict__ dq) {
  static_assert(!BOTH || (!SPLIT && 64 * NW % (D / 8) == 0 && D == 128), "16 lanes share a row; rows that are redone read delta");
  if (BOTH && (int)blockIdx.x >= dkv_blocks) {
    dq_block<NW, QS, D, SPLIT, LINES>(blockIdx.x - dkv_blocks, S, q, k, v, ld, o, dout, ldo, lse, delta_out, dq, ldd, scale, nh, mb, rope, head_dim);
    return;
  }
  const int dd = SPLIT ? head_dim : D;
  extern __shared__ __align__(16) char smem_raw[];
  e16* smem = reinterpret_cast<e16*>(smem_raw);                 // [2][Q tile | dO tile]
  float* stats = reinterpret_cast<float*>(smem + 4 * TILE<D>);       // [2][lse2[64] | delta[64]]
  constexpr int KWV = NW / QS;   // groups of 32 keys
  const int tid = threadIdx.x, lane = tid & 63, wave = QS == 1 ? tid >> 6 : (tid >> 6) % KWV, half = QS == 1 ? 0 : (tid >> 6) / KWV;
  const BlockId bid = block_id(blockIdx.x, nh, mb);
  const int kb = bid.rank, h = bid.h, b = bid.b;                   // early key blocks (most work) first
  const int64_t tok0 = (int64_t)b * S;
  const e16* qh = q + tok0 * ld + h * dd;
  const e16* kh = k + tok0 * ld + h * dd;
  const e16* vh = v + tok0 * ld + h * dd;
  const e16* doh = dout + tok0 * ldo + h * dd;
  const __amdgpu_buffer_rsrc_t rsq = head_rsrc(qh, ld, S, dd), rsdo = head_rsrc(doh, ldo, S, dd);
  const float* lse_h = lse + ((int64_t)b * nh + h) * S;
  const float* dlt_h = BOTH ? nullptr : delta + ((int64_t)b * nh + h) * S;
  const __amdgpu_buffer_rsrc_t rso = head_rsrc(BOTH ? o + tok0 * ldo + h * dd : doh, ldo, S, dd);
  const int k0 = kb * 32 * KWV, wk0 = k0 + wave * 32;
  const int my_k = wk0 + (lane & 31);
  const float scale_log2 = scale * LOG2E;

  // K fragments stay in registers; the wave's 32 rows of V go to a private LDS block instead and are
  // read back as B operands (same fragment pattern as the A operands), which keeps the kernel within
  // the register budget of two waves per SIMD.
  // Everything the kernel reads before its loop (the first tile, K, V) is in flight before the first wait: a small LLaMA step
  // (S = 256, 16 launches) is 18 us shorter for it, 4 x 16 heads of 64 at S = 1000 98 -> 97 us.
  TileRegs<64 * NW, D> qr, dor, orow;   // orow: of O
  float statr = 0.f;
  bool stat_in = false;
  // The scaling of lse and the zeros past S wait for put(): either would make the wave wait here, for the tile's loads too.
  auto fetch = [&](int t) {
    fetch_tile(qr, rsq, (int)ld, t * TR, tid, dd);
    fetch_tile(dor, rsdo, (int)ldo, t * TR, tid, dd);
    if constexpr (BOTH) fetch_tile(orow, rso, (int)ldo, t * TR, tid, dd);
    if (tid < (BOTH ? 64 : 128)) {
      const int r = t * TR + (tid & 63);
      stat_in = r < S;
      statr = (BOTH || tid < 64 ? lse_h : dlt_h)[min(r, S - 1)];
    }
  };
  auto put = [&](int buf) {
    put_tile(qr, smem + buf * 2 * TILE<D>, tid);
    put_tile(dor, smem + buf * 2 * TILE<D> + TILE<D>, tid);
    if (tid < (BOTH ? 64 : 128)) stats[buf * 128 + tid] = stat_in ? statr * (tid < 64 ? LOG2E : 1.0f) : 0.f;
    if constexpr (BOTH) {   // rows past S are zeros
#pragma unroll
      for (int i = 0; i < 8 * D / (64 * NW); ++i) {
        float x = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) x = fmaf((float)dor.v[i][e], (float)orow.v[i][e], x);
#pragma unroll
        for (int m = 1; m < D / 8; m *= 2) x += __shfl_xor(x, m, 64);
        if (tid % (D / 8) == 0) stats[buf * 128 + 64 + tid / (D / 8) + 64 * NW / (D / 8) * i] = x;
      }
    }
  };
  const int t_begin = k0 / TR, t_end = (S - 1) / TR + 1;
  fetch(t_begin);
  e16x8 kf[D / 16];
  if constexpr (LINES) load_lines<D>(kf, kh, ld, wk0, S, lane, dd);
  else load_row_frags<D>(kf, kh, ld, wk0, S, lane, dd);
  if (QS == 1 || half == 0) {   // QS = 2: the first of the two waves brings the rows, the barrier before the loop publishes them
    e16* Vw = reinterpret_cast<e16*>(stats + 256) + wave * 32 * LDT<D>;
    const __amdgpu_buffer_rsrc_t rsv = head_rsrc(vh, ld, S, dd);   // rows past S read as zero
    union { u32x4 u; e16x8 h; } w[D / 16];
#pragma unroll
    for (int i = 0; i < D / 16; ++i) {
      const int vv = lane + 64 * i, r = vv / (D / 8), c = (vv % (D / 8)) * 8;
      w[i].u = __builtin_amdgcn_raw_buffer_load_b128(rsv, c < dd ? (int)(((unsigned)(wk0 + r) * (unsigned)ld + c) * 2u) : (int)0x80000000, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < D / 16; ++i) {
      const int vv = lane + 64 * i, r = vv / (D / 8), c = (vv % (D / 8)) * 8;
      *reinterpret_cast<e16x8*>(Vw + r * LDT<D> + c) = w[i].h;
    }
  }
  const e16* Vw = reinterpret_cast<e16*>(stats + 256) + wave * 32 * LDT<D>;
  f32x16 dkacc[D / 32], dvacc[D / 32], dklo[SPLIT && LO_ACC ? D / 32 : 1], dvlo[SPLIT && LO_ACC ? D / 32 : 1];
#pragma unroll
  for (int i = 0; i < D / 32; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      dkacc[i][r] = dvacc[i][r] = 0.f;
      if (SPLIT && LO_ACC) dklo[SPLIT && LO_ACC ? i : 0][r] = dvlo[SPLIT && LO_ACC ? i : 0][r] = 0.f;
    }

  if constexpr (LINES) {
    to_frags<D>(kf, smem + (tid >> 6) * 32 * LDT<D>, lane);
    __syncthreads();
  }
  put(0);
  __syncthreads();
  for (int t = t_begin; t < t_end; ++t) {
    const int buf = (t - t_begin) & 1;
    const e16* Qt = smem + buf * 2 * TILE<D>;
    const e16* dOt = Qt + TILE<D>;
    const float* st = stats + buf * 128;
    if (t + 1 < t_end) fetch(t + 1);
    const int qrow0 = t * TR;
    if (qrow0 + (QS == 2 ? 32 * half + 31 : TR - 1) >= wk0) {   // otherwise every query of the tile precedes this wave's keys
      const bool diag = qrow0 < wk0 + 31;
#pragma unroll
      for (int i = 0; i < 2 / QS; ++i) {
        const int ib = QS == 2 ? half : i;
        f32x16 sacc, pacc;
#pragma unroll
        for (int r = 0; r < 16; ++r) sacc[r] = pacc[r] = 0.f;
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
          sacc = ZS_ATTN_MFMA(lds_frag<D>(Qt, ib * 32, 16 * s, lane), kf[s], sacc, 0, 0, 0);
          pacc = ZS_ATTN_MFMA(lds_frag<D>(dOt, ib * 32, 16 * s, lane), lds_frag<D>(Vw, 0, 16 * s, lane), pacc,
                                                         0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int qi = ib * 32 + acc_row(r, lane);
          const float p = __builtin_amdgcn_exp2f(fmaf(sacc[r], scale_log2, -st[qi]));
          sacc[r] = p;
          pacc[r] = p * (pacc[r] - st[64 + qi]) * (SPLIT ? DS_SCALE : 1.0f);
        }
        if (diag || qrow0 + TR > S) {   // queries before this lane's key, and rows past the end, contribute nothing
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int qi = ib * 32 + acc_row(r, lane);
            if (qrow0 + qi < my_k || qrow0 + qi >= S) sacc[r] = pacc[r] = 0.f;
          }
        }
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          const e16x8 pf = pack8(sacc, s2), dsf = pack8(pacc, s2);
          e16x8 pl = pf, dsl = dsf;
          if constexpr (SPLIT) { pl = pack8_lo(sacc, s2, pf, LO_SCALE); dsl = pack8_lo(pacc, s2, dsf, LO_SCALE); }
#pragma unroll
          for (int db = 0; db < D / 32; ++db) {
            const e16x8 dot = lds_frag_tr<D>(dOt, ib * 32 + 16 * s2, db * 32, lane);
            dvacc[db] = ZS_ATTN_MFMA(dot, pf, dvacc[db], 0, 0, 0);
            if constexpr (SPLIT) {
              f32x16& a = LO_ACC ? dvlo[LO_ACC ? db : 0] : dvacc[db];
              a = ZS_ATTN_MFMA(dot, pl, a, 0, 0, 0);
            }
            const e16x8 qt = lds_frag_tr<D>(Qt, ib * 32 + 16 * s2, db * 32, lane);
            dkacc[db] = ZS_ATTN_MFMA(qt, dsf, dkacc[db], 0, 0, 0);
            if constexpr (SPLIT) {
              f32x16& a = LO_ACC ? dklo[LO_ACC ? db : 0] : dkacc[db];
              a = ZS_ATTN_MFMA(qt, dsl, a, 0, 0, 0);
            }
          }
        }
      }
    }
    if (t + 1 < t_end) put(buf ^ 1);
    __syncthreads();
  }
  if constexpr (QS == 2) {
    merge_halves<D>(dvacc, dvlo, reinterpret_cast<f32x4*>(smem_raw), half, wave, lane);
    merge_halves<D>(dkacc, dklo, reinterpret_cast<f32x4*>(smem_raw), half, wave, lane);
  }
  if constexpr (SPLIT && LO_ACC && QS == 1) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        dkacc[db][r] = fmaf(dklo[db][r], LO_UNIT, dkacc[db][r]);
        dvacc[db][r] = fp32_value(fmaf(dvlo[db][r], LO_UNIT, dvacc[db][r]));   // stored as it is
      }
  }
  unsigned redo = 0;
  if constexpr (SPLIT) redo = rows_of(redo_lds<NW>(smem_raw), wave, half == 0, my_k < S, mark_of(dkacc) + mark_of(dvacc));
  if (half == 0 && (LINES || my_k < S)) {
    e16* to_k = dk + tok0 * ldd + h * dd;
    e16* to_v = dv + tok0 * ldd + h * dd;
    if constexpr (LINES) store_rows<D>(dvacc, 1.0f, rows_lds<NW, D, SPLIT>(smem_raw, wave), to_v, ldd, wk0, S, lane, dd, redo);
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) dkacc[db][r] *= SPLIT ? scale / DS_SCALE : scale;
    if (rope) unrotate_row<D, SPLIT ? 1 : 2>(dkacc, rope, min(my_k, S - 1), lane, dd);   // the registers that dV leaves: no spills
    if constexpr (LINES) store_rows<D>(dkacc, 1.0f, rows_lds<NW, D, SPLIT>(smem_raw, wave), to_k, ldd, wk0, S, lane, dd, redo);
    else {
      store_direct<D, SPLIT>(dkacc, 1.0f, to_k, ldd, my_k, S, lane, dd, redo);
      store_direct<D, SPLIT>(dvacc, 1.0f, to_v, ldd, my_k, S, lane, dd, redo);
    }
  }
  if constexpr (SPLIT) {
    if (__builtin_expect(any_row(redo_lds<NW>(smem_raw).masks, KWV, lane), 0))
      redo_dkv_rows<NW>(smem_raw, KWV, k0, S, dd, qh, kh, vh, ld, doh, ldo, lse_h, dlt_h, scale, rope,
                        dk + tok0 * ldd + h * dd, dv + tok0 * ldd + h * dd, ldd);
  }
}

template <int D> constexpr size_t SMEM_FWD = 4 * TILE<D> * sizeof(e16);                    // 77824 for D = 128
template <int D> constexpr size_t smem_dkv(int nw) {
  return 4 * TILE<D> * sizeof(e16) + 256 * sizeof(float) + (size_t)nw * 32 * LDT<D> * sizeof(e16);
}

// Blocks of 256 rows (8 waves) instead of 128 (4 waves): for the key blocks of the dK/dV kernel whenever that still
// gives every CU a workgroup; for the query blocks of the forward and dQ kernels only from S = 4096 on (measured: 7 % and
// 3 % faster at S = 4096 with 32 heads, 7 % slower at S = 2048 with 80 head-sequences, where a block has half the tiles to
// amortise its idle waves on the diagonal).
inline bool wide_blocks(int S, int nh, int mb) { return cdiv(S, 256) * nh * mb >= 256; }
inline bool wide_query_blocks(int S, int nh, int mb) { return wide_blocks(S, nh, mb) && S >= 4096; }

// Whether the row blocks and results of a kernel pass through LDS as whole lines (D: padded head dim).  With one or two of a block's
// four waves at work the way round costs more than it saves, and in the forward of narrow heads, with its shorter rows, at any
// length.  us, lines : direct, 2 x 16 heads, forward of 128 columns S = 32 5.2 : 4.6, 64 5.4 : 5.2, 100 7.2 : 7.6; of 64 S = 64 5.1 : 4.7, 1000
// 25.3 : 24.8, of 96 200 10.4 : 9.9; backward of 128 columns S = 32 9.6 : 8.8, 64 9.6 : 10.2; of 96 S = 64 15.9 : 14.7, 128 20.2 : 22.4.  dQ of
// a padded 64 or 96 columns wants all four waves or two blocks (S = 192 loses 3 to 7 %, 128 gains as much), of a padded 128 the form
// in which two waves share rows, which lengths over 256 have; half heads over 64, one wave per SIMD, neither gain nor lose but at S = 128.  dK/dV of 64 columns, long: S = 4096, 4 heads 101.9 : 98.2.
template <int D, bool SPLIT> bool lines_fwd(int S) { return D == 128 && (SPLIT ? S >= 256 : S > 64); }
template <int D, bool SPLIT> bool lines_dq(int S) { return SPLIT ? D < 128 && (S >= 256 || (S > 96 && S <= 128)) : S > 64; }
template <int D, bool SPLIT> bool lines_dkv(int S) { return SPLIT ? S > 64 && (D > 64 || S <= 1024) : S > 32; }

template <typename K> hipError_t set_smem(K kern, size_t bytes, bool& done) {
  if (done) return hipSuccess;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess) done = true;
  return e;
}

// One launch of each kernel with NW waves; `set` remembers that its LDS size has been allowed.
template <int NW, int D, bool SPLIT, bool LINES>
hipError_t launch_fwd(hipStream_t st, int mb, int S, int nh, int d, const void* q, const void* k, const void* v, int64_t ld, void* o,
                      int64_t ldo, float* lse) {
  static bool set = false;
  const hipError_t e = set_smem(attn_fwd_kernel<NW, D, SPLIT, LINES>, SMEM_FWD<D>, set);
  if (e != hipSuccess) return e;
  // SPLIT adds scale_lo * score: above zero, so that a masked score stays -inf
  float hi = LOG2E / sqrtf((float)d), lo = 0.f;
  if (SPLIT) {
    const double c = 1.4426950408889634 / sqrt((double)d);
    if ((double)hi >= c) hi = nextafterf(hi, 0.f);
    lo = (float)(c - (double)hi);
  }
  hipLaunchKernelGGL((attn_fwd_kernel<NW, D, SPLIT, LINES>), dim3((unsigned)(cdiv(S, 32 * NW) * nh * mb)), dim3(64 * NW), SMEM_FWD<D>, st, S,
                     (const e16*)q, (const e16*)k, (const e16*)v, ld, (e16*)o, ldo, lse, hi, lo, nh, mb, d);
  return hipGetLastError();
}
template <int NW, int QS, int D, bool SPLIT, bool LINES>
hipError_t launch_dq(hipStream_t st, int mb, int S, int nh, int d, const void* q, const void* k, const void* v, int64_t ld, const void* o,
                     const void* dout, int64_t ldo, const float* lse, float* delta, void* dq, int64_t ldd, const float2* rope) {
  static bool set = false;
  const hipError_t e = set_smem(attn_bwd_dq_kernel<NW, QS, D, SPLIT, LINES>, SMEM_FWD<D>, set);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((attn_bwd_dq_kernel<NW, QS, D, SPLIT, LINES>), dim3((unsigned)(cdiv(S, 32 * (NW / QS)) * nh * mb)), dim3(64 * NW), SMEM_FWD<D>, st,
                     S, (const e16*)q, (const e16*)k, (const e16*)v, ld, (const e16*)o, (const e16*)dout, ldo, lse, delta, (e16*)dq,
                     ldd, 1.0f / sqrtf((float)d), nh, mb, rope, d);
  return hipGetLastError();
}
template <int NW, int QS, int D, bool SPLIT, bool LINES>
hipError_t launch_dkv(hipStream_t st, int mb, int S, int nh, int d, const void* q, const void* k, const void* v, int64_t ld,
                      const void* dout, int64_t ldo, const float* lse, const float* delta, void* dk, void* dv, int64_t ldd,
                      const float2* rope) {
  static bool set = false;
  const hipError_t e = set_smem(attn_bwd_dkv_kernel<NW, QS, D, SPLIT, false, LINES>, smem_dkv<D>(NW / QS), set);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((attn_bwd_dkv_kernel<NW, QS, D, SPLIT, false, LINES>), dim3((unsigned)(cdiv(S, 32 * (NW / QS)) * nh * mb)), dim3(64 * NW), smem_dkv<D>(NW / QS),
                     st, S, (const e16*)q, (const e16*)k, (const e16*)v, ld, (const e16*)dout, ldo, lse, delta, (e16*)dk, (e16*)dv,
                     ldd, 1.0f / sqrtf((float)d), nh, mb, rope, d, 0, nullptr, nullptr, nullptr);
  return hipGetLastError();
}
// dQ and dK/dV together, 8 waves to a block of 128 rows, two of them per 32 rows.
template <int D, bool LINES>
hipError_t launch_bwd(hipStream_t st, int mb, int S, int nh, const void* q, const void* k, const void* v, int64_t ld, const void* o, const void* dout,
                      int64_t ldo, const float* lse, float* delta, void* dq, void* dk, void* dv, int64_t ldd, const float2* rope) {
  constexpr size_t SMEM = smem_dkv<D>(4) > SMEM_FWD<D> ? smem_dkv<D>(4) : SMEM_FWD<D>;
  static bool set = false;
  const hipError_t e = set_smem(attn_bwd_dkv_kernel<8, 2, D, false, true, LINES>, SMEM, set);
  if (e != hipSuccess) return e;
  const int blocks = (int)(cdiv(S, 128) * nh * mb);
  hipLaunchKernelGGL((attn_bwd_dkv_kernel<8, 2, D, false, true, LINES>), dim3((unsigned)(2 * blocks)), dim3(512), SMEM, st, S, (const e16*)q, (const e16*)k,
                     (const e16*)v, ld, (const e16*)dout, ldo, lse, nullptr, (e16*)dk, (e16*)dv, ldd, 1.0f / sqrtf((float)D), nh, mb, rope, D,
                     blocks, (const e16*)o, delta, (e16*)dq);
  return hipGetLastError();
}
// Blocks of 128 rows: with 8 waves, two of them per 32 rows, or with 4.  The kernels' LDS leaves a CU one workgroup (dK/dV) or
// two (dQ), so the 4-wave forms keep 4 waves of a CU at work, or 8 where dQ has two workgroups for it.  Sharing rows costs a
// merge at the end (16 KB per pair and accumulator through LDS), which a row block with four tiles does not win back in dQ.
// 16 heads of 128, S = 2048: dK/dV 112 : 77 us, dQ 72 : 57 us (4 : 8 waves); 8 heads, S = 1000: both 92 : 67 us; 4 heads,
// S = 256: dK/dV 24 : 20 us, dQ 17.9 : 18.8 us.  dQ shares rows while every CU has one block; a second round of 8-wave
// workgroups costs more than the two 4-wave ones that a CU holds side by side, unless the sequences are so long that the blocks
// differ a lot in their work.  Both directions, S = 513, 98 heads (490 blocks) 83 us shared, 75 not; S = 1700, 24 heads (336 blocks)
// 104 and 117.  Of 116 shapes with 216 to 550 blocks the rule takes the faster form but for 1.6 %.
// Where 2 x blocks leave CUs idle, or nearly, dQ and dK/dV share a launch and the time is that of dK/dV, whose blocks then form delta
// themselves, with additions in another order than dQ's: fp32 sums that may differ in their last place, and 16-bit gradients that now
// and then round the other way.  Separate : together, us: 4 heads, S = 256 31.4 : 20.0; 32 heads, S = 512 45.5 : 32.9; 16 heads, S = 2048 (256 blocks) 115 :
// 100.  Up to 256 blocks the long sequences' unequal blocks fill one another's gaps; 288 blocks are a tie at S = 2048, 480 lose 22 %.
// Sequences of one or two blocks have equal ones, and a second round costs what it saves: S = 128, 160 blocks 27.7 : 28.2, 240 30.4 : 33.8;
// S = 200, 192 blocks 32.2 : 26.5, 200 33.6 : 35.9; S = 300, 252 blocks 38.3 : 39.5.
template <int D, bool SPLIT>
hipError_t bwd_128(hipStream_t st, int mb, int S, int nh, int d, const void* q, const void* k, const void* v, int64_t ld, const void* o,
                   const void* dout, int64_t ldo, const float* lse, float* delta, void* dq, void* dk, void* dv, int64_t ldd,
                   const float2* rope, bool wide_dkv) {
  if constexpr (SPLIT && LO_ACC && D > 64) {   // the low accumulators of wide half heads leave no registers for 8 waves
    const hipError_t e = launch_dq<4, 1, D, SPLIT, false>(st, mb, S, nh, d, q, k, v, ld, o, dout, ldo, lse, delta, dq, ldd, rope);
    if (e != hipSuccess) return e;
    return lines_dkv<D, SPLIT>(S) ? launch_dkv<4, 1, D, SPLIT, true>(st, mb, S, nh, d, q, k, v, ld, dout, ldo, lse, delta, dk, dv, ldd, rope)
                                  : launch_dkv<4, 1, D, SPLIT, false>(st, mb, S, nh, d, q, k, v, ld, dout, ldo, lse, delta, dk, dv, ldd, rope);
  } else {
    const int64_t per_head = cdiv(S, 128), blocks = per_head * nh * mb;
    if constexpr (!SPLIT && D == 128)
      if (!wide_dkv && blocks <= (per_head == 1 ? 128 : per_head < 4 ? 192 : 256) &&
          attn_bwd_apart((int64_t)mb * S, 2ll * nh * d, k, v, 2 * ld, o, 2 * ldo, dq, dk, dv, 2 * ldd))
        return lines_dkv<D, SPLIT>(S) ? launch_bwd<D, true>(st, mb, S, nh, q, k, v, ld, o, dout, ldo, lse, delta, dq, dk, dv, ldd, rope)
                                      : launch_bwd<D, false>(st, mb, S, nh, q, k, v, ld, o, dout, ldo, lse, delta, dq, dk, dv, ldd, rope);
    const hipError_t e = S > 256 && blocks < 512 && blocks <= 256 + 28 * (per_head > 6 ? per_head - 6 : 0)
                             ? launch_dq<8, 2, D, SPLIT, true>(st, mb, S, nh, d, q, k, v, ld, o, dout, ldo, lse, delta, dq, ldd, rope)
                         : lines_dq<D, SPLIT>(S) ? launch_dq<4, 1, D, SPLIT, !(SPLIT && D == 128)>(st, mb, S, nh, d, q, k, v, ld, o, dout, ldo, lse, delta, dq, ldd, rope)
                                                 : launch_dq<4, 1, D, SPLIT, false>(st, mb, S, nh, d, q, k, v, ld, o, dout, ldo, lse, delta, dq, ldd, rope);
    if (e != hipSuccess || wide_dkv) return e;
    return lines_dkv<D, SPLIT>(S) ? launch_dkv<8, 2, D, SPLIT, true>(st, mb, S, nh, d, q, k, v, ld, dout, ldo, lse, delta, dk, dv, ldd, rope)
                                  : launch_dkv<8, 2, D, SPLIT, false>(st, mb, S, nh, d, q, k, v, ld, dout, ldo, lse, delta, dk, dv, ldd, rope);
  }
}

}  // namespace

#ifdef ZS_ATTN_SPLIT
hipError_t ZS_ATTN_NAME(attn_fwd_split)(hipStream_t st, int mb, int S, int nh, int d, const void* q, const void* k, const void* v,
                         int64_t ld, void* o, int64_t ldo, float* lse) {
  if (d >= 128 || (int64_t)S * ld * 2 >= (1ll << 31)) return hipErrorInvalidValue;      // 32-bit buffer offsets
  if (d <= 64) return launch_fwd<4, 64, true, false>(st, mb, S, nh, d, q, k, v, ld, o, ldo, lse);
  if (d <= 96) return launch_fwd<4, 96, true, false>(st, mb, S, nh, d, q, k, v, ld, o, ldo, lse);
  return lines_fwd<128, true>(S) ? launch_fwd<4, 128, true, true>(st, mb, S, nh, d, q, k, v, ld, o, ldo, lse) : launch_fwd<4, 128, true, false>(st, mb, S, nh, d, q, k, v, ld, o, ldo, lse);
}

hipError_t ZS_ATTN_NAME(attn_bwd_split)(hipStream_t st, int mb, int S, int nh, int d, const void* q, const void* k, const void* v,
                         int64_t ld, const void* o, const void* dout, int64_t ldo, const float* lse, float* delta,
                         void* dq, void* dk, void* dv, int64_t ldd, const float2* rope) {
  if (d >= 128 || (int64_t)S * (ld > ldo ? ld : ldo) * 2 >= (1ll << 31)) return hipErrorInvalidValue;   // 32-bit buffer offsets
  if (d <= 64) return bwd_128<64, true>(st, mb, S, nh, d, q, k, v, ld, o, dout, ldo, lse, delta, dq, dk, dv, ldd, rope, false);
  if (d <= 96) return bwd_128<96, true>(st, mb, S, nh, d, q, k, v, ld, o, dout, ldo, lse, delta, dq, dk, dv, ldd, rope, false);
  return bwd_128<128, true>(st, mb, S, nh, d, q, k, v, ld, o, dout, ldo, lse, delta, dq, dk, dv, ldd, rope, false);
}
#else
#ifndef ZS_ATTN_F16
bool attn_mfma_supported(DType dt, int S, int d) { return (dt == BF16 || dt == F16) && d == 128 && S >= 1; }
#endif

hipError_t ZS_ATTN_NAME(attn_fwd_mfma)(hipStream_t st, int mb, int S, int nh, int d, const void* q, const void* k, const void* v,
                         int64_t ld, void* o, int64_t ldo, float* lse) {
  if ((int64_t)S * ld * 2 >= (1ll << 31)) return hipErrorInvalidValue;      // 32-bit buffer offsets
  // 256 queries per workgroup when that still gives every CU a workgroup, else 128
  return wide_query_blocks(S, nh, mb) ? launch_fwd<8, 128, false, true>(st, mb, S, nh, d, q, k, v, ld, o, ldo, lse)
         : lines_fwd<128, false>(S)   ? launch_fwd<4, 128, false, true>(st, mb, S, nh, d, q, k, v, ld, o, ldo, lse)
                                      : launch_fwd<4, 128, false, false>(st, mb, S, nh, d, q, k, v, ld, o, ldo, lse);
}

hipError_t ZS_ATTN_NAME(attn_bwd_mfma)(hipStream_t st, int mb, int S, int nh, int d, const void* q, const void* k, const void* v,
                         int64_t ld, const void* o, const void* dout, int64_t ldo, const float* lse, float* delta,
                         void* dq, void* dk, void* dv, int64_t ldd, const float2* rope) {
  if ((int64_t)S * (ld > ldo ? ld : ldo) * 2 >= (1ll << 31)) return hipErrorInvalidValue;   // 32-bit buffer offsets
  const bool wide = wide_blocks(S, nh, mb);
  const hipError_t e =
      wide_query_blocks(S, nh, mb) ? launch_dq<8, 1, 128, false, true>(st, mb, S, nh, d, q, k, v, ld, o, dout, ldo, lse, delta, dq, ldd, rope)
                                   : bwd_128<128, false>(st, mb, S, nh, d, q, k, v, ld, o, dout, ldo, lse, delta, dq, dk, dv, ldd, rope, wide);
  if (e != hipSuccess || !wide) return e;
  return lines_dkv<128, false>(S) ? launch_dkv<8, 1, 128, false, true>(st, mb, S, nh, d, q, k, v, ld, dout, ldo, lse, delta, dk, dv, ldd, rope)
                                  : launch_dkv<8, 1, 128, false, false>(st, mb, S, nh, d, q, k, v, ld, dout, ldo, lse, delta, dk, dv, ldd, rope);
}
#endif

}  // namespace zs

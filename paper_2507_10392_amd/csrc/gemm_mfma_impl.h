// 16-bit (bf16 or IEEE half) GEMM on the CDNA4 matrix cores (v_mfma_f32_16x16x32_bf16 / _f16), fp32 accumulation: the tile kernel,
// templated on the workgroup tile BM x BN and the number of wavefronts.
//
// One workgroup of 4 (2 x 2) or 8 (2 x 4 or 4 x 2) wavefronts computes a BM x BN tile of C; each wavefront owns
// its part as MFMA blocks of 16x16 (4 accumulator registers per block and lane).
// The K loop walks 64-wide slabs.  A slab of each operand is fetched from HBM with 16-byte buffer
// loads into registers one or two iterations ahead and stored into one of two LDS buffers:
//   * contraction index contiguous in memory  -> LDS [row][k], 128-byte rows whose 16-byte pieces are
//     permuted by the row index (piece p of row r at position p ^ r%8); an MFMA operand fragment
//     (8 consecutive k of one row) is one ds_read_b128;
//   * row index contiguous in memory (B of y = x W with W stored [in,out]; both operands of
//     dW = x^T dy) -> LDS [k][row], k-lines padded by 32 elements, pairs of 16-row chunks swapped on
//     the odd eights of k; the fragment is two ds_read_b64_tr_b16, the LDS transpose read of gfx950,
//     each returning 4 consecutive k.
// Permutation and padding keep slab stores and fragment reads free of bank conflicts (measured per
// access pattern: the LDS does not serve a wave's 16-byte accesses in groups of 16 consecutive lanes).
// Workgroup ids are remapped so that the 8 XCDs (ids are dealt round-robin to them) each work
// on a compact patch of C and re-use their own L2's A rows and B columns.
// The 256x256 tile runs 8 wavefronts (128 accumulator registers each, two waves per SIMD); the 128x128 tile
// runs 4 and needs 64 accumulator registers and 74 KB of LDS, so two workgroups share a CU.  Either way a
// SIMD has a second wave to issue MFMAs while the first waits for memory, LDS or a barrier.  The 256x192 and 256x128
// tiles (8 waves of 64 x 96 and 64 x 64) are for grids that fill the chip better with them.
//
// What bounds the smaller tiles is the rate at which a CU gets lines that its L1 does not hold: with the MFMAs taken out of the
// 256x128 kernel, 2048 x 4096, K = 8192, takes 104 of 122 us, with the loads taken out instead 86, and loading three
// slabs ahead instead of two changes nothing.  Lines that are not cold come faster (512 x 4096, K = 12288 on 128x128 tiles 85 us
// with operands in the memory-side cache, 129 us without).  So a bigger tile, which needs fewer lines per flop, beats a smaller
// one wherever the grid still fills the CUs, and rows that are no multiple of 128 bytes apart cost up to half as much again.
#pragma once
#include "kernels.h"

namespace zs {
namespace gemm_impl {

constexpr int BK = 64;
constexpr int LDK = BK;                           // [row][k] layout: 128-byte rows, no padding; the 16-byte piece p of row r sits at
                                                  // position p ^ (r % 8), which keeps both the slab stores (8 rows x 8 pieces per wave)
                                                  // and the fragment reads (16 rows x 4 pieces per wave) free of bank conflicts
// [k][row] slabs: k-lines are padded by RPAD elements.  A transpose read serves 32 lanes per cycle, which
// touch 8 k-lines x 32 bytes; k-lines are 16 banks apart (mod 64) and the chunk swap of store_rmajor moves
// the second four lines by 8 banks, so those are 64 different banks.
constexpr int RPAD = 32;
constexpr int slab_elems(int R) { return R * LDK > BK * (R + RPAD) ? R * LDK : BK * (R + RPAD); }

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

template <int R, int NT> struct Frag { u32x4 v[R * 8 / NT]; };   // one thread's share of an R x 64 slab, 16 bytes each

// Operands are read through raw buffer descriptors: the per-lane offset is one VGPR, the per-load
// offset a scalar, and anything at or beyond num_records reads as zero, which handles the ragged edge
// along each operand's OUTER dimension for free.  Along the inner (contiguous) dimension the pieces past
// the edge get a per-lane offset that is out of range (DEAD, below).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}
// A per-lane byte offset of DEAD lies beyond every num_records (operand extents are below 2^30 bytes), so a
// lane whose piece must read as zero is simply sent there: no masks or branches in the K loop.
constexpr int DEAD = 0x40000000;

// Operand stored [rows, K] (k contiguous), ld = row stride.  With NT threads, thread t carries vectors
// v = t + NT*i: row = v/8, k-vector = v%8 (= t%8 for every i).  voff = ((t/8)*ld + (t%8)*8)*2 bytes (+ segment shift).
// Rows past the operand's last row lie beyond num_records; k-vectors at or past K (ragged last slab, and
// slabs past the end) would run into the next row and are sent out of range.
template <int R, int NT>
__device__ __forceinline__ void load_kmajor(Frag<R, NT>& f, __amdgpu_buffer_rsrc_t rs, int voff, int ld, int row0, int k0,
                                            int K, int tid, int i0 = 0, int i1 = R * 8 / NT) {
  const int vo = k0 + (tid & 7) * 8 >= K ? DEAD : voff;
#pragma unroll
  for (int i = 0; i < R * 8 / NT; ++i)
    if (i >= i0 && i < i1) f.v[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, vo, ((row0 + (NT / 8) * i) * ld + k0) * 2, 0);
}
// (load_kmajor, like the other three, handles vectors [i0, i1) of the thread's share)
template <int R, int NT>
__device__ __forceinline__ void store_kmajor(const Frag<R, NT>& f, bf16* lds, int tid, int i0 = 0, int i1 = R * 8 / NT) {
  static_assert((NT / 8) % 8 == 0, "a thread's row keeps its value mod 8 over the passes");
  bf16* p = lds + (tid >> 3) * LDK + (((tid & 7) ^ ((tid >> 3) & 7)) * 8);
#pragma unroll
  for (int i = 0; i < R * 8 / NT; ++i)
    if (i >= i0 && i < i1) *reinterpret_cast<u32x4*>(p + (NT / 8) * i * LDK) = f.v[i];
}

// Operand stored [K, rows] (row index contiguous).  A k-line of the slab is R/8 vectors; thread t carries
// vectors v = t + NT*i: k = v/(R/8), row-vector = v%(R/8).  Where R/8 divides NT that row-vector is the same for every i and one
// offset serves all; else (R = 192) each pass has its own.
// Row-vectors at or past the operand's last row (ragged edge tile) would read the next k-line: out of range.
template <int R, int NT> struct Lines {
  static constexpr int PER = R / 8, N = NT % PER == 0 ? 1 : R * 8 / NT, KSTEP = NT / PER;   // KSTEP: k-lines of a pass (N = 1)
  static_assert(N > 1 || KSTEP % 16 == 0, "bit 3 of a thread's k-line must not depend on the pass");
};
template <int R, int NT> struct LineOffsets { int v[Lines<R, NT>::N]; };
// two: the tile's first R/2 rows come from one matrix (rows row0 .. of `nrows`) and its last R/2 rows are the same rows of a second
// matrix lying `second` elements behind the first: gate and up projections side by side.
template <int R, int NT, bool two>
__device__ __forceinline__ LineOffsets<R, NT> voff_rmajor(int ld, int tid, int row0, int nrows, int second) {
  constexpr int PER = R / 8, HALF = two ? PER / 2 : PER;
  LineOffsets<R, NT> o;
#pragma unroll
  for (int i = 0; i < Lines<R, NT>::N; ++i) {
    const int v = tid + NT * i, j = v % PER, jj = j % HALF;
    o.v[i] = row0 + jj * 8 >= nrows ? DEAD : ((v / PER) * ld + jj * 8 + (j >= HALF ? second : 0)) * 2;
  }
  return o;
}
template <int R, int NT>
__device__ __forceinline__ void load_rmajor(Frag<R, NT>& f, __amdgpu_buffer_rsrc_t rs, const LineOffsets<R, NT>& voff, int ld, int row0, int k0,
                                            int i0 = 0, int i1 = R * 8 / NT) {
  typedef Lines<R, NT> L;
#pragma unroll
  for (int i = 0; i < R * 8 / NT; ++i)
    if (i >= i0 && i < i1)
      f.v[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, voff.v[L::N == 1 ? 0 : i], ((k0 + (L::N == 1 ? L::KSTEP * i : 0)) * ld + row0) * 2, 0);
}
template <int R, int NT>
__device__ __forceinline__ void store_rmajor(const Frag<R, NT>& f, bf16* lds, int tid, int i0 = 0, int i1 = R * 8 / NT) {
  typedef Lines<R, NT> L;
  constexpr int LDR = R + RPAD;
#pragma unroll
  for (int i = 0; i < R * 8 / NT; ++i)
    if (i >= i0 && i < i1) {
      const int v = L::N == 1 ? tid : tid + NT * i, kl = v / L::PER;   // N = 1: k-line of pass 0; passes add multiples of 16
      // 16-row chunks swap in pairs on odd eights of k
      *reinterpret_cast<u32x4*>(lds + (kl + (L::N == 1 ? L::KSTEP * i : 0)) * LDR + (((v % L::PER) ^ (((kl >> 3) & 1) << 1)) * 8)) = f.v[i];
    }
}

// MFMA operand fragment for lane (row = lane%16, g = lane/16): the 8 values k = k32 + 8g .. +7 of that row
// (row0 is a multiple of 16, so the row's value mod 8 is the lane's).
__device__ __forceinline__ bf16x8 frag_kmajor(const bf16* tile, int row0, int k32, int lane) {
  return *reinterpret_cast<const bf16x8*>(tile + (row0 + (lane & 15)) * LDK + (((k32 >> 3) + (lane >> 4)) ^ (lane & 7)) * 8);
}
// Same fragment from a [k][row] tile.  One transpose read serves 16 lanes: lane r of the group points at
// 4 consecutive rows of k-line (r/4) and receives the 4 k-lines' values of ONE row; group g reads k-lines k32 + 8g ...
// The LDS serves two groups per cycle, here the SAME 16 rows of k-lines 8 apart, i.e. the same banks; so the slab is
// stored with each pair of 16-row chunks swapped on the odd eights of k (store_rmajor), and the read undoes it.
template <int R> __device__ __forceinline__ bf16x8 frag_rmajor(const bf16* tile, int row0, int k32, int lane) {
  constexpr int LDR = R + RPAD;
  const int r = lane & 15, gi = lane >> 4;
  const bf16* p = tile + (k32 + 8 * gi + (r >> 2)) * LDR + ((row0 + 4 * (r & 3)) ^ ((gi & 1) << 4));
  union { struct { s16x4 a, b; } s; bf16x8 v; } u;
  u.s.a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
  u.s.b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * LDR));
  return u.v;
}

// Workgroup id -> tile origin.  Ids are dealt round-robin to the 8 XCDs, so id%8 picks the XCD; each XCD
// is given a contiguous run of the tile order, and that order walks groups of 8 tile rows column by
// column, so the tiles an XCD works on at one time share A rows and B columns in its L2.
template <int BM, int BN>
__device__ __forceinline__ void tile_origin(int pid, int tiles_m, int tiles_n, int& m0, int& n0) {
  const int ntiles = tiles_m * tiles_n;
  const int per = ntiles / 8;                             // ids [0, 8*per) are remapped, the rest stay
  if (pid < per * 8) pid = (pid % 8) * per + pid / 8;
  int tm, tn;
  gemm_tile_of(pid, tiles_m, tiles_n, tm, tn);
  m0 = tm * BM;
  n0 = tn * BN;
}

// All epilogues pass the tile through LDS (free after the K loop) as fp32, in two halves of BM/2 rows: every wave's first MI/2 rows
// of blocks, then its last.  So after the first half every wave has half of its accumulator registers free, for the
// residual, angles, gate and up values of the second: those loads go out before the first half's stores, and the wait for them
// stands behind no store.
// The MFMAs were issued with the operands swapped, mfma(B fragment, A fragment), which yields the
// transposed block: acc[i][j][r] is C[row, col] of 16x16 block (i, j) with row = lane%16 and col = 4*(lane/16) + r,
// so a lane owns 4 consecutive columns per block and writes them as one float4.
template <int BN> struct Staging { static constexpr int LDW = BN + 4; };   // padded row (floats)

// RW: rows of a wave.  Row of the tile that staged row r of a half holds.
template <int RW> __device__ __forceinline__ int staged_row(int r, int half) { return r / (RW / 2) * RW + half * (RW / 2) + r % (RW / 2); }

template <int BN, int MI, int NJ>
__device__ __forceinline__ void stage_quads(float* stage, f32x4 (&acc)[MI][NJ], int half, int wm, int wn, int lane) {
  constexpr int LDW = Staging<BN>::LDW;
#pragma unroll
  for (int i = 0; i < MI / 2; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      *reinterpret_cast<f32x4*>(stage + (wm / 2 + i * 16 + (lane & 15)) * LDW + wn + j * 16 + 4 * (lane >> 4)) = acc[half * (MI / 2) + i][j];
}

// Epilogue for C (fp32) += product (no bias, no residual).  Ct points at the tile's first element, of which rows x cols
// exist.  After staging, ALL threads walk the half tile 4 columns at a time: the old values of C are loaded 16 bytes per
// lane (consecutive lanes, consecutive pieces of a row), all loads of a half in flight across the barriers, then sum and
// store.  The first half's loads go out before the barrier that ends the K loop (4096 x 4096, K = 512 on 128x128 tiles 38 -> 34 us);
// the second half's wait until the first half's stores are out: with many rounds of workgroups at HBM rate reads, then
// writes, then reads again are faster than all reads first (4096 x 32000, K = 2048 552 : 572 us).  Loads and stores go through a buffer descriptor over the tile: rows past the last one fall beyond num_records
// and columns past the last one are sent there, so the ragged edge needs no branches.  A tile belongs to one workgroup and
// launches are ordered by the stream, so the sum over microbatches is formed in a fixed order.  overwrite: the tile is
// stored as it is (a partial sum that another kernel adds to C).
template <int BM, int BN, int NT, int MI, int NJ>
__device__ __forceinline__ void epilogue_accum(float* Ct, int ldc, int rows, int cols, bool overwrite, f32x4 (&acc)[MI][NJ],
                                               int wm, int wn, int tid, float* stage) {
  constexpr int LDW = Staging<BN>::LDW;
  static_assert((BM / 2) * LDW * 4 <= 2 * (slab_elems(BM) + slab_elems(BN)) * 2, "staging tile must fit the K-loop buffers");
  constexpr int VPR = BN / 4;                              // float4 per row
  constexpr int NS = NT % VPR == 0 ? NT : 8 * VPR;         // threads that store: whole rows at a time (BN = 192: 384 of 512)
  constexpr int NV = (BM / 2) * VPR / NS;                  // float4 per thread and half
  static_assert(NS <= NT && (BM / 2) * VPR % NS == 0, "a half is whole passes");
  const __amdgpu_buffer_rsrc_t rsC = make_rsrc(Ct, (uint32_t)((int64_t)(rows - 1) * ldc + cols) * 4u);
  const int lr0 = tid / VPR, cv = tid % VPR;               // vector v = tid + NS*it: staged row lr0 + (NS/VPR)*it, same columns
  const bool col_ok = cv * 4 < cols && tid < NS;           // cols is a multiple of 4
  u32x4 old[2][NV];
  auto offset = [&](int half, int it) {
    return col_ok ? (int)((uint32_t)(staged_row<16 * MI>(lr0 + (NS / VPR) * it, half) * ldc + cv * 4) * 4u) : (int)0x80000000u;
  };
  auto load = [&](int half) {
#pragma unroll
    for (int it = 0; it < NV; ++it)
      old[half][it] = overwrite ? u32x4{0u, 0u, 0u, 0u} : __builtin_amdgcn_raw_buffer_load_b128(rsC, offset(half, it), 0, 0);
  };
  load(0);
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    __syncthreads();
    stage_quads<BN, MI, NJ>(stage, acc, half, wm, wn, tid & 63);
    if (half == 1) load(1);
    __syncthreads();
#pragma unroll
    for (int it = 0; it < NV; ++it) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(stage + (lr0 + (NS / VPR) * it) * LDW + cv * 4);
      union { u32x4 u; f32x4 f; } o;
      o.u = old[half][it];
      o.f += x;
      __builtin_amdgcn_raw_buffer_store_b128(o.u, rsC, offset(half, it), 0, 0);
    }
  }
}

// The matrix-core instruction for the element type E; fragments travel as 16-bit containers (bf16x8).
// 16x16x32 rather than 32x32x16: the same flops per cycle, but per flop it moves a fifth fewer register bytes (A, B, C
// and D of one instruction), and the chip, which runs these kernels at its power limit, clocks higher for it: with random
// operands in registers and no memory traffic 2.08 PFLOP/s are sustained against 1.79-1.85.
template <typename E> __device__ __forceinline__ f32x4 mfma_16x16x32(bf16x8 a, bf16x8 b, f32x4 c);
template <> __device__ __forceinline__ f32x4 mfma_16x16x32<bf16>(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
template <> __device__ __forceinline__ f32x4 mfma_16x16x32<f16>(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// Epilogue for 16-bit output (E = bf16 or IEEE half): after staging, ALL threads read rows back 8 columns at a time, add bias and
// residual in fp32, round once to bf16 and store 16 bytes per lane, consecutive lanes covering
// consecutive 16-byte pieces of a row of C.  A thread keeps its 8 columns through all rows it visits, so the bias is
// loaded once, and what depends on the row (residual, rotary angles, or the gate and up values of GLU = 2) is loaded
// for a whole half before the staging barrier: the loads' latency runs under the staging instead of once per row.
template <typename E, int BM, int BN, int NT, int MI, int NJ, int GLU>
__device__ __forceinline__ void epilogue_store(const Gemm& g, int z, f32x4 (&acc)[MI][NJ], int m0, int n0, int wm,
                                               int wn, int tid, float* stage) {
  constexpr int LDW = Staging<BN>::LDW;
  static_assert((BM / 2) * LDW * 4 <= 2 * (slab_elems(BM) + slab_elems(BN)) * 2, "staging tile must fit the K-loop buffers");
  constexpr int VPR = BN / 8;                              // 16-byte output vectors per row
  constexpr int NS = NT % VPR == 0 ? NT : 16 * VPR;        // threads that store: whole rows at a time (BN = 192: 384 of 512)
  constexpr int NV = (BM / 2) * VPR / NS;                  // vectors per thread and half
  constexpr int RSTEP = NS / VPR;                          // rows between a thread's consecutive vectors
  static_assert(NS <= NT && ((BM / 2) * VPR) % NS == 0, "a thread keeps its columns");
  typedef typename Vec<E>::type E8;
  const int lane = tid & 63;
  const E* bias = g.bias ? (const E*)g.bias + (int64_t)z * g.sBias : nullptr;
  const E* R = g.resid ? (const E*)g.resid + (int64_t)z * g.sC : nullptr;
  E* Cz = (E*)g.C + (int64_t)z * g.sC;
  const bool rope = g.rope && z < g.rope_batches;
  const int lr0 = tid / VPR, cv = (tid % VPR) * 8, col = tid < NS ? n0 + cv : g.N;
  const bool full = col + 8 <= g.N;                        // all 8 columns exist: the vector path
  const bool pre_resid = GLU == 0 && R, pre_rope = GLU == 0 && rope && !R;
  E8 bb = {};
  if (GLU == 0 && bias && full) bb = *reinterpret_cast<const E8*>(bias + col);
  u32x4 pre0[2][NV], pre1[2][NV];                          // one source address per slot, so each slot has one load
  const bool want0 = full && (GLU == 2 || pre_resid || pre_rope), want1 = full && (GLU == 2 || pre_rope);
  auto load = [&](int half) {
#pragma unroll
    for (int it = 0; it < NV; ++it) {
      const int row = m0 + staged_row<16 * MI>(lr0 + RSTEP * it, half);
      const E* src0 = nullptr;
      const E* src1 = nullptr;
      if (GLU == 2) {
        src0 = (const E*)g.gu + (int64_t)row * g.gu_ld + col;
        src1 = src0 + g.gu_up;
      } else if (pre_resid) {
        src0 = R + (int64_t)row * g.ldr + col;
      } else if (pre_rope) {                               // (cos, sin) of pairs 0,1 and 2,3 at this row's position
        const float2* cs = g.rope + (int64_t)(row % g.rope_S) * (g.rope_d / 2) + (col % g.rope_d) / 2;
        src0 = reinterpret_cast<const E*>(cs);
        src1 = reinterpret_cast<const E*>(cs + 2);
      }
      pre0[half][it] = pre1[half][it] = u32x4{0, 0, 0, 0};
      if (want0 && row < g.M) pre0[half][it] = *reinterpret_cast<const u32x4*>(src0);
      if (want1 && row < g.M) pre1[half][it] = *reinterpret_cast<const u32x4*>(src1);
    }
  };
  load(0);
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    __syncthreads();                                       // K-loop reads / previous half's reads are done
    stage_quads<BN, MI, NJ>(stage, acc, half, wm, wn, lane);
    if (half == 0) load(1);
    __syncthreads();
#pragma unroll
    for (int it = 0; it < NV; ++it) {
      const int lr = lr0 + RSTEP * it, row = m0 + staged_row<16 * MI>(lr, half);
      if (row >= g.M || col >= g.N) continue;
      const f32x4 x0 = *reinterpret_cast<const f32x4*>(stage + lr * LDW + cv);
      const f32x4 x1 = *reinterpret_cast<const f32x4*>(stage + lr * LDW + cv + 4);
      float x[8] = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
      if (GLU == 2) {   // x is da: (gate, up) of these 8 columns become (dgate, dup) in place (N is a multiple of 8)
        E* pg = (E*)g.gu + (int64_t)row * g.gu_ld + col;
        const E8 gg = __builtin_bit_cast(E8, pre0[half][it]), uu = __builtin_bit_cast(E8, pre1[half][it]);
        E8 og, ou;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          float dg, du;
          glu_df(x[e], (float)gg[e], (float)uu[e], dg, du);
          og[e] = (E)dg;
          ou[e] = (E)du;
        }
        *reinterpret_cast<E8*>(pg) = og;
        *reinterpret_cast<E8*>(pg + g.gu_up) = ou;
        continue;
      }
      if (full) {
        if (bias) {
#pragma unroll
          for (int e = 0; e < 8; ++e) x[e] += (float)bb[e];
        }
        if (R) {
          const E8 rr = __builtin_bit_cast(E8, pre0[half][it]);
#pragma unroll
          for (int e = 0; e < 8; ++e) x[e] += (float)rr[e];
        }
        if (rope) {   // rotate the 4 adjacent pairs by the angles of this row's position
          f32x4 t0, t1;
          if (pre_rope) {
            t0 = __builtin_bit_cast(f32x4, pre0[half][it]);
            t1 = __builtin_bit_cast(f32x4, pre1[half][it]);
          } else {
            const f32x4* cs = reinterpret_cast<const f32x4*>(g.rope + (int64_t)(row % g.rope_S) * (g.rope_d / 2) + (col % g.rope_d) / 2);
            t0 = cs[0];
            t1 = cs[1];
          }
          const float c4[4] = {t0[0], t0[2], t1[0], t1[2]}, s4[4] = {t0[1], t0[3], t1[1], t1[3]};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float u = x[2 * i], w = x[2 * i + 1];
            x[2 * i] = u * c4[i] - w * s4[i];
            x[2 * i + 1] = u * s4[i] + w * c4[i];
          }
        }
        E8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (E)x[e];
        *reinterpret_cast<E8*>(Cz + (int64_t)row * g.ldc + col) = o;
      } else {
        for (int e = 0; e < 8 && col + e < g.N; ++e) {
          float y = x[e];
          if (bias) y += (float)bias[col + e];
          if (R) y += (float)R[(int64_t)row * g.ldr + col + e];
          Cz[(int64_t)row * g.ldc + col + e] = (E)y;
        }
      }
    }
  }
}

// Epilogue of the gate|up projection (GLU = 1): the tile's first BN/2 columns are gate columns c0 .. and its last
// BN/2 the up columns of the same index.  Both are rounded and stored into gu, and silu(gate) * up of the rounded
// values goes to C: the three arrays the batched product followed by the activation kernel would leave.
template <typename E, int BM, int BN, int NT, int MI, int NJ>
__device__ __forceinline__ void epilogue_glu(const Gemm& g, f32x4 (&acc)[MI][NJ], int m0, int c0, int wm, int wn, int tid,
                                             float* stage) {
  constexpr int LDW = Staging<BN>::LDW;
  typedef typename Vec<E>::type E8;
  const int lane = tid & 63;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    __syncthreads();
    stage_quads<BN, MI, NJ>(stage, acc, half, wm, wn, lane);
    __syncthreads();
    constexpr int VPR = BN / 16;                           // 8-column pieces of each matrix per row
#pragma unroll
    for (int it = 0; it < (BM / 2) * VPR / NT; ++it) {
      const int v = tid + NT * it;
      const int lr = v / VPR, cv = (v % VPR) * 8, col = c0 + cv;
      const int row = m0 + staged_row<16 * MI>(lr, half);
      if (row >= g.M || col >= g.N) continue;              // N is a multiple of 8
      const float* sp = stage + lr * LDW + cv;
      const f32x4 g0 = *reinterpret_cast<const f32x4*>(sp), g1 = *reinterpret_cast<const f32x4*>(sp + 4);
      const f32x4 u0 = *reinterpret_cast<const f32x4*>(sp + BN / 2), u1 = *reinterpret_cast<const f32x4*>(sp + BN / 2 + 4);
      E8 og, ou, oa;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        og[e] = (E)(e < 4 ? g0[e & 3] : g1[e & 3]);
        ou[e] = (E)(e < 4 ? u0[e & 3] : u1[e & 3]);
        oa[e] = (E)glu_f((float)og[e], (float)ou[e]);
      }
      E* pg = (E*)g.gu + (int64_t)row * g.gu_ld + col;
      *reinterpret_cast<E8*>(pg) = og;
      *reinterpret_cast<E8*>(pg + g.gu_up) = ou;
      *reinterpret_cast<E8*>((E*)g.C + (int64_t)row * g.ldc + col) = oa;
    }
  }
}

// NW wavefronts: 4 as a 2 x 2 grid, or 8 as 2 (m) x 4 (n), on oblong tiles 4 x 2, in which case two waves share each SIMD and one
// wave's loads, LDS traffic and barrier waits overlap the other's MFMAs.
template <typename E, int BM, int BN, int NW, int TA, int TB, int SEG, int ACC, int GLU>
__global__ __launch_bounds__(64 * NW, (NW == 4 && BM * BN <= 128 * 128) ? 2 : 1) void gemm_mfma_kernel(Gemm g, int tiles_m,
                                                                                                        int tiles_n) {
  constexpr int NT = 64 * NW, WM = BM > BN ? 4 : 2, WN = NW / WM;   // threads; waves along m and n
  constexpr int MI = BM / (16 * WM), NJ = BN / (16 * WN);           // 16x16 blocks per wave along m and n
  constexpr int SLAB_A = slab_elems(BM), SLAB_B = slab_elems(BN);   // LDS elements per operand slab, either layout
  extern __shared__ __align__(16) char smem_raw[];
  bf16* smem = reinterpret_cast<bf16*>(smem_raw);        // [2 buffers][A slab | B slab]

  // A launch of a cut product (multi-part K, fp32 accumulation) covers tile_count positions of the tile order from tile_base
  // on, counted over all batches; its ids are dealt to the XCDs like those of a whole grid.
  int m0, n0, z = blockIdx.y, sub = 0;                    // sub: position inside the launch's range
  if (SEG && TA == 1 && TB == 0 && ACC && g.tile_count > 0) {
    const int per = g.tile_count / 8;
    sub = blockIdx.x;
    if (sub < per * 8) sub = (sub % 8) * per + sub / 8;
    const int pos = g.tile_base + sub, ntiles = tiles_m * tiles_n;
    int tm, tn;
    gemm_tile_of(pos % ntiles, tiles_m, tiles_n, tm, tn);
    z = pos / ntiles;
    m0 = tm * BM;
    n0 = tn * BN;
  } else {
    tile_origin<BM, BN>(blockIdx.x, tiles_m, tiles_n, m0, n0);
  }
  const bf16* A = (const bf16*)g.A + (int64_t)z * g.sA;
  const bf16* B = (const bf16*)g.B + (int64_t)z * g.sB;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave / WN) * (BM / WM), wn = (wave % WN) * (BN / WN);
  static_assert(GLU == 0 || (GLU == 1 && !TA && !TB && !SEG && !ACC) || (GLU == 2 && !TA && TB && !SEG && !ACC), "fused gated unit");
  const int nb0 = GLU == 1 ? n0 / 2 : n0;                // first column of the tile inside B (GLU = 1: inside each of the two)

  f32x4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;

  // While slab kt is multiplied out of one LDS buffer, slab kt+1 (loaded during the previous iteration) is written into the
  // other buffer BETWEEN the MFMA steps, and each register that has been written is loaded again at once, with its part of slab
  // kt+1+STAGES.  The LDS writes thereby overlap MFMAs instead of forming a phase of their own in which every wave of
  // the workgroup writes and the matrix cores idle.  A's vectors go before B's: written and loaded in turn, operands
  // whose rows straddle cache lines took up to 20 % longer (648 x 3040, K = 13824, rows 16 bytes off: 147 : 177 us).  With two
  // stages the 128x128 tile's loads have two slabs' time: 2048 x 2048, K = 8192 91 -> 76 us (80 with one); the
  // other tiles have no registers for them or gain nothing.
  constexpr int STAGES = BM == 128 ? 2 : 1;
  Frag<BM, NT> fa[STAGES];
  Frag<BN, NT> fb[STAGES];
  const int lda = (int)g.lda, ldb = (int)g.ldb;
  // PAIR: the K range is made of g.nx+1 parts of kseg rows, each with operands of its own (both row-contiguous)
  constexpr bool PAIR = SEG && TA == 1 && TB == 0;
  const int K1 = PAIR ? g.kseg : g.K;                    // rows of a part (or of the only one)
  const __amdgpu_buffer_rsrc_t rsA =
      make_rsrc(A, (uint32_t)(TA == 0 ? ((int64_t)(g.M - 1) * lda + g.K) : ((int64_t)(K1 - 1) * lda + g.M)) * 2u);
  const int nseg = (SEG && !PAIR) ? g.K / g.kseg : 1;
  const __amdgpu_buffer_rsrc_t rsB = make_rsrc(
      B, (uint32_t)(TB == 1 ? ((int64_t)(nseg - 1) * g.segB + (int64_t)(g.N - 1) * ldb + (SEG ? g.kseg : g.K))
                            : ((int64_t)(K1 - 1) * ldb + g.N + (GLU == 1 ? g.sB : 0))) * 2u);
  // Descriptors of part p >= 1 (the last part has the rows that remain); a part past the last one gets an empty
  // range, so a surplus slab reads zeros.
  // A launch may cut the K range into chunks of chunk_parts parts (grid.z chunks): this workgroup then multiplies the
  // parts p0..p1 only; chunk 0 adds its tile to C, the others store theirs as partial sums.
  const int chunk = (PAIR && ACC) ? (int)blockIdx.z : 0;
  const int cparts = (PAIR && ACC && g.chunk_parts > 0 && gridDim.z > 1) ? g.chunk_parts : g.nx + 1;
  const int p0 = chunk * cparts, p1 = min(g.nx, p0 + cparts - 1);
  auto part_a = [&](int p) {
    const int rows = p < g.nx ? K1 : g.K - g.nx * K1;
    return (p >= 1 && p <= p1) ? make_rsrc((const bf16*)g.Ax[p - 1] + (int64_t)z * g.sA, (uint32_t)((int64_t)(rows - 1) * lda + g.M) * 2u)
                               : make_rsrc(A, 0u);
  };
  auto part_b = [&](int p) {
    const int rows = p < g.nx ? K1 : g.K - g.nx * K1;
    return (p >= 1 && p <= p1) ? make_rsrc((const bf16*)g.Bx[p - 1] + (int64_t)z * g.sB, (uint32_t)((int64_t)(rows - 1) * ldb + g.N) * 2u)
                               : make_rsrc(B, 0u);
  };
  // The load cursor: descriptors and first row (PAIR: inside the part) of the next slab to be fetched.
  __amdgpu_buffer_rsrc_t curA = PAIR && p0 > 0 ? part_a(p0) : rsA, curB = PAIR && p0 > 0 ? part_b(p0) : rsB;
  int curk = 0, curp = p0;
  auto advance = [&](bool odd) {                           // odd: past a slab of odd number; parts are pairs of slabs, but for the last
    curk += BK;
    if (PAIR && odd && curk >= (curp < g.nx ? K1 : g.K - g.nx * K1)) {
      ++curp;
      curk = 0;
      curA = part_a(curp);
      curB = part_b(curp);
    }
  };
  const int voffA = ((tid >> 3) * lda + (tid & 7) * 8) * 2, voffB = ((tid >> 3) * ldb + (tid & 7) * 8) * 2;   // k contiguous
  const LineOffsets<BM, NT> lineA = voff_rmajor<BM, NT, false>(lda, tid, m0, g.M, 0);                           // row contiguous
  const LineOffsets<BN, NT> lineB = voff_rmajor<BN, NT, GLU == 1>(ldb, tid, nb0, g.N, (int)g.sB);

  constexpr int VA = BM * 8 / NT, VB = BN * 8 / NT;        // 16-byte vectors per thread and slab
  // Loads the thread's vectors [a0, a1) of A and [b0, b1) of B of the slab under the cursor.
  auto fetch = [&](Frag<BM, NT>& fa, Frag<BN, NT>& fb, int a0, int a1, int b0, int b1) {
    if (TA == 0) load_kmajor<BM, NT>(fa, curA, voffA, lda, m0, curk, g.K, tid, a0, a1);
    else load_rmajor<BM, NT>(fa, curA, lineA, lda, m0, curk, a0, a1);
    if (TB == 1) {
      int vo = voffB;
      if (SEG && !PAIR) {  // the thread's k offset inside the slab is fixed, so one segment lookup per slab
        const int seg = (curk + (tid & 7) * 8) / g.kseg;
        vo += seg * ((int)g.segB - g.kseg) * 2;          // element (n, k) of segment seg lies at seg*segB + n*ldb + k - seg*kseg
      }
      load_kmajor<BN, NT>(fb, curB, vo, ldb, n0, curk, g.K, tid, b0, b1);
    } else {
      load_rmajor<BN, NT>(fb, curB, lineB, ldb, nb0, curk, b0, b1);
    }
  };
  auto stash_a = [&](int buf, const Frag<BM, NT>& fa, int i0 = 0, int i1 = 64) {
    bf16* As = smem + buf * (SLAB_A + SLAB_B);
    if (TA == 0) store_kmajor<BM, NT>(fa, As, tid, i0, i1); else store_rmajor<BM, NT>(fa, As, tid, i0, i1);
  };
  auto stash_b = [&](int buf, const Frag<BN, NT>& fb, int i0 = 0, int i1 = 64) {
    bf16* Bs = smem + buf * (SLAB_A + SLAB_B) + SLAB_A;
    if (TB == 1) store_kmajor<BN, NT>(fb, Bs, tid, i0, i1); else store_rmajor<BN, NT>(fb, Bs, tid, i0, i1);
  };
  // multiplies the slab in LDS buffer `buf`; after each of the eight regions of MFMAs it writes a quarter of one operand's part of
  // the next slab (held in fa, fb) into the other buffer, which nobody reads now, and loads the same registers again.
  // The loads are spread out because the CU's load unit takes 16 cycles per 1 KB wave load, and a wave that issues its whole
  // share at once (64 loads per workgroup and slab, all waves at the same point of the loop) waits in that unit's queue for
  // hundreds of cycles in which it issues no MFMA.  The scheduling fences keep the compiler from gathering the loads
  // at the end of the loop body again.
  static_assert(MI == 8 || MI == 4, "a share of the loads and stores goes out after every MI/4 rows of MFMA blocks");
  // A slab is multiplied in 8 regions of MI/4 rows of blocks each.  The schedule is laid down by hand, with scheduling
  // fences between its parts: a region first issues the LDS reads of the NEXT region's fragments, then its own MFMAs,
  // then a quarter of one operand's share of the next slab's stores, then its share of the global loads.
  auto multiply = [&](int buf, Frag<BM, NT>& fa, Frag<BN, NT>& fb) {
    const bf16* As = smem + buf * (SLAB_A + SLAB_B);
    const bf16* Bs = As + SLAB_A;
    constexpr int RI = MI / 4;                             // rows of blocks per region
    bf16x8 a[2][RI], b[2][NJ];
    auto read_a = [&](int e) {                             // fragments of region e = 4 ks + q
#pragma unroll
      for (int ii = 0; ii < RI; ++ii) {
        const int row = wm + ((e & 3) * RI + ii) * 16, k32 = (e >> 2) * 32;
        a[e & 1][ii] = TA == 0 ? frag_kmajor(As, row, k32, lane) : frag_rmajor<BM>(As, row, k32, lane);
      }
    };
    auto read_b = [&](int ks) {
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        b[ks][j] = TB == 1 ? frag_kmajor(Bs, wn + j * 16, ks * 32, lane) : frag_rmajor<BN>(Bs, wn + j * 16, ks * 32, lane);
    };
    read_b(0);
    read_a(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (e == 2) read_b(1);
      if (e < 7) read_a(e + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ii = 0; ii < RI; ++ii)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[(e & 3) * RI + ii][j] = mfma_16x16x32<E>(b[e >> 2][j], a[e & 1][ii], acc[(e & 3) * RI + ii][j]);
      const int i0 = e & 3, i1 = i0 + 1;
      if (e < 4) stash_a(buf ^ 1, fa, i0 * VA / 4, i1 * VA / 4);
      else stash_b(buf ^ 1, fb, i0 * VB / 4, i1 * VB / 4);
      __builtin_amdgcn_sched_barrier(0);
      if (e < 4) fetch(fa, fb, i0 * VA / 4, i1 * VA / 4, 0, 0);
      else fetch(fa, fb, 0, 0, i0 * VB / 4, i1 * VB / 4);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // Slabs past K read zeros (their loads are out of range), so the loop needs no conditions: it walks K in
  // pairs of slabs and a surplus slab contributes nothing.
  int nk = (g.K + BK - 1) / BK;
  if (PAIR && ACC && gridDim.z > 1) {                      // this chunk's parts only
    const int last = p1 < g.nx ? K1 : g.K - g.nx * K1;
    nk = ((p1 - p0) * K1 + last + BK - 1) / BK;
  }
  if constexpr (MI == 4) {
    bf16x8 a[2][MI], b[2][NJ];                             // fragments of the half slab being multiplied and of the next one
    // Waves with 4 rows of blocks have registers for the fragments of a whole half slab (32 k) ahead, so the barrier stands
    // between a slab's halves: behind it the next slab is complete in LDS and this slab's fragments are all in registers.
    // This multiplies the half whose fragments are in a[ks], b[ks].  Meanwhile the fragments of the next half are read from
    // LDS (`buf`, its half ks ^ 1; read), and the vectors of fa (part 0) or fb (part 1) go to LDS buffer `to` (stash) and are
    // loaded again (more).
    auto half_slab = [&](int ks, int buf, int to, Frag<BM, NT>& fa, Frag<BN, NT>& fb, int part, bool read, bool stash, bool more) {
      const bf16* As = smem + buf * (SLAB_A + SLAB_B);
      const bf16* Bs = As + SLAB_A;
      const int nx = ks ^ 1, k32 = nx * 32;
#pragma unroll
      for (int e = 0; e < MI; ++e) {
        if (e == 0 && read) {
#pragma unroll
          for (int j = 0; j < NJ; ++j) b[nx][j] = TB == 1 ? frag_kmajor(Bs, wn + j * 16, k32, lane) : frag_rmajor<BN>(Bs, wn + j * 16, k32, lane);
        } else if (e == 1 && read) {
#pragma unroll
          for (int i = 0; i < MI; ++i) a[nx][i] = TA == 0 ? frag_kmajor(As, wm + i * 16, k32, lane) : frag_rmajor<BM>(As, wm + i * 16, k32, lane);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[e][j] = mfma_16x16x32<E>(b[ks][j], a[ks][e], acc[e][j]);
        const int i0 = e * (part ? VB : VA) / 4, i1 = (e + 1) * (part ? VB : VA) / 4;
        const int a0 = part ? 0 : i0, a1 = part ? 0 : i1, b0 = part ? i0 : 0, b1 = part ? i1 : 0;
        if (stash) {
          stash_a(to, fa, a0, a1);
          stash_b(to, fb, b0, b1);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (more) fetch(fa, fb, a0, a1, b0, b1);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // From slab 0 in LDS to the fragments of its first half in registers and slab 1's part of A in LDS.
    auto begin = [&](bool more) {
      if (STAGES == 1 || more) fetch(fa[0], fb[0], 0, VA, 0, VB);
      advance(STAGES == 1);
      __syncthreads();
#pragma unroll
      for (int j = 0; j < NJ; ++j) b[0][j] = TB == 1 ? frag_kmajor(smem + SLAB_A, wn + j * 16, 0, lane) : frag_rmajor<BN>(smem + SLAB_A, wn + j * 16, 0, lane);
#pragma unroll
      for (int i = 0; i < MI; ++i) a[0][i] = TA == 0 ? frag_kmajor(smem, wm + i * 16, 0, lane) : frag_rmajor<BM>(smem, wm + i * 16, 0, lane);
      stash_a(1, fa[1 % STAGES]);
      if (more) fetch(fa[1 % STAGES], fb[1 % STAGES], 0, VA, 0, 0);
    };
    // A pair of slabs; pairs: how many follow, 2: two or more.
    auto pair = [&](int pairs) {
      const bool next = pairs > 0, more = pairs > 1;
      half_slab(0, 0, 1, fa[1 % STAGES], fb[1 % STAGES], 1, true, true, next);
      advance(STAGES == 2);
      __syncthreads();
      half_slab(1, 1, 0, fa[0], fb[0], 0, true, next, more);
      half_slab(0, 1, 0, fa[0], fb[0], 1, true, next, more);
      if (next) {
        advance(STAGES == 1);
        __syncthreads();
      }
      half_slab(1, 0, 1, fa[1 % STAGES], fb[1 % STAGES], 0, next, next, more);
    };
#pragma unroll
    for (int i = 0; i < STAGES; ++i) {
      fetch(fa[i], fb[i], 0, VA, 0, VB);
      advance(i & 1);
    }
    stash_a(0, fa[0]);
    stash_b(0, fb[0]);
    if constexpr (STAGES == 2) {
      // Slabs past the end cost their loads' issue (16 cycles per wave) although they read zeros, so the last two pairs of slabs
      // load none.  us on 128x128 tiles, 694 x 6888 (x W^T), with loads up to the fourth slab past the end : up to the end: K = 64
      // 9.6 : 8.4, K = 256 10.9 : 10.5, K = 1024 19.3 : 18.9.  The other tiles have no registers for further bodies.
      if (nk > 2) {
        begin(true);
        for (int kt = 0; kt + 4 < nk; kt += 2) pair(2);
        pair(1);
      } else {
        begin(false);
      }
      pair(0);
    } else {
      begin(true);
      for (int kt = 0; kt < nk; kt += 2) pair(2);
    }
  } else {
    fetch(fa[0], fb[0], 0, VA, 0, VB);
    advance(false);
    stash_a(0, fa[0]);
    stash_b(0, fb[0]);
    fetch(fa[0], fb[0], 0, VA, 0, VB);
    advance(true);
    __syncthreads();
    for (int kt = 0; kt < nk; kt += 2) {
      multiply(0, fa[0], fb[0]);
      advance(false);
      __syncthreads();
      multiply(1, fa[0], fb[0]);
      advance(true);
      __syncthreads();
    }
  }

  if (ACC) {
    if (chunk == 0) {
      float* Ct = (float*)g.C + (int64_t)z * g.sC + (int64_t)m0 * g.ldc + n0;
      epilogue_accum<BM, BN, NT, MI, NJ>(Ct, (int)g.ldc, min(BM, g.M - m0), min(BN, g.N - n0), !PAIR && g.c_overwrite, acc, wm, wn, tid,
                                         reinterpret_cast<float*>(smem_raw));
    } else {   // partial tile number (chunk-1) * tile_count + position inside the launch's range
      const int64_t slot = (int64_t)(chunk - 1) * g.tile_count + sub;
      epilogue_accum<BM, BN, NT, MI, NJ>((float*)g.ws + slot * (BM * BN), BN, BM, BN, true, acc, wm, wn, tid,
                                         reinterpret_cast<float*>(smem_raw));
    }
  }
  else if (GLU == 1) epilogue_glu<E, BM, BN, NT, MI, NJ>(g, acc, m0, nb0, wm, wn, tid, reinterpret_cast<float*>(smem_raw));
  else epilogue_store<E, BM, BN, NT, MI, NJ, GLU>(g, z, acc, m0, n0, wm, wn, tid, reinterpret_cast<float*>(smem_raw));
}

template <typename E, int BM, int BN, int NW, int TA, int TB, int SEG, int ACC, int GLU = 0>
hipError_t launch2(hipStream_t st, const Gemm& g) {
  constexpr size_t SMEM_BYTES = 2 * (slab_elems(BM) + slab_elems(BN)) * sizeof(bf16);
  static bool configured = false;
  auto kern = gemm_mfma_kernel<E, BM, BN, NW, TA, TB, SEG, ACC, GLU>;
  if (!configured) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)SMEM_BYTES);
    if (e != hipSuccess) return e;
    configured = true;
  }
  const int tiles_m = (int)cdiv(g.M, BM), tiles_n = (int)cdiv(g.N, GLU == 1 ? BN / 2 : BN);   // a gate|up tile holds BN/2 columns of each
  const bool range = SEG && TA == 1 && TB == 0 && ACC && g.tile_count > 0;   // part of a cut product
  const bool chunks = range && g.chunk_parts > 0 && g.nchunks > 1;
  dim3 grid((unsigned)(tiles_m * tiles_n), (unsigned)g.batch), blk(64 * NW);
  if (range) grid = dim3((unsigned)g.tile_count, 1u, chunks ? (unsigned)g.nchunks : 1u);
  hipLaunchKernelGGL(kern, grid, blk, SMEM_BYTES, st, g, tiles_m, tiles_n);
  return hipGetLastError();
}

template <typename E, int BM, int BN, int NW, int TA, int TB, int SEG> hipError_t launch(hipStream_t st, const Gemm& g) {
  return g.c_f32_accum ? launch2<E, BM, BN, NW, TA, TB, SEG, 1>(st, g) : launch2<E, BM, BN, NW, TA, TB, SEG, 0>(st, g);
}

// The square tiles take every form, the oblong ones those of gemm_mfma_oblong.
template <typename E, int BM, int BN, int NW> hipError_t gemm_mfma_tile(hipStream_t st, const Gemm& g) {
  if (g.glu == 1) return launch2<E, BM, BN, NW, 0, 0, 0, 0, 1>(st, g);
  if (g.glu == 2) return launch2<E, BM, BN, NW, 0, 1, 0, 0, 2>(st, g);
  if constexpr (BM == BN) {
    if (g.nx) return launch<E, BM, BN, NW, 1, 0, 1>(st, g);
    if (g.kseg) return g.transA ? launch<E, BM, BN, NW, 1, 1, 1>(st, g) : launch<E, BM, BN, NW, 0, 1, 1>(st, g);
    if (!g.transA && !g.transB) return launch<E, BM, BN, NW, 0, 0, 0>(st, g);
    if (!g.transA && g.transB) return launch<E, BM, BN, NW, 0, 1, 0>(st, g);
    if (g.transA && !g.transB) return launch<E, BM, BN, NW, 1, 0, 0>(st, g);
    return launch<E, BM, BN, NW, 1, 1, 0>(st, g);
  } else {
    if (!gemm_mfma_oblong(g)) return hipErrorInvalidValue;
    if (g.transA) return launch2<E, BM, BN, NW, 1, 0, 0, 1>(st, g);
    if (!g.transB) return launch2<E, BM, BN, NW, 0, 0, 0, 0>(st, g);
    if (g.kseg) return launch2<E, BM, BN, NW, 0, 1, 1, 0>(st, g);
    return launch<E, BM, BN, NW, 0, 1, 0>(st, g);
  }
}

}  // namespace gemm_impl
}  // namespace zs

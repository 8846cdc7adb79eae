// 16-bit (bf16 / fp16) MFMA GEMM: argument checks and the choice of workgroup tile.  The kernels live in
// gemm_mfma_impl.h, one translation unit per tile shape.
#include "kernels.h"

#include <algorithm>

namespace zs {

hipError_t gemm_mfma_256x256(hipStream_t st, const Gemm& g);   // 8 wavefronts
hipError_t gemm_mfma_256x192(hipStream_t st, const Gemm& g);
hipError_t gemm_mfma_256x128(hipStream_t st, const Gemm& g);   // 8 wavefronts
hipError_t gemm_mfma_128x128(hipStream_t st, const Gemm& g);   // 4 wavefronts, two workgroups per CU
hipError_t gemm_mfma_256x256_f16(hipStream_t st, const Gemm& g);
hipError_t gemm_mfma_256x192_f16(hipStream_t st, const Gemm& g);
hipError_t gemm_mfma_256x128_f16(hipStream_t st, const Gemm& g);
hipError_t gemm_mfma_128x128_f16(hipStream_t st, const Gemm& g);

namespace {
bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }
int g_force_tile = 0;   // 0 automatic; 1: 256x256, 2: 128x128, 3: 256x192, 4: 256x128 (set through gemm_mfma_force_tile)
}  // namespace

// The kernel needs 16-byte aligned rows for its vector loads: base pointers 16-byte aligned and
// every leading dimension, batch stride and segment size a multiple of 8 elements; the extent
// along each operand's contiguous axis must be a multiple of 8 as well.  K may be anything when neither operand is
// k-contiguous (weight gradients over an odd number of tokens): k-lines past the end lie behind both descriptors.
bool gemm_mfma_supported(DType dt, const Gemm& g) { return g.K % 8 == 0 && gemm_mfma_takes(dt, g); }

bool gemm_mfma_takes(DType dt, const Gemm& g) {
  if ((dt != BF16 && dt != F16) || g.act) return false;
  if (g.M < 1 || g.N < 1 || g.K < 1 || g.batch < 1) return false;
  if (!aligned16(g.A) || !aligned16(g.B)) return false;
  if (g.lda % 8 || g.ldb % 8 || g.sA % 8 || g.sB % 8) return false;
  if (g.K % 8 && !(g.transA && !g.transB)) return false;   // k-contiguous operands are read 8 k at a time; tails are zero-filled
  if (g.transA && g.M % 8) return false;           // row-contiguous operands are read 8 rows at a time
  if (!g.transB && g.N % 8) return false;
  if (g.glu) {   // gated unit fused into the store
    if (g.glu != 1 && g.glu != 2) return false;
    if (g.transA || (g.glu == 1) == (g.transB != 0)) return false;   // 1: y = x [Wg | Wu]; 2: da = dy Wd^T
    if (g.c_f32_accum || g.batch != 1 || g.bias || g.resid || g.rope || g.kseg || g.nx) return false;
    if (!g.gu || !aligned16(g.gu) || g.gu_ld % 8 || g.gu_up % 8 || g.N % 8) return false;
    if (g.glu == 1 && g.sB <= 0) return false;
  }
  if (g.nx) {   // multi-part K range of an accumulating product
    if (g.nx < 0 || g.nx >= GEMM_MAX_PARTS) return false;
    // the K loop takes two slabs of 64 rows per step, and a step must lie inside one part
    if (!g.transA || g.transB || !g.c_f32_accum || g.kseg <= 0 || g.kseg % 128 || (int64_t)g.kseg * g.nx >= g.K) return false;
    for (int p = 0; p < g.nx; ++p)
      if (!g.Ax[p] || !g.Bx[p] || !aligned16(g.Ax[p]) || !aligned16(g.Bx[p])) return false;
  } else if (g.kseg) {
    if (!g.transB || g.kseg % 8 || g.segB % 8 || g.K % g.kseg) return false;
  }
  // the bf16 epilogue moves 8 consecutive columns per 16-byte access
  if (!g.c_f32_accum) {
    if (!aligned16(g.C) || g.ldc % 8 || g.sC % 8) return false;
    if (g.resid && (!aligned16(g.resid) || g.ldr % 8)) return false;
    if (g.bias && (!aligned16(g.bias) || g.sBias % 8)) return false;
    // the fused rotation works on whole 8-column vectors that do not straddle heads
    if (g.rope && (g.N % 8 || g.rope_d % 8 || g.rope_S < 1 || ((uintptr_t)g.rope & 15))) return false;
  } else {
    if (g.rope) return false;
    // the accumulating epilogue updates 4 consecutive floats per 16-byte access through 32-bit byte offsets
    if (!aligned16(g.C) || g.ldc % 4 || g.sC % 4 || g.N % 4) return false;
    if (g.bias || g.resid) return false;
    if (((int64_t)g.M + 256) * g.ldc * 4 >= (1ll << 31)) return false;
  }
  // byte offsets inside one operand are 32-bit in the kernel
  // every part of a multi-part range has a descriptor of its own; the last part may be the longest
  const int64_t rowsA = g.nx ? ((int64_t)g.K - (int64_t)g.nx * g.kseg > g.kseg ? (int64_t)g.K - (int64_t)g.nx * g.kseg : g.kseg) : g.K;
  const int64_t extA = (g.transA ? rowsA * g.lda : (int64_t)g.M * g.lda) * 2;
  const int64_t nseg = g.kseg ? g.K / g.kseg : 1;
  const int64_t nsegB = g.nx ? 1 : nseg;
  const int64_t extB = (g.transB ? (nsegB - 1) * g.segB + (int64_t)g.N * g.ldb : rowsA * g.ldb + (g.glu == 1 ? g.sB : 0)) * 2;
  if (extA >= (1ll << 30) || extB >= (1ll << 30)) return false;
  // k-lines that fill up the last pair of slabs lie behind the descriptors, unless their offsets wrap around: few rows, far apart.
  // (With one operand k-contiguous its zeros stand against them.)
  if (g.transA && !g.transB && cdiv(rowsA, 128) * 128 * (g.lda > g.ldb ? g.lda : g.ldb) * 2 >= (1ll << 32)) return false;
  return true;
}

// Which tile: the MI355X has 256 CUs.  256x256 tiles (8 waves, one workgroup per CU) move the fewest LDS and L2 bytes per flop
// and run at the highest rate; 256x192 and 256x128 (8 waves, one per CU) and 128x128 (4 waves, two per CU) waste less of
// the last round of workgroups and give small products enough workgroups to fill the chip.  The tile with the smallest estimated
// time is taken.  The estimate: per round of workgroups a fixed time (first loads, store) and a time per 64-wide slab, which
// grows by 0.3 with the share of the chip at work (the clock drops); and the traffic of the result.  Constants fitted to 830
// times of 207 products (M 256 .. 8000, N 768 .. 16000, K 64 .. 14000, the three layouts): of these the pick is on the geometric mean
// within 0.3 % of the fastest tile, 12 % at worst; of 640 others, half of them with K up to 600, within 0.5 %, 18 % at worst (762 x 5904,
// K = 312, da: 18.6 on 128x128, 15.8 on 256x128).  us, bf16, 256x256 : 128x128 : 256x192 : 256x128: 2048 x 4096, K = 12288
// 244 : 207 : 221 : 185; 2048 x 5120, K = 12288 (dx) 248 : 310 : 219 : 349; 2048 x 6144, K = 2048 50 : 54 : 48 : 61;
// 2048 x 2048, K = 12288 225 : 119 : 201 : 155; 4096 x 11008, K = 4096 (dx) 297 : 357 : 318 : 348.
namespace {
struct TileTimes { int width, cus; double slab, round, store; };   // us; cus: workgroups that run side by side
constexpr TileTimes TILE_TIMES[4] = {{256, 256, 1.10, 5.9, 1.0}, {128, 512, 0.774, 4.0, 0.52}, {192, 256, 0.895, 5.9, 0.8}, {128, 256, 0.68, 4.0, 1.0}};
constexpr double HALF_SLAB = 0.492, HALF_ROUND = 2.4;              // 128x128, a round of at most 256 tiles: one per CU
constexpr double LAUNCH = 2.7, CROWDED = 0.294, STORE_RATE = 8.0e6; // us, -, bytes per us

// Estimated time of a grid of `small` 128x128 tiles in units of one round of 256x256 tiles: full rounds hold
// 512 small tiles (two per CU, each at 0.8 of the big tile's rate); a remainder of at most 256 tiles runs
// one per CU.
double small_rounds(int64_t small) {
  const int64_t rem = small % 512;
  return ((double)(small / 512) * 2.0 + (rem == 0 ? 0.0 : rem <= 256 ? 1.0 : 2.0)) * 0.25 / 0.8;
}
// Tile columns of a grid of tiles `width` wide: a gate|up tile (glu = 1) covers width/2 columns of each matrix.
int64_t tile_cols(const Gemm& g, int width) { return cdiv(g.N, g.glu == 1 ? width / 2 : width); }

double tile_us(const Gemm& g, int tile) {
  const TileTimes& t = TILE_TIMES[tile - 1];
  const double slabs = (double)cdiv(g.K, 64);
  const int64_t n = cdiv(g.M, tile == 2 ? 128 : 256) * tile_cols(g, t.width) * g.batch;
  const double bytes = (double)g.M * g.N * g.batch * (g.c_f32_accum ? (g.c_overwrite ? 4.0 : 8.0) : g.glu == 1 ? 6.0 : g.glu == 2 ? 8.0 : g.resid ? 4.0 : 2.0);
  const bool half = tile == 2 && n % 512 > 0 && n % 512 <= 256;
  const int64_t full = n / t.cus + (n % t.cus > 0 && !half);
  const double used = tile == 2 ? std::min(1.0, n / ((full + 0.5 * half) * 512.0)) : (double)n / (double)(full * t.cus);
  const double grow = 1.0 + CROWDED * used, grow_half = 1.0 + CROWDED * std::min(1.0, n / 512.0);
  return LAUNCH + full * (slabs * t.slab * grow + t.round) + (half ? slabs * HALF_SLAB * grow_half + HALF_ROUND : 0.0) + t.store * bytes / STORE_RATE;
}
}  // namespace

int gemm_mfma_pick_tile(const Gemm& g) {
  if (g_force_tile) return g_force_tile;
  int best = 1;
  double us = tile_us(g, 1);
  for (int tile = 2; tile <= (gemm_mfma_oblong(g) ? 4 : 2); ++tile) {
    const double t = tile_us(g, tile);
    if (t < us) { us = t; best = tile; }
  }
  return best;
}

double gemm_mfma_us(const Gemm& g) { return tile_us(g, gemm_mfma_pick_tile(g)); }

void gemm_mfma_force_tile(int id) { g_force_tile = id; }

namespace {

hipError_t run_tile(hipStream_t st, DType dt, const Gemm& g, int tile) {
  typedef hipError_t (*Run)(hipStream_t, const Gemm&);
  static const Run run[2][4] = {{gemm_mfma_256x256, gemm_mfma_128x128, gemm_mfma_256x192, gemm_mfma_256x128},
                                {gemm_mfma_256x256_f16, gemm_mfma_128x128_f16, gemm_mfma_256x192_f16, gemm_mfma_256x128_f16}};
  return run[dt == F16][tile - 1](st, g);
}

// Columns [0, n1) and [n1, N) of a product as products of their own.
bool cut_columns(DType dt, const Gemm& g, int64_t n1, Gemm& head, Gemm& tail) {
  if (n1 < 1 || n1 >= g.N || (g.rope && n1 % g.rope_d)) return false;
  head = g; tail = g;
  head.N = (int)n1;
  tail.N = g.N - (int)n1;
  const int64_t cb = g.c_f32_accum ? 4 : 2;
  tail.C = (char*)g.C + n1 * cb;
  if (g.bias) tail.bias = (const char*)g.bias + n1 * 2;
  if (g.resid) tail.resid = (const char*)g.resid + n1 * 2;
  if (g.gu) tail.gu = (char*)g.gu + n1 * 2;
  const int64_t boff = (g.transB ? n1 * g.ldb : n1) * 2;
  tail.B = (const char*)g.B + boff;
  for (int p = 0; p < g.nx; ++p) tail.Bx[p] = (const char*)g.Bx[p] + boff;
  return gemm_mfma_takes(dt, head) && gemm_mfma_takes(dt, tail);
}

// A grid of 256x256 tiles that ends in a round with few tiles (1376 tiles = 5 rounds + 96 tiles on 256 CUs) pays a whole round
// for them.  So the product may be cut along N: as many leading tile columns as fit the whole rounds run on 256-row tiles
// `wide`, the remaining ones on whatever tile suits them.
bool split_tail(DType dt, const Gemm& g, int wide, Gemm& head, Gemm& tail) {
  const int width = TILE_TIMES[wide - 1].width;
  const int64_t col = cdiv(g.M, 256) * g.batch, tiles = col * tile_cols(g, width);   // col: tiles per tile column
  if (tiles < 256 || tiles % 256 == 0) return false;
  return cut_columns(dt, g, tiles / 256 * 256 / col * (g.glu == 1 ? width / 2 : width), head, tail);
}

// ---- K range of the last round's tiles cut into chunks -------------------------------------------------------------
// A multi-part product whose 256x256 tiles do not fill whole rounds of 256 workgroups runs as two launches of the same
// kernel over ranges of its tile order (counted over all batches): the leading tiles, whole rounds, as they are, and the
// remaining `rem` tiles as rem x nchunks workgroups, each multiplying chunk_parts of the parts.  Chunk 0 adds to C; the
// other chunks leave partial tiles in scratch, which add_partials_kernel adds to C in the order of the chunks.
struct KCut {
  Gemm head, tail;
  int rem = 0;              // tiles of the cut-off range
  int64_t ws_need = 0;      // bytes of partial tiles
};

constexpr int64_t KCUT_MAX_WS = 256ll << 20;   // no plan wants more scratch than this

// Times of the cut-off tiles are estimated in units of one part on one tile, 2*256*256*kseg flops at the 5.3 TFLOP/s a
// CU sustains.  A round of workgroups costs its parts plus about 20 us for its first loads and its store pass; the second
// kernel reads the partial tiles and reads and writes C at about 4 TB/s.  Measured at 11008 x 4096 with 8 parts of 4096 rows:
// 2538 us uncut, 2458 us in 4 chunks of 2 parts (the estimate says 79 us less); with 4 parts a cut costs time, and is not made.
double kcut_part_seconds(int kseg) { return 2.0 * 256.0 * 256.0 * (double)kseg / 5.3e12; }
double kcut_round_fixed_parts(int kseg) { return 20e-6 / kcut_part_seconds(kseg); }
double kcut_fixup_parts(int rem, int nch, int kseg) {
  const double bytes = (double)(nch - 1 + 2) * rem * 256.0 * 256.0 * 4.0;
  return bytes / 4.0e12 / kcut_part_seconds(kseg);
}

bool plan_kcut(DType dt, const Gemm& g, KCut& k) {
  if (!g.nx || !g.c_f32_accum || !g.transA || g.transB || g.kseg < 1) return false;
  const int64_t tm = cdiv(g.M, 256), tn = cdiv(g.N, 256), tiles = tm * tn * g.batch, rem = tiles % 256;
  if (tiles < 256 || rem == 0 || tiles >= (1ll << 30)) return false;
  const int parts = g.nx + 1;
  const double fx = kcut_round_fixed_parts(g.kseg);
  double t_now = (double)parts + fx;                                  // a whole round
  Gemm h2, t2;
  // The other way is priced in one form: remaining tiles that are whole tile columns, and at most 128, on 128x128 tiles.  What else
  // gemm_mfma would cut along N counts as a whole round here.
  if (rem <= 128 && rem % (tm * g.batch) == 0 && split_tail(dt, g, 1, h2, t2))
    t_now = std::min(t_now, small_rounds(cdiv(t2.M, 128) * tile_cols(t2, 128) * t2.batch) * (parts + fx));
  double best = t_now * 0.97;                                         // a cut has to win at least 3 %
  int best_cp = 0;
  for (int cp = 1; cp < parts; ++cp) {
    const int nch = (int)cdiv(parts, cp);
    if ((int64_t)(nch - 1) * rem * 256 * 256 * 4 > KCUT_MAX_WS) continue;
    const double t = (double)cdiv(rem * nch, 256) * (cp + fx) + kcut_fixup_parts((int)rem, nch, g.kseg);
    if (t < best) { best = t; best_cp = cp; }
  }
  if (!best_cp) return false;
  k.rem = (int)rem;
  k.head = g; k.tail = g;
  k.head.ws = nullptr; k.head.ws_bytes = 0; k.head.chunk_parts = 0; k.head.nchunks = 1;
  k.head.tile_base = 0; k.head.tile_count = (int)(tiles - rem);
  k.tail.tile_base = (int)(tiles - rem); k.tail.tile_count = (int)rem;
  k.tail.chunk_parts = best_cp;
  k.tail.nchunks = (int)cdiv(parts, best_cp);
  k.ws_need = (int64_t)(k.tail.nchunks - 1) * rem * 256 * 256 * 4;
  return true;
}

// C tile += partial tile of chunk 1, then of chunk 2, ...: one workgroup per quarter tile (64 rows), 16 bytes per lane.
// Tile `idx` of the range is position tile_base + idx of the tile order.
__global__ __launch_bounds__(256) void add_partials_kernel(float* C, int64_t ldc, int64_t sC, int M, int N, int tiles_m, int tiles_n,
                                                           int tile_base, int tile_count, const float* __restrict__ partial, int nadd) {
  const int idx = blockIdx.x >> 2, quarter = blockIdx.x & 3;
  const int pos = tile_base + idx, ntiles = tiles_m * tiles_n;
  int tm, tn;
  gemm_tile_of(pos % ntiles, tiles_m, tiles_n, tm, tn);
  const int m0 = tm * 256 + quarter * 64, n0 = tn * 256;
  float* Cz = C + (int64_t)(pos / ntiles) * sC;
  const float* P0 = partial + (int64_t)idx * 65536 + quarter * 64 * 256;
  const int64_t chunk_stride = (int64_t)tile_count * 65536;
#pragma unroll 4
  for (int v = threadIdx.x; v < 64 * 64; v += 256) {
    const int r = v >> 6, c = (v & 63) * 4;
    if (m0 + r >= M || n0 + c >= N) continue;                         // N is a multiple of 4
    float* pc = Cz + (int64_t)(m0 + r) * ldc + n0 + c;
    f32x4 s = *reinterpret_cast<const f32x4*>(pc);
    for (int a = 0; a < nadd; ++a) s += *reinterpret_cast<const f32x4*>(P0 + a * chunk_stride + r * 256 + c);
    *reinterpret_cast<f32x4*>(pc) = s;
  }
}

}  // namespace

// ---- parts of K side by side ---------------------------------------------------------------------------------------
// A forward product or an input gradient over few tokens has few tiles and a long K (512 x 4096 with K = 22016: 128 tiles of 128x128,
// half the CUs idle, and each of the others waits for cold lines of the weights).  With scratch for as many fp32 results the two
// halves of its K, or an input gradient's segments (gate and up; Q, K and V), run as a batch, and a second kernel adds them, bias
// and residual, and rounds: taken when the estimate of both kernels (the second one at 4.5 TB/s) is the shorter time.  us: 512 x
// 4096, K = 22016 in 2 parts 176 -> 130 (128x128 tiles); K = 12288 in 3 segments 129 -> 82;
// forward, K = 11008 105 -> 65, K = 4096 49 -> 37.
namespace {
bool plan_parts(DType dt, const Gemm& g, Gemm& best) {
  if (g_force_tile || !g.ws || g.transA || g.c_f32_accum || g.batch != 1 || (g.transB && (g.bias || g.resid)) || g.rope || g.glu || g.nx) return false;
  const int64_t tiles = cdiv(g.M, 128) * cdiv(g.N, 128);
  if (tiles > 128 || g.N % 8 || ((uintptr_t)g.ws & 15)) return false;
  double us = 0.95 * gemm_mfma_us(g);
  best.batch = 1;
  for (int n = 2; n <= 3; ++n) {
    if (g.kseg ? (int64_t)n * g.kseg != g.K : n > 2 || g.K % 16) continue;
    if (g.ws_bytes < 4ll * n * g.M * g.N) continue;
    Gemm h = g;
    h.ws = nullptr; h.ws_bytes = 0; h.kseg = 0; h.segB = 0;
    h.K = g.K / n; h.sA = h.K; h.sB = g.kseg ? g.segB : g.transB ? h.K : (int64_t)h.K * g.ldb;
    h.bias = h.resid = nullptr; h.ldr = 0; h.sBias = 0;
    h.C = g.ws; h.ldc = g.N; h.sC = (int64_t)g.M * g.N;
    h.batch = n; h.c_f32_accum = 1; h.c_overwrite = 1;
    const double t = gemm_mfma_us(h) + LAUNCH + (double)g.M * g.N * (4 * n + (g.resid ? 4 : 2)) / 4.5e6;
    if (t < us && gemm_mfma_takes(dt, h)) { us = t; best = h; }
  }
  return best.batch > 1;
}

// C = p[0] + p[1] + .. in this order (+ bias, + residual R), rounded: 8 columns per thread.
template <typename E, int n>
__global__ __launch_bounds__(256) void add_parts_kernel(int64_t nvec, int vec_per_row, const float* __restrict__ p, int64_t part, E* C,
                                                        int64_t ldc, const E* __restrict__ bias, const E* R, int64_t ldr) {
  typedef typename Vec<E>::type E8;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= nvec) return;
  const int64_t row = i / vec_per_row, col = (i % vec_per_row) * 8;
  f32x4 v[n][2];
  E8 bb = {}, rr = {};
  if (bias) bb = *reinterpret_cast<const E8*>(bias + col);
  if (R) rr = *reinterpret_cast<const E8*>(R + row * ldr + col);
#pragma unroll
  for (int z = 0; z < n; ++z) {
    const f32x4* a = reinterpret_cast<const f32x4*>(p + z * part + i * 8);
    v[z][0] = a[0];
    v[z][1] = a[1];
  }
#pragma unroll
  for (int z = 1; z < n; ++z) { v[0][0] += v[z][0]; v[0][1] += v[z][1]; }
  E8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    float x = v[0][e / 4][e & 3];
    if (bias) x += (float)bb[e];
    if (R) x += (float)rr[e];
    o[e] = (E)x;
  }
  *reinterpret_cast<E8*>(C + row * ldc + col) = o;
}
template <typename E> hipError_t add_parts(hipStream_t st, const Gemm& g, int n) {
  const int64_t nvec = (int64_t)g.M * g.N / 8;
  auto kern = n == 2 ? add_parts_kernel<E, 2> : add_parts_kernel<E, 3>;
  hipLaunchKernelGGL(kern, dim3((unsigned)cdiv(nvec, 256)), dim3(256), 0, st, nvec, g.N / 8, (const float*)g.ws, (int64_t)g.M * g.N, (E*)g.C, g.ldc, (const E*)g.bias, (const E*)g.resid, g.ldr);
  return hipGetLastError();
}
}  // namespace

int gemm_mfma_parts(DType dt, const Gemm& g) {
  Gemm h;
  return plan_parts(dt, g, h) ? h.batch : 1;
}

int64_t gemm_mfma_ws_bytes(const Gemm& g) {
  KCut k;
  return (!g_force_tile && plan_kcut(BF16, g, k)) ? k.ws_need : 0;
}

hipError_t gemm_mfma(hipStream_t st, DType dt, const Gemm& g) {
  const int tile = gemm_mfma_pick_tile(g);
  if (g.ws && !g_force_tile) {
    KCut k;
    if (plan_kcut(dt, g, k) && k.ws_need <= g.ws_bytes && ((uintptr_t)g.ws & 15) == 0 && gemm_mfma_takes(dt, g)) {
      hipError_t e = run_tile(st, dt, k.head, 1);
      if (e != hipSuccess) return e;
      e = run_tile(st, dt, k.tail, 1);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(add_partials_kernel, dim3((unsigned)(k.rem * 4)), dim3(256), 0, st, (float*)g.C, g.ldc, g.sC, g.M, g.N,
                         (int)cdiv(g.M, 256), (int)cdiv(g.N, 256), k.tail.tile_base, k.tail.tile_count, (const float*)g.ws,
                         k.tail.nchunks - 1);
      return hipGetLastError();
    }
  }
  Gemm parts;
  if (plan_parts(dt, g, parts)) {
    const hipError_t e = run_tile(st, dt, parts, gemm_mfma_pick_tile(parts));
    return e != hipSuccess ? e : dt == F16 ? add_parts<f16>(st, g, parts.batch) : add_parts<bf16>(st, g, parts.batch);
  }
  if (!g_force_tile) {
    Gemm head, tail, h, t;
    double us = tile_us(g, tile);
    int wide = 0;
    for (int w : {1, 3}) {
      if (w == 3 && !gemm_mfma_oblong(g)) continue;
      if (!split_tail(dt, g, w, h, t)) continue;
      const double cut = (tile_us(h, w) + gemm_mfma_us(t) + 1.0) * 1.03;   // cuts come out 3 % above their estimate
      if (cut < us) { us = cut; wide = w; head = h; tail = t; }
    }
    if (wide) {
      const hipError_t e = run_tile(st, dt, head, wide);
      return e != hipSuccess ? e : run_tile(st, dt, tail, gemm_mfma_pick_tile(tail));
    }
  }
  return run_tile(st, dt, g, tile);
}

}  // namespace zs

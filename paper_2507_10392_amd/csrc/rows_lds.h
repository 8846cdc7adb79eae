// k-contiguous operands of the small products' kernels (gemm_f32.hip, gemm_small.hip), brought in through LDS.
//
// Read straight into fragments, neighbouring lanes of a load lie in different rows, and the address unit takes their 16-byte pieces one
// by one, four times as long as whole lines.  So a wave loads two slabs at a time, 128 bytes of each row and 8 rows a load, puts
// them into LDS that no other wave touches (no barrier, only wave_lds_order), the 16-byte piece p of row r at
// position p ^ r % 8, which spreads both the stores and the fragment reads over the banks, and reads the fragments back.  A slab is 64
// bytes of k: 16 fp32 or 32 16-bit values.
#pragma once
#include "common.h"

namespace zs {

template <int NB> struct Rows { u32x4 v[2 * NB]; };   // NB blocks of 16 rows, two slabs
// at: byte offset of the lane's piece (lane % 8) of its first row (lane / 8), or past every descriptor; ld: bytes between rows
template <int NB> __device__ __forceinline__ void load_rows(Rows<NB>& f, __amdgpu_buffer_rsrc_t rs, unsigned at, unsigned ld, unsigned soff) {
#pragma unroll
  for (int i = 0; i < 2 * NB; ++i) f.v[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)at, (int)(soff + 8 * i * ld), 0);
}
// wave_lds_order() belongs between put_rows and get_rows, and between get_rows and the next put_rows.
template <int NB> __device__ __forceinline__ void put_rows(const Rows<NB>& f, u32x4* lds, int lane) {
  u32x4* p = lds + (lane & ~7) + ((lane & 7) ^ (lane >> 3));
#pragma unroll
  for (int i = 0; i < 2 * NB; ++i) p[64 * i] = f.v[i];
}
// Both in one, for the first SLABS of the two slabs, one block of 16 rows after the other: a block's reads run beside the next one's writes.
template <int NB, int SLABS, typename V> __device__ __forceinline__ void turn_rows(V (&v)[SLABS][NB], const Rows<NB>& f, u32x4* lds, int lane) {
  u32x4* p = lds + (lane & ~7) + ((lane & 7) ^ (lane >> 3));
  const u32x4* r = lds + (lane & 15) * 8;
  wave_lds_order();   // what was here has been read
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    p[128 * b] = f.v[2 * b];
    p[128 * b + 64] = f.v[2 * b + 1];
    wave_lds_order();
#pragma unroll
    for (int h = 0; h < SLABS; ++h) v[h][b] = __builtin_bit_cast(V, r[128 * b + ((4 * h + (lane >> 4)) ^ (lane & 7))]);
  }
}
// Fragments of one of the two slabs: lane l gets piece l / 16 of row l % 16 of every block.
template <int NB, typename V> __device__ __forceinline__ void get_rows(V (&v)[NB], const u32x4* lds, int slab, int lane) {
  const u32x4* p = lds + (lane & 15) * 8 + ((4 * slab + (lane >> 4)) ^ (lane & 7));
#pragma unroll
  for (int b = 0; b < NB; ++b) v[b] = __builtin_bit_cast(V, p[128 * b]);
}

}  // namespace zs

// Device helpers shared by the FP8 GEMM kernels.
#pragma once

#include "kernels.h"

namespace qe {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
// Output vectors at element alignment: global accesses are the same single
// instructions at any address (unaligned access is the device's normal mode),
// so rows of odd strides are written like aligned ones.
typedef float v4f_out __attribute__((ext_vector_type(4), aligned(4)));
typedef int v2i_out __attribute__((ext_vector_type(2), aligned(2)));

constexpr int BK = 128;
// Tiles are numbered down groups of kGroupM row tiles, column after column,
// and each XCD takes a contiguous range of that order, so a round's 32 tiles
// on one XCD are 4 row tiles x 8 column tiles sharing their operand slabs in
// its L2.  Measured on MI355X over the Llama-3-70B stage's twelve products:
// 4 rows 1.2% faster than 8 (two runs), 2 rows 1.8% slower, 16 rows 5%
// slower; the 8B stage's products are level between 4, 6 and 8.
constexpr int kGroupM = 4;


// Cache policy of the epilogue's output traffic (stores, and the destination
// reads of the accumulate mode): non-temporal.  The output is written once
// and not read again by this kernel, so keeping it out of the L2 leaves the L2
// to the operand rows and columns that later tiles of the grid re-read;
// measured on MI355X over the Llama-3-8B stage's twelve products: -3.7% time
// with FP32 / BF16 stores, -5% in accumulate mode, most on the seven-round
// shapes.
constexpr int kNT = 2;  // the buffer instructions' nt bit

// LDS rows of a K tile are 128 bytes; 16-byte chunk c of row r is stored at
// chunk c ^ row_swizzle(r).  ds_read_b128 serves 16 lanes at a time, and not
// consecutive ones: lanes 0-3, 12-15, 20-23, 24-27 together, then 4-7, 8-11,
// 16-19, 28-31, and the same again 32 lanes up (256 bytes of 64 banks).  A
// fragment read (lane l: row l & 15, chunk 2 (l >> 4) or the next) therefore
// meets every row of 16 once per group, half of them one chunk pair further,
// and row bits 1, 2, 3 -> 1, 4, 6 put those 16 chunks into 16 different bank
// quads.  Measured on MI355X (one wave, dependent reads): 71.0 cycles a read,
// as for a linear 1 KB read (70.7); r >> 1 in its place 74.7, no swizzle 82.7.
__device__ __forceinline__ int row_swizzle(int r) { return ((r >> 1) & 1) ^ (((r >> 2) & 1) * 4) ^ (((r >> 3) & 1) * 6); }

// Offset of 16-byte chunk `chunk` of operand row `row` in the first K tile.  A
// reduction shorter than that tile has no chunks past the row's last one: they
// fall back to it, so that loads of whole tiles issued for their place in the
// pipeline only (the large tiles issue them past the last full K tile, from the
// first one) read no byte past the operand, whatever its row stride.
__host__ __device__ inline uint32_t chunk_offset(int64_t row, int64_t ld, int chunk, int64_t k) {
  const int last = k >= BK ? BK / 16 - 1 : (k > 0 ? int(k - 1) / 16 : 0);
  return uint32_t(row * ld) + uint32_t(chunk < last ? chunk : last) * 16u;
}

__device__ __forceinline__ uint4 mask_tail(uint4 v, int64_t valid) {
  // keep bytes [0, valid), zero the rest; branch-free
  uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int64_t nb = valid - 4 * q;  // bytes of this dword to keep
    const int k = nb <= 0 ? 0 : (nb >= 4 ? 4 : int(nb));
    w[q] &= uint32_t((uint64_t(1) << (8 * k)) - 1u);
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// Two floats to two bf16 (round to nearest even, NaN stays a quiet NaN with
// its sign and top payload bits) with the gfx950 packed conversion; bit-equal
// to the integer form (u + 0x7fff + ((u >> 16) & 1)) >> 16 on every input,
// which was checked on MI355X over all exponents, boundaries, denormals and NaNs.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf16x2_bits(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{lo, hi}, bf16x2_t));
}
__device__ __forceinline__ uint16_t bf16_bits(float f) { return uint16_t(bf16x2_bits(f, 0.0f)); }

__device__ __forceinline__ int pow2_exponent(const float *p) { return int((__float_as_uint(*p) >> 23) & 0xffu) - 127; }

// Workgroups are dealt to the 8 XCDs round-robin; renumber so that each XCD
// gets a contiguous range of tiles (shared A rows / B columns stay in one L2).
__device__ __forceinline__ int xcd_remap(int wg, int total) {
  const int per = total / 8, rem = total % 8;
  const int xcd = wg % 8, idx = wg / 8;
  return xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
}

}  // namespace

// Destinations whose rows are vector-aligned (BF16: 8 bytes, FP32: 16 bytes per
// lane): the branch-free epilogue of the large tiles takes only these.
inline int gemm_vec_ok(const GemmParams &g) {
  const uintptr_t cp = reinterpret_cast<uintptr_t>(g.c);
  return g.ldc % 4 == 0 && cp % (g.out == 1 ? 8 : 16) == 0 ? 1 : 0;
}

}  // namespace qe

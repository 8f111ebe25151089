// The product X X^T on the binary16 matrix cores, to fp32 accuracy: device
// building blocks shared by the K build and the on-the-fly sweep.
//
// Point i is scaled by a power of two s_i that brings its largest coordinate
// into [2^14, 2^15) (exact) and each coordinate is taken as two binary16
// values, hi = its rounding and lo = the rest rounded.  hi + lo is the fp32
// value itself for three coordinates of four and one unit in the last place
// off otherwise (a coordinate below 2^-25 of the row's largest is held to
// 2^-39 of it).  Then
//   s_i s_j x_i . x_j = sum_t hi hi + hi lo + lo hi   (+ lo lo, below 2^-22 of a product)
// with exact products and fp32 sums: three v_mfma_f32_32x32x16_f16 take 16
// coordinates, in the time of 1.5 v_mfma_f32_32x32x2_f32 (2 coordinates
// each), and round the sum 3 times per 16 coordinates instead of 8 times.
//
// The split points are kept in operand order: for each block of 32 points
// and each chunk of 16 coordinates one 1 KB unit of hi and one of lo, a unit
// being the 64 lanes' 16-byte operands (lane (l, h) = lane % 32, lane / 32
// holds point l of the block at coordinates 8h .. 8h + 7 of the chunk).  A
// unit is one wavefront's load, from global memory to LDS or to registers,
// without bank conflicts or address arithmetic per row.
#pragma once
#include "tile_mma.h"

namespace kkm {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));

constexpr int kUnit = 512;  // binary16 values in a unit

// unit (block of 32 points, chunk of 16 coordinates, part): part 0 = hi, 1 = lo
__host__ __device__ inline int64_t split_unit(int64_t blk, int nch, int c, int part) {
  return (blk * nch + c) * 2 + part;
}

// acc += A B^T of one chunk, for 2 x 2 blocks of 32 x 32 (hi in part 0).
__device__ inline void split_mfma(const half8 (&a)[2][2], const half8 (&b)[2][2], floatx16 (&acc)[2][2]) {
  // a block's three products are four instructions apart, so none waits for
  // the one before it
#pragma unroll
  for (int p = 0; p < 3; ++p)
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int bj = 0; bj < 2; ++bj)
        acc[bi][bj] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[bi][p == 2], b[bj][p == 1], acc[bi][bj], 0, 0, 0);
}

}  // namespace kkm

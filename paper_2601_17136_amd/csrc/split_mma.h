// The product X X^T on the binary16 matrix cores, to fp32 accuracy: device
// building blocks shared by the K build and the on-the-fly sweep.
//
// Point i is scaled by a power of two s_i that brings its largest coordinate
// into [2^14, 2^15) (exact) and each coordinate is taken as two binary16
// values, hi = its rounding and lo = the rest rounded.  hi + lo is the fp32
// value itself for three coordinates of four and one unit in the last place
// off otherwise, down to 2^-15 of the row's largest; from there on a coordinate
// is held to 2^-39 of the largest (points with many of those keep the fp32
// products: split_runs).  Then
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

#include <type_traits>

namespace kkm {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));

constexpr int kUnit = 512;  // binary16 values in a unit

// unit (block of 32 points, chunk of 16 coordinates, part): part 0 = hi, 1 = lo
__host__ __device__ inline int64_t split_unit(int64_t blk, int nch, int c, int part) {
  return (blk * nch + c) * 2 + part;
}

// The matrix instruction's sum is not rounded without bias, which the sums of K
// over a cluster, and the objective's differences of them, would show.  Part of
// it goes down (towards minus infinity, in sums of either sign): about 0.6e-9 +
// 2.6e-11 d of a sum of positive products over d coordinates.  So the last part
// of the chunks is added to the negated sum, with the rows' operands negated:
// there the same rounding goes the other way; a sum of positive products grows
// with the chunks, and the two parts cancel when the first has 1/sqrt(2) of
// them.  Another part makes such a sum smaller whichever its sign, by 1.4e-9 at
// d = 25 .. 784, so the turn comes 1.6 chunks earlier, which leaves that much
// upwards.  Mean error of the entries between points of uniform coordinates, at
// a turn that balances the first part alone / here: -1.1e-9 / -0.2e-9 at d = 25,
// -2.4e-9 / -0.5e-9 at 54, -2.3e-9 / -0.2e-9 at 100, -0.6e-9 / 0.3e-9 at 301,
// 1.2e-9 / 2.7e-9 at 784; the objective's error on image-like points falls from
// 1.2e-8 .. 9.9e-8 to 0.1e-8 .. 8.5e-8 (half of it or less at most widths).  The
// result is the negated product.  nch >= 2.
__device__ inline int split_turn(int nch) { return (nch * 45 - 72) >> 6; }
__device__ inline void split_negate(floatx16 (&acc)[2][2]) {
#pragma unroll
  for (int bi = 0; bi < 2; ++bi)
#pragma unroll
    for (int bj = 0; bj < 2; ++bj) acc[bi][bj] = -acc[bi][bj];
}
// One lane's 8 coordinates v, scaled by sc, as hi at u and lo one unit further.
__device__ inline void split_store(const float (&v)[8], float sc, half_t* u) {
  half8 hi, lo;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float x = v[e] * sc;
    hi[e] = (half_t)x;
    lo[e] = (half_t)(x - (float)hi[e]);
  }
  *(half8*)u = hi;
  *(half8*)(u + kUnit) = lo;
}

// acc += A B^T of one chunk, for 2 x 2 blocks of 32 x 32 (hi in part 0).  SWAP:
// lo hi before hi lo, so that entry (j, i) adds the products in (i, j)'s order.
template <bool SWAP = false>
__device__ inline void split_mfma(const half8 (&a)[2][2], const half8 (&b)[2][2], floatx16 (&acc)[2][2]) {
  // a block's three products are four instructions apart, so none waits for
  // the one before it
#pragma unroll
  for (int p = 0; p < 3; ++p)
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int bj = 0; bj < 2; ++bj)
        acc[bi][bj] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[bi][p == (SWAP ? 1 : 2)], b[bj][p == (SWAP ? 2 : 1)], acc[bi][bj], 0, 0, 0);
}

typedef __attribute__((address_space(1))) const void gvoid;
typedef __attribute__((address_space(3))) void lvoid;

constexpr int kSplitLds = 2 * 16 * 1024;  // split_tile's LDS: two chunks of 16 units

// The wavefront's 64 x 64 quarter (wm = wave / 2, wn = wave % 2) of the tile
// whose 128 rows start at block rb and whose columns start at block cb of the
// split points, negated (split_turn), laid out as mma_tile's.  256 threads.  A chunk's units (4 row
// and 4 column blocks, hi and lo) go from global memory straight to LDS, double
// buffered: chunk c + 1 is requested once chunk c's operands are in registers
// and arrives during its products; one barrier per chunk and one at the end.
template <bool SWAP = false>
__device__ inline void split_tile(const half_t* __restrict__ Xf, int nch, int64_t rb, int64_t cb, char* lds, int wave,
                                  int lane, floatx16 (&acc)[2][2]) {
  constexpr int kPer = 4;  // units per wavefront: unit u = 4 wave + v is part u % 2 of block u / 2
  const int wm = wave >> 1, wn = wave & 1;
  const half_t* src[kPer];
#pragma unroll
  for (int v = 0; v < kPer; ++v) {
    const int u = wave * kPer + v, blk = u >> 1;
    src[v] = Xf + split_unit(blk < 4 ? rb + blk : cb + (blk - 4), nch, 0, u & 1) * kUnit + lane * 8;
  }
  auto fetch = [&](int c) {
    char* dst = lds + (c & 1) * (kSplitLds / 2) + wave * (kPer * 1024);
#pragma unroll
    for (int v = 0; v < kPer; ++v)
      __builtin_amdgcn_global_load_lds((gvoid*)(src[v] + (int64_t)c * (2 * kUnit)), (lvoid*)(dst + v * 1024), 16, 0, 0);
  };
  fetch(0);
#pragma unroll
  for (int bi = 0; bi < 2; ++bi)
#pragma unroll
    for (int bj = 0; bj < 2; ++bj)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[bi][bj][r] = 0.f;
  auto step = [&](int c, auto negated) {
    // chunk c has arrived (this wavefront's units; the barrier: everyone's),
    // and everyone has read chunk c - 1, whose buffer chunk c + 1 takes
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    __syncthreads();
    const char* st = lds + (c & 1) * (kSplitLds / 2) + lane * 16;
    half8 a[2][2], b[2][2];
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int p = 0; p < 2; ++p) a[bi][p] = *(const half8*)(st + ((wm * 2 + bi) * 2 + p) * 1024);
#pragma unroll
    for (int bj = 0; bj < 2; ++bj)
#pragma unroll
      for (int p = 0; p < 2; ++p) b[bj][p] = *(const half8*)(st + ((4 + wn * 2 + bj) * 2 + p) * 1024);
    __builtin_amdgcn_sched_barrier(0);
    if (c + 1 < nch) fetch(c + 1);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (negated) {
#pragma unroll
      for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int p = 0; p < 2; ++p) a[bi][p] = -a[bi][p];
    }
    split_mfma<SWAP>(a, b, acc);
  };
  const int turn = split_turn(nch);
  int c = 0;
  for (; c < turn; ++c) step(c, std::false_type{});
  split_negate(acc);
  for (; c < nch; ++c) step(c, std::true_type{});
  __syncthreads();
}

// kappa from acc = -s_i s_j x_i . x_j: si = -1/s_i; cj = 1/s_j times -2c
// (Gaussian, c = -gamma log2 e), gamma (polynomial) or 1 (linear), a product
// with a power of two and so exact; u = c(|x_i|^2 + |x_j|^2).
// DEG: the polynomial's degree, or 0 for any (a loop per entry).
template <int KIND, int DEG>
__device__ inline float kappa_split(float acc, float si, float cj, float u, const KappaParams& kp) {
  const float b = acc * si;
  if (KIND == GAUSS) return __builtin_amdgcn_exp2f(fminf(fmaf(b, cj, u), 0.f));
  if (KIND == LINEAR) return b * cj;
  float t = fmaf(b, cj, kp.coef0), v = 1.f;
  if (DEG == 2) return t * t;
  for (int e = kp.degree; e > 0; e >>= 1) {
    if (e & 1) v *= t;
    t *= t;
  }
  return v;
}

// The pass over a tile's entries in its versions, the one that applies:
// pass(integral_constant<P>) with P = 0 in general, 1 for the Gaussian with
// the fix-up estimate, 2 for the polynomial of degree 2 (the paper's kernel:
// the general loop costs a few scalar branches per entry).
template <int KIND, typename F>
__device__ inline void kappa_pass(bool est, const KappaParams& kp, F&& pass) {
  if (KIND == GAUSS && est) pass(std::integral_constant<int, 1>{});
  else if (KIND == POLY && kp.degree == 2) pass(std::integral_constant<int, 2>{});
  else pass(std::integral_constant<int, 0>{});
}

template <int KIND>
__device__ inline float col_factor(float inv, const KappaParams& kp) {
  return KIND == GAUSS ? inv * kp.m2c : KIND == POLY ? inv * kp.gamma : inv;
}

}  // namespace kkm

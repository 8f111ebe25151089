// K = kappa(X X^T) with the product on the binary16 matrix cores (split_mma.h):
// the K build from kSplitMinDpad coordinates up wherever the split points are
// held (kkm_capi.cpp), all storages, panels and blocks.  gemm_kappa.hip keeps
// the build on the fp32 matrix cores, for fewer coordinates, for points that
// split_runs turns down and for memory budgets without room for the split
// points.
//
// Tiles, layouts and epilogue are those of gemm_kappa.hip: the upper block
// triangle of 128 x 128 tiles (I <= J), an entry's accumulator register and
// lane as there (both matrix instructions hold a 32 x 32 block alike).  Entries
// (i, j) and (j, i) would add hi lo and lo hi in different orders: on a diagonal
// tile the one with i <= j is stored in both places, and a panel's tiles below
// the diagonal add them in the other order (split_mfma).  So K is exactly
// symmetric, and a panel or block holds the bits of the full K.
#include "split_mma.h"

#include <algorithm>
#include <type_traits>

namespace kkm {

namespace {

// Height of a band of tiles (Bands): the ~100 workgroups an XCD runs at once
// cover a band's rows by a dozen columns, and their chunks meet in its L2.
constexpr int kBand = 8;

// What a build's epilogue writes and where.
template <typename KT>
struct BuildOut {
  KT* K;
  const float* kw;  // binary16 row scales or null
  float* diagK;
  int2* fix_list;
  unsigned long long* fix_count;
  long long seg_cap;
  int64_t n, ld;
  int packed;
  int64_t r0, r1, c0, c1;  // panel: rows and columns of the block
};

// Lists the Gaussian entries marked in mk (bit 31 - 2r - bj of mk[bi]: entry r
// of the 32 x 32 block (bi, bj)) for recomputation: the square layouts each
// pair once (i < j), a panel every entry it stores off the diagonal (on a
// diagonal tile (i, j) and (j, i) as (i, j), i < j, is marked).  A scan of the
// lanes' counts and one atomic per wavefront give the slots.
template <typename KT, bool PANEL>
__device__ inline void list_fixups(unsigned (&mk)[2], int64_t gi0, int64_t gj0, bool diagonal, bool inside,
                                   const BuildOut<KT>& o) {
  const bool both = PANEL && diagonal;
  auto stored = [&](int64_t gi, int64_t gj) { return gi < o.r1 && gj < o.c1; };
  const int lane = threadIdx.x & 63, l32 = lane & 31, h = lane >> 5;
  const int seg = (int)(blockIdx.x % kFixSegs);
  auto entry = [&](int bi, int bit, int64_t& gi, int64_t& gj) {
    const int g = 31 - bit, r = g >> 1;
    gi = gi0 + bi * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
    gj = gj0 + (g & 1) * 32 + l32;
  };
  unsigned cnt = 0;
#pragma unroll
  for (int bi = 0; bi < 2; ++bi) {
    if (!inside)  // a diagonal or last tile: drop what is not listed
      for (unsigned m = mk[bi]; m; m &= m - 1u) {
        int64_t gi, gj;
        entry(bi, __ffs(m) - 1, gi, gj);
        if (!(both ? gi < gj : PANEL ? stored(gi, gj) : gi < gj && gj < o.n)) mk[bi] &= ~(m & -m);
        else if (both) cnt += (stored(gi, gj) ? 1u : 0u) + (stored(gj, gi) ? 1u : 0u);
      }
    if (!both) cnt += (unsigned)__popc(mk[bi]);
  }
  unsigned pre = cnt;  // inclusive scan over the lanes
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const unsigned v = __shfl_up(pre, d, 64);
    if (lane >= d) pre += v;
  }
  const unsigned total = __shfl(pre, 63, 64);
  unsigned long long base = 0;
  if (lane == 0 && total) base = atomicAdd(o.fix_count + seg, (unsigned long long)total);
  base = __shfl(base, 0, 64) + (pre - cnt);
#pragma unroll
  for (int bi = 0; bi < 2; ++bi)
    for (unsigned m = mk[bi]; m; m &= m - 1u) {
      int64_t gi, gj;
      entry(bi, __ffs(m) - 1, gi, gj);
      auto put = [&](int64_t i, int64_t j) {
        if (base < (unsigned long long)o.seg_cap)
          o.fix_list[(int64_t)seg * o.seg_cap + (int64_t)base] = make_int2((int)i, (int)j);
        ++base;
      };
      if (!both || stored(gi, gj)) put(gi, gj);
      if (both && stored(gj, gi)) put(gj, gi);
    }
}

// One wavefront's part of tile (I, J): rows gi0 .. gi0 + 63, columns gj0 ..
// gj0 + 63.  rinv, rcn: the rows' -1/s and c|x|^2 (Gaussian) or |x|^2, in LDS;
// rw, cw: for binary16 storage, 1/kw of the rows and columns, in LDS (a load and
// a division per stored row took 20 us of a small build);
// cf, cnj: the columns' factor (col_factor) and c|x|^2.  est:
// Gaussian entries of the tile may need the fix-up.  Tw: 32 x 65 floats of LDS
// of the wavefront's own (mirror tiles and binary16 storage), ordered within
// the wavefront.
template <int KIND, typename KT, bool PANEL>
__device__ inline void build_epilogue(floatx16 (&acc)[2][2], const float* rinv, const float* rcn, const float* rw,
                                      const float* cw,
                                      const float (&cf)[2], const float (&cnj)[2], int64_t I, int64_t J,
                                      int64_t gi0, int64_t gj0, bool est, float* Tw, const KappaParams& kp,
                                      const BuildOut<KT>& o) {
  constexpr bool kHalf = sizeof(KT) == 2;
  const int lane = threadIdx.x & 63, l32 = lane & 31, h = lane >> 5;
  unsigned mk[2];  // the lane's entries whose estimate calls for the fix-up
  // (the two versions' common loads and sums are kept from being merged ahead
  // of the branch, where they would hold a register per entry)
  auto kpass = [&](auto e_) {
    constexpr int P = decltype(e_)::value;
    asm volatile("; version %0" ::"n"(P) : "memory");
#pragma unroll
    for (int bi = 0; bi < 2; ++bi) {
      // u = c|x_i|^2 + c|x_j|^2 rounds the same for (i, j) and (j, i) only
      // if the products are not fused into the sum
#pragma clang fp contract(off)
      mk[bi] = 0u;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float4 s4 = *(const float4*)(rinv + bi * 32 + 8 * q + 4 * h);
        float4 n4 = {0.f, 0.f, 0.f, 0.f};
        if (KIND == GAUSS) n4 = *(const float4*)(rcn + bi * 32 + 8 * q + 4 * h);
        const float si[4] = {s4.x, s4.y, s4.z, s4.w}, cn[4] = {n4.x, n4.y, n4.z, n4.w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int bj = 0; bj < 2; ++bj) {
            const float u = KIND == GAUSS ? cn[e] + cnj[bj] : 0.f;
            const float v = kappa_split<KIND, P == 2 ? 2 : 0>(acc[bi][bj][4 * q + e], si[e], cf[bj], u, kp);
            if (P == 1) mk[bi] = 2u * mk[bi] + (u * v < kp.fix_uthr ? 1u : 0u);
            acc[bi][bj][4 * q + e] = v;
          }
        __builtin_amdgcn_sched_barrier(0);  // the rows' factors are not read further ahead (registers)
      }
    }
  };
  kappa_pass<KIND>(est, kp, kpass);
  if (KIND == GAUSS && est) {
    unsigned any = 0u;
#pragma unroll
    for (int bi = 0; bi < 2; ++bi) any |= mk[bi];
    if (__ballot(any != 0u))
      list_fixups<KT, PANEL>(mk, gi0, gj0, I == J,
                                 I != J && (PANEL ? gi0 + 64 <= o.r1 && gj0 + 64 <= o.c1 : gj0 + 64 <= o.n), o);
  }

  // The rows of tile (I, J) lie at a fixed stride S in every layout (packed:
  // ld - 128 I), entry (i, j) at Kb + (i - gi0) S + (j - gj0).  Columns j <
  // clim hold entries, clim <= j < cend hold 0 (the padding of a row), j >=
  // cend lie past the row's end.  Non-temporal: K is not read again here.
  KT* Kb;
  int64_t S, rlim, clim, cend;
  if (PANEL) {
    Kb = o.K + (gi0 - o.r0) * o.ld + (gj0 - o.c0);
    S = o.ld;
    rlim = o.r1;
    clim = o.c1;
    cend = o.c0 + o.ld;
  } else {
    Kb = o.K + (o.packed ? packed_row(I * kTile, o.ld) + (gi0 - I * kTile) * (o.ld - I * kTile) : gi0 * o.ld) + gj0;
    S = o.packed ? o.ld - I * kTile : o.ld;
    rlim = o.n;
    clim = o.n;
    cend = o.ld;
  }
  if (I == J) {
    // a diagonal tile: diag K, and each pair from its entry with i <= j, stored
    // in both places
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int r = 0; r < 16; ++r)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj) {
          const int il = bi * 32 + 8 * (r >> 2) + 4 * h + (r & 3), jl = bj * 32 + l32;
          const int64_t gi = gi0 + il, gj = gj0 + jl;
          float v = acc[bi][bj][r];
          // exp(0), or kappa of the squared norm: a square's lo lo, which the
          // product leaves out, is never negative, so tr K would come out low (2^-25 of it)
          if (gi == gj) v = KIND == GAUSS ? 1.f : kappa<KIND>(rcn[il], 0.f, 0.f, kp);
          if (gi > gj) continue;
          if (PANEL) {
            if (gi == gj && gi < rlim && gj < clim) o.diagK[gi] = v;
            if (gi < rlim && gj < cend) Kb[il * S + jl] = (KT)(gj < clim ? v : 0.f);
            if (gi < gj && gj < rlim && gi < cend) Kb[(gj - gi0) * S + (gi - gj0)] = (KT)(gi < clim ? v : 0.f);
            continue;
          }
          if (gi >= rlim || gj >= cend) continue;
          if (gi == gj && gj < clim) o.diagK[gi] = v;
          if (gj >= clim) v = 0.f;
          const float wi = kHalf ? rw[il] : 1.f;
          Kb[il * S + jl] = (KT)(v * wi);
          if (gi < gj && gj < clim) {
            const float wj = kHalf ? cw[jl] : 1.f;
            Kb[(gj - gi0) * S + (gi - gj0)] = (KT)(v * wj);
          }
        }
    return;
  }
  const bool full = gi0 + 64 <= rlim && gj0 + 64 <= clim;
  if (!kHalf) {
    // fp32 goes straight from the matrix layout: each instruction writes rows
    // il and il + 4, 32 consecutive floats (128 bytes) each, at a uniform row
    // address plus one per-lane 32-bit offset (S < kMaxKStride)
    const unsigned lane_b = ((unsigned)(4 * h) * (unsigned)S + (unsigned)l32) * 4u;
    char* const Kc = (char*)Kb;
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int iu = bi * 32 + 8 * (r >> 2) + (r & 3);
        char* const rowp = Kc + (size_t)iu * (size_t)S * 4u;
        const float v0 = acc[bi][0][r], v1 = acc[bi][1][r];
        if (full) {
          __builtin_nontemporal_store(v0, (float*)(rowp + lane_b));
          __builtin_nontemporal_store(v1, (float*)(rowp + lane_b + 128u));
          continue;
        }
        if (gi0 + 4 * h + iu >= rlim) continue;
        const int64_t j0 = gj0 + l32, j1 = j0 + 32;
        if (j0 < cend) __builtin_nontemporal_store(j0 < clim ? v0 : 0.f, (float*)(rowp + lane_b));
        if (j1 < cend) __builtin_nontemporal_store(j1 < clim ? v1 : 0.f, (float*)(rowp + lane_b + 128u));
      }
  }
  auto ordered = [] {  // the wavefront's own LDS tile: what is written is read after it
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  if (kHalf) {
    // binary16 goes through the LDS tile, one row's 128 contiguous bytes per instruction
#pragma unroll
    for (int bi = 0; bi < 2; ++bi) {
#pragma unroll
      for (int bj = 0; bj < 2; ++bj)
#pragma unroll
        for (int r = 0; r < 16; ++r) Tw[(8 * (r >> 2) + 4 * h + (r & 3)) * 65 + bj * 32 + l32] = acc[bi][bj][r];
      ordered();
      const int64_t gj = gj0 + lane;
      const int nrows = (int)min<int64_t>(32, rlim - (gi0 + bi * 32));
      KT* dst = Kb + (int64_t)(bi * 32) * S + lane;
      auto put = [&](int rr) {
        __builtin_nontemporal_store((KT)((gj < clim ? Tw[rr * 65 + lane] : 0.f) * rw[bi * 32 + rr]), dst + rr * S);
      };
      if (gj < cend) {
        if (nrows >= 32) {
#pragma unroll
          for (int rr = 0; rr < 32; ++rr) put(rr);
        } else {
          for (int rr = 0; rr < nrows; ++rr) put(rr);
        }
      }
      ordered();
    }
  }
  if (!PANEL && !o.packed) {  // full storage: tile (J, I), rows j, columns i
#pragma unroll
    for (int bj = 0; bj < 2; ++bj) {
#pragma unroll
      for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int r = 0; r < 16; ++r) Tw[l32 * 65 + bi * 32 + 8 * (r >> 2) + 4 * h + (r & 3)] = acc[bi][bj][r];
      ordered();
      const int64_t gi = gi0 + lane;  // I < J, so gi < n
      const int64_t gj1 = gj0 + bj * 32;
      const int nrows = (int)min<int64_t>(32, o.n - gj1);
      KT* dst = o.K + gj1 * o.ld + gi;
      auto put = [&](int rr) {
        const float v = Tw[rr * 65 + lane];
        __builtin_nontemporal_store((KT)(kHalf ? v * cw[bj * 32 + rr] : v), dst + rr * o.ld);
      };
      if (nrows >= 32) {
#pragma unroll
        for (int rr = 0; rr < 32; ++rr) put(rr);
      } else {
        for (int rr = 0; rr < nrows; ++rr) put(rr);
      }
      ordered();
    }
  }
}

// The tiles of a launch: bands of kBand row tiles by their columns, column by
// column.  Square layouts: a band starts at the column of its first row, and
// the few tiles left of a row's diagonal tile do nothing.
struct Bands {
  int64_t rows, cols;  // row and column tiles
  bool square;
  __host__ __device__ int64_t before(int64_t band) const {  // tiles in earlier bands
    return kBand * (band * cols - (square ? kBand * (band * (band - 1) / 2) : 0));
  }
  __host__ __device__ int64_t nbands() const { return (rows + kBand - 1) / kBand; }
  __host__ __device__ int64_t height(int64_t band) const {
    const int64_t p = rows - band * kBand;
    return p < kBand ? p : kBand;
  }
  __host__ __device__ int64_t first_col(int64_t band) const { return square ? band * kBand : 0; }
  __host__ __device__ int64_t total() const {
    const int64_t b = nbands() - 1;
    return before(b) + height(b) * (cols - first_col(b));
  }
  // tile t: row tile m, column tile j
  __device__ void tile(int64_t t, int64_t& m, int64_t& j) const {
    const int64_t last = nbands() - 1;
    int64_t band;
    if (square) {  // before(x) = t, for real x
      const double a = 0.5 * (double)(kBand * kBand), s = (double)(kBand * cols) + a;
      const double disc = s * s - 4.0 * a * (double)t;
      band = (int64_t)((s - sqrt(disc > 0.0 ? disc : 0.0)) / (2.0 * a));
      band = min(max(band, (int64_t)0), last);
      while (band < last && before(band + 1) <= t) ++band;
      while (band > 0 && before(band) > t) --band;
    } else {
      band = min(t / (kBand * cols), last);
    }
    const int64_t u = t - before(band), p = height(band);
    m = band * kBand + u % p;
    j = first_col(band) + u / p;
  }
};

}  // namespace

// Bound by the matrix cores (three binary16 products per fp32 one) at d of a
// few hundred, by its stores below.  Measured on packed K against the fp32
// matrix cores (gemm_kappa.hip): n = 20000, d = 784 2.78 -> 0.98 ms; n = 60000,
// d = 780 21.9 -> 8.5 ms (products at 1.0 PFLOP/s, where a library product of
// binary16 matrices runs at 1.4); n = 50000, d = 128 3.1 -> 1.55 ms; n = 5000, d
// = 300 91 -> 45 us; n = 120000, d = 54 9.0 -> 6.4 ms (4.5 TB/s of stores, which
// alone run at 5.3); binary16 storage, n = 40001, d = 301 4.3 -> 1.9 ms.
//
// Workgroup: a 128 x 128 tile, wavefront (wm, wn) its 64 x 64 quarter.  A
// chunk's units go from global memory straight to LDS, double buffered: chunk c
// + 1 is requested once chunk c's operands are in registers and arrives during
// its products; one barrier per chunk.  256 x 128 tiles (128 x 64 per
// wavefront) need a quarter less LDS traffic per product but leave two
// wavefronts per SIMD instead of three or four, and measured slower at every
// width: n = 60000, d = 128 2.29 ms against 2.06, n = 40000, d = 784 3.71
// against 3.63, n = 120000, d = 54 6.74 against 6.43.
template <int KIND, typename KT, bool PANEL>
__global__ __launch_bounds__(256, 3) void gemm_split_kernel(
    const half_t* __restrict__ Xf, const float* __restrict__ xinv, const float* __restrict__ nrm,
    const unsigned* __restrict__ maxnrm_bits, const float* __restrict__ bmax, int nch, Bands bands,
    int64_t T, KappaParams kp, BuildOut<KT> o) {
  constexpr int kTBytes = 4 * 32 * 65 * 4;
  __shared__ __attribute__((aligned(1024))) char lds[kSplitLds > kTBytes ? kSplitLds : kTBytes];
  __shared__ __attribute__((aligned(16))) float rinv[kTile], rcn[kTile];
  __shared__ float rw[sizeof(KT) == 2 ? kTile : 1], cw[sizeof(KT) == 2 ? kTile : 1];
  const float maxnrm = __uint_as_float(*maxnrm_bits);
  if (!split_runs<KIND, PANEL>(maxnrm_bits, kp)) return;  // gemm_kappa_kernel builds K then (uniform)

  // Workgroup b runs on XCD b % 8: each XCD takes a contiguous run of tiles.
  const int64_t b = blockIdx.x;
  const int64_t per = T >> 3, rem = T & 7, x = b & 7;
  const int64_t t = x * per + (x < rem ? x : rem) + (b >> 3);
  int64_t I, J;
  bands.tile(t, I, J);
  if (PANEL) {
    I += o.r0 / kTile;
    J += o.c0 / kTile;
  } else if (J < I) {
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31;
  const int64_t row0 = I * kTile, col0 = J * kTile;

  if (tid < kTile) {  // the rows' and columns' factors
    rinv[tid] = -xinv[row0 + tid];  // the product comes negated
    rcn[tid] = KIND == GAUSS ? kp.neg_g_log2e * nrm[row0 + tid] : nrm[row0 + tid];
  }
  if (sizeof(KT) == 2 && tid < kTile) {  // (a row past n is not stored)
    rw[tid] = o.kw && row0 + tid < o.n ? 1.f / o.kw[row0 + tid] : 1.f;
    cw[tid] = o.kw && col0 + tid < o.n ? 1.f / o.kw[col0 + tid] : 1.f;
  }
  float cf[2], cnj[2] = {0.f, 0.f};
#pragma unroll
  for (int bj = 0; bj < 2; ++bj) {
    const int64_t j = col0 + wn * 64 + bj * 32 + l32;
    cf[bj] = col_factor<KIND>(xinv[j], kp);
    if (KIND == GAUSS) cnj[bj] = kp.neg_g_log2e * nrm[j];
  }

  floatx16 acc[2][2];
  const int64_t gi0 = row0 + wm * 64, gj0 = col0 + wn * 64;
  // ends with a barrier: the buffers become LDS tiles
  if (PANEL && I > J) split_tile<true>(Xf, nch, row0 / 32, col0 / 32, lds, wave, lane, acc);
  else split_tile(Xf, nch, row0 / 32, col0 / 32, lds, wave, lane, acc);

  if (gi0 >= (PANEL ? o.r1 : o.n) || (I == J && gi0 > gj0)) return;  // nothing stored
  const bool est = KIND == GAUSS && (bmax ? gauss_needs_fix(1.f, bmax[I], bmax[J], kp)
                                          : gauss_needs_fix(1.f, maxnrm, maxnrm, kp));
  build_epilogue<KIND, KT, PANEL>(acc, rinv + wm * 64, rcn + wm * 64, rw + wm * 64, cw + wn * 64, cf, cnj, I, J, gi0,
                                      gj0, est,
                                      (float*)lds + wave * (32 * 65), kp, o);
}

namespace {

template <int KIND, typename KT, bool PANEL>
void launch_kind(const SplitPoints& sp, const float* nrm, const unsigned* maxnrm_bits, const float* bmax,
                 int64_t rows, int64_t cols, const KappaParams& kp, const BuildOut<KT>& o,
                 hipStream_t s) {
  const Bands bands{rows, cols, !PANEL};
  const int64_t T = bands.total();
  hipLaunchKernelGGL((gemm_split_kernel<KIND, KT, PANEL>), dim3((unsigned)T), dim3(256), 0, s, sp.Xf, sp.xinv, nrm,
                     maxnrm_bits, bmax, sp.nch, bands, T, kp, o);
}

template <typename KT, bool PANEL>
hipError_t launch_typed(const SplitPoints& sp, const float* nrm, const unsigned* maxnrm_bits, const float* bmax,
                        int64_t rows, int64_t cols, const KappaParams& kp, const BuildOut<KT>& o,
                        hipStream_t s) {
  switch (kp.kind) {
    case LINEAR: launch_kind<LINEAR, KT, PANEL>(sp, nrm, maxnrm_bits, bmax, rows, cols, kp, o, s); break;
    case POLY: launch_kind<POLY, KT, PANEL>(sp, nrm, maxnrm_bits, bmax, rows, cols, kp, o, s); break;
    default: launch_kind<GAUSS, KT, PANEL>(sp, nrm, maxnrm_bits, bmax, rows, cols, kp, o, s); break;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_split(const SplitPoints& sp, const float* nrm, const unsigned* maxnrm_bits, int64_t n,
                             int64_t ld, bool packed, bool f16, const float* kw, const KappaParams& kp, void* K,
                             float* diagK, int2* fix_list, unsigned long long* fix_count, long long seg_cap,
                             const float* bmax, hipStream_t s) {
  if (ld >= kMaxKStride) return hipErrorInvalidValue;
  const int64_t nt = (n + kTile - 1) / kTile;
  if (sp.rows < nt * kTile) return hipErrorInvalidValue;
  if (f16) {
    const BuildOut<half_t> o{(half_t*)K, kw, diagK, fix_list, fix_count, seg_cap, n, ld, packed, 0, n, 0, n};
    return launch_typed<half_t, false>(sp, nrm, maxnrm_bits, bmax, nt, nt, kp, o, s);
  }
  const BuildOut<float> o{(float*)K, kw, diagK, fix_list, fix_count, seg_cap, n, ld, packed, 0, n, 0, n};
  return launch_typed<float, false>(sp, nrm, maxnrm_bits, bmax, nt, nt, kp, o, s);
}

hipError_t launch_gemm_split_panel(const SplitPoints& sp, const float* nrm, const unsigned* maxnrm_bits, int64_t n,
                                   int64_t r0, int64_t r1, int64_t c0, int64_t c1, int64_t ld, const KappaParams& kp,
                                   float* K, float* diagK, int2* fix_list, unsigned long long* fix_count,
                                   long long seg_cap, hipStream_t s) {
  if (r0 % kTile || r1 <= r0 || r1 > n || c0 % kTile || c1 <= c0 || c1 > n || ld % kTile || ld < c1 - c0 ||
      ld >= kMaxKStride)
    return hipErrorInvalidValue;
  const int64_t nt = (n + kTile - 1) / kTile, rows = (r1 - r0 + kTile - 1) / kTile, cols = ld / kTile;
  if (sp.rows < nt * kTile || c0 / kTile + cols > nt) return hipErrorInvalidValue;
  const BuildOut<float> o{K, nullptr, diagK, fix_list, fix_count, seg_cap, n, ld, 0, r0, r1, c0, c1};
  return launch_typed<float, true>(sp, nrm, maxnrm_bits, nullptr, rows, cols, kp, o, s);
}

}  // namespace kkm

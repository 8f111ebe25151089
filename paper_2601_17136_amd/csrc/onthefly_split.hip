// The on-the-fly update (onthefly.hip) with the product on the binary16 matrix
// cores (split_mma.h), from kSplitMinDpad coordinates up.  Work items, tables,
// partials and reduction are onthefly.hip's; its sweeps on the fp32 matrix
// cores run beside this one and do nothing where this one does its work
// (split_runs), and alone where there is no room for the sorted split points.
#include "split_mma.h"

namespace kkm {

namespace {

// Whether the sweep reads the fp32 points: an entry may need the fix-up, or
// the fp32 sweeps run.
__device__ inline bool reads_fp32(const unsigned* maxnrm_bits, const KappaParams& kp) {
  const float m = __uint_as_float(*maxnrm_bits);
  if (kp.kind == GAUSS) return !split_runs<GAUSS, false>(maxnrm_bits, kp) || gauss_needs_fix(1.f, m, m, kp);
  return kp.kind == POLY ? !split_runs<POLY, false>(maxnrm_bits, kp) : !split_runs<LINEAR, false>(maxnrm_bits, kp);
}

}  // namespace

// The split points in sorted order (block b: sorted positions 32 b .. 32 b +
// 31, position p holds point perm[p]; zero past n), their 1/s, norms and
// clusters (-1 past n), and their fp32 coordinates where the sweep reads them.
__global__ __launch_bounds__(256) void gather_split_kernel(const float* __restrict__ Xp, const float* __restrict__ nrm,
                                                           const float* __restrict__ xinv,
                                                           const unsigned* __restrict__ maxnrm_bits,
                                                           const int* __restrict__ perm, const int* __restrict__ cl,
                                                           int64_t n, int d_pad, int k, KappaParams kp,
                                                           half_t* __restrict__ Xf, float* __restrict__ xinv_s,
                                                           float* __restrict__ Xs, float* __restrict__ nrm_s,
                                                           int* __restrict__ cs) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, l = lane & 31, h = lane >> 5;
  const int64_t p = (int64_t)blockIdx.x * 32 + l;
  const int64_t src = p < n ? (int64_t)perm[p] : -1;
  const float inv = src >= 0 ? xinv[src] : 1.f;
  if (w == 0 && h == 0) {
    const int c = src >= 0 ? cl[src] : -1;
    xinv_s[p] = inv;
    nrm_s[p] = src >= 0 ? nrm[src] : 0.f;
    cs[p] = src < 0 ? -1 : (c < 0 ? 0 : (c >= k ? k - 1 : c));
  }
  const bool fp32 = reads_fp32(maxnrm_bits, kp);
  const float sc = 1.f / inv;  // powers of two
  const int nch = (d_pad + 15) / 16;
  for (int c = w; c < nch; c += 4) {
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const int col = 16 * c + 8 * h;
    if (col < d_pad) {
      float4 x0 = {0.f, 0.f, 0.f, 0.f}, x1 = x0;
      if (src >= 0) {
        x0 = *(const float4*)(Xp + src * d_pad + col);
        x1 = *(const float4*)(Xp + src * d_pad + col + 4);
      }
      if (fp32) {
        *(float4*)(Xs + p * d_pad + col) = x0;
        *(float4*)(Xs + p * d_pad + col + 4) = x1;
      }
      v[0] = x0.x, v[1] = x0.y, v[2] = x0.z, v[3] = x0.w;
      v[4] = x1.x, v[5] = x1.y, v[6] = x1.z, v[7] = x1.w;
    }
    split_store(v, sc, Xf + split_unit(blockIdx.x, nch, c, 0) * kUnit + lane * 8);
  }
}

// One work item: row block I against the column tiles of a segment.
//
// NCH > 0 (NCH chunks, at most kRegMaxDpad coordinates): the block's operands
// stay in LDS for the whole sweep, each wavefront reads its 64 columns'
// straight into registers, and partials are kept per wavefront half, so the
// four wavefronts never wait for each other.  NCH = 0: both operands go
// through LDS per chunk (split_tile) and the wavefronts' sums meet there.
// Bound by the vector work on the tile's entries (kappa, row and column sums)
// at small widths, by the matrix cores beyond.  One sweep, against the fp32
// matrix cores: n = 60000, d = 54 Gaussian 2.11 -> 0.98 ms, polynomial 2.59 ->
// 0.78 ms; n = 16000, d = 784 1.89 -> 0.58 ms; n = 30000, d = 128 1.28 -> 0.49
// ms.  At NCH > 0 three wavefronts per SIMD (168 registers, some spilled)
// measured 12% slower than two, and reading the next tile's columns during
// this one's sums no faster.
template <int KIND, int NCH>
__global__ __launch_bounds__(256, 2) void onthefly_split_kernel(
    const half_t* __restrict__ Xf, const float* __restrict__ xinv_s, const float* __restrict__ Xs,
    const float* __restrict__ nrm_s, const int* __restrict__ cs, const unsigned* __restrict__ maxnrm_bits,
    const int* __restrict__ off, const int* __restrict__ cA, const int* __restrict__ nruns,
    const int64_t* __restrict__ cbase, const float* __restrict__ bmax, int64_t n, int d_pad, int64_t ld, int nt,
    int nseg, int k, KappaParams kp, float* __restrict__ Epart, float* __restrict__ Cpart) {
  constexpr bool kNarrow = NCH > 0;
  constexpr int kHalves = kNarrow ? 2 : 1;
  __shared__ __attribute__((aligned(1024))) char lds[kNarrow ? 4 * NCH * 2 * 1024 : kSplitLds];
  __shared__ __attribute__((aligned(16))) float rinv[kTile], rcn[kTile];
  const float maxnrm = __uint_as_float(*maxnrm_bits);
  if (!split_runs<KIND, false>(maxnrm_bits, kp)) return;  // the fp32 sweep runs
  int s = 0;
  int64_t first = 0;  // items before segment s
  while (s + 1 < nseg && first + otf_seg_begin(s + 1, nt, nseg) <= (int64_t)blockIdx.x) {
    first += otf_seg_begin(s + 1, nt, nseg);
    ++s;
  }
  const int I = (int)((int64_t)blockIdx.x - first);
  const int sb = otf_seg_begin(s, nt, nseg), se = otf_seg_begin(s + 1, nt, nseg);
  if (I >= se) return;
  const int jt0 = sb > I ? sb : I, jt1 = se;
  const int64_t row0 = (int64_t)I * kTile;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, l32 = lane & 31, h = lane >> 5;
  const int runA = cA[I], nr = nruns[I];
  const int nch = kNarrow ? NCH : (d_pad + 15) / 16;
  float* const cp = Cpart + cbase[I] * (kHalves * kTile);
  if (tid < kTile) {
    rinv[tid] = -xinv_s[row0 + tid];  // the product comes negated
    rcn[tid] = KIND == GAUSS ? kp.neg_g_log2e * nrm_s[row0 + tid] : 0.f;
  }
  if constexpr (kNarrow) {
    // the rows of the chunks from the turn on go to LDS negated (split_turn)
    const uint4* src = (const uint4*)(Xf + split_unit(row0 / 32, NCH, 0, 0) * kUnit);
    for (int f = tid; f < 4 * NCH * 2 * 64; f += 256) {
      const unsigned neg = f / 128 % NCH >= split_turn(NCH) ? 0x80008000u : 0u;
      uint4 x = src[f];
      x.x ^= neg, x.y ^= neg, x.z ^= neg, x.w ^= neg;
      ((uint4*)lds)[f] = x;
    }
  }
  __syncthreads();
  const bool fix = KIND == GAUSS && gauss_needs_fix(1.f, maxnrm, maxnrm, kp);

  float rowacc[2][16];
#pragma unroll
  for (int bi = 0; bi < 2; ++bi)
#pragma unroll
    for (int r = 0; r < 16; ++r) rowacc[bi][r] = 0.f;

  // Row side: the running sums reduced over the lanes (a fixed xor tree) and
  // written as cluster c's partial of segment s (kNarrow: half wn; else the
  // two halves added).
  auto flush = [&](int c) {
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float v = rowacc[bi][r];
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 8, 64);
        v += __shfl_xor(v, 4, 64);
        v += __shfl_xor(v, 2, 64);
        v += __shfl_xor(v, 1, 64);
        rowacc[bi][r] = v;
      }
    float* ep = Epart + (((int64_t)s * k + c) * kHalves + (kNarrow ? wn : 0)) * ld + row0;
    if constexpr (!kNarrow) {
      ep = (float*)lds + wn * kTile;  // free between tiles
      __syncthreads();
    }
    if (l32 == 0) {
      int rb = wm * 64 + 4 * h;
      asm volatile("" : "+v"(rb));
#pragma unroll
      for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int il = rb + bi * 32 + 8 * (r >> 2) + (r & 3);
          if (!kNarrow || row0 + il < n) ep[il] = rowacc[bi][r];
        }
    }
    if constexpr (!kNarrow) {
      __syncthreads();
      if (tid < kTile && row0 + tid < n)
        Epart[((int64_t)s * k + c) * ld + row0 + tid] = ((float*)lds)[tid] + ((float*)lds)[kTile + tid];
      __syncthreads();
    }
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int r = 0; r < 16; ++r) rowacc[bi][r] = 0.f;
  };

  // Column side of tile (I, J), J > I: column sums over the rows in sorted
  // positions [lo, hi), written as run u (kNarrow: half wm; else added).
  auto column_side = [&](int J, int u, bool all_rows, int lo, int hi, const floatx16 (&t)[2][2]) {
    float c0 = 0.f, c1 = 0.f;
    if (all_rows) {
#pragma unroll
      for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          c0 += t[bi][0][r];
          c1 += t[bi][1][r];
        }
    } else {
      int rb = wm * 64 + 4 * h - (lo - (int)row0);
      asm volatile("" : "+v"(rb));  // (see below)
      const unsigned len = (unsigned)(hi - lo);
#pragma unroll
      for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const bool in = (unsigned)(rb + bi * 32 + 8 * (r >> 2) + (r & 3)) < len;
          c0 += in ? t[bi][0][r] : 0.f;
          c1 += in ? t[bi][1][r] : 0.f;
        }
    }
    c0 += __shfl_xor(c0, 32, 64);
    c1 += __shfl_xor(c1, 32, 64);
    float* dst = cp + ((int64_t)(J - I - 1) * nr + u) * (kHalves * kTile);
    if constexpr (kNarrow) {
      if (h == 0) {
        dst[wm * kTile + wn * 64 + l32] = c0;
        dst[wm * kTile + wn * 64 + 32 + l32] = c1;
      }
    } else {
      float* csum = (float*)lds;  // [wm][128], free between tiles
      __syncthreads();
      if (h == 0) {
        csum[wm * kTile + wn * 64 + l32] = c0;
        csum[wm * kTile + wn * 64 + 32 + l32] = c1;
      }
      __syncthreads();
      if (tid < kTile) dst[tid] = csum[tid] + csum[kTile + tid];
    }
  };

  int cur = cs[(int64_t)jt0 * kTile];
  for (int J = jt0; J < jt1; ++J) {
    const int64_t col0 = (int64_t)J * kTile;
    // the columns' factors and clusters arrive during the products
    float ci[2], cnj[2] = {0.f, 0.f};
#pragma unroll
    for (int bj = 0; bj < 2; ++bj) {
      const int64_t j = col0 + wn * 64 + bj * 32 + l32;
      ci[bj] = xinv_s[j];
      if (KIND == GAUSS) cnj[bj] = nrm_s[j];
    }
    floatx16 acc[2][2];
    if constexpr (kNarrow) {
#pragma unroll
      for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[bi][bj][r] = split_turn(NCH) ? 0.f : -0.f;
      const half_t* bs = Xf + split_unit(col0 / 32 + wn * 2, NCH, 0, 0) * kUnit + lane * 8;
      const char* as = lds + (wm * 2 * NCH * 2) * 1024 + lane * 16;
      half8 b[2][2][2];
      auto fetch = [&](int c) {
#pragma unroll
        for (int bj = 0; bj < 2; ++bj)
#pragma unroll
          for (int p = 0; p < 2; ++p) b[c & 1][bj][p] = *(const half8*)(bs + ((bj * NCH + c) * 2 + p) * kUnit);
      };
      fetch(0);
#pragma unroll
      for (int c = 0; c < NCH; ++c) {
        if (c + 1 < NCH) fetch(c + 1);
        half8 a[2][2];
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
          for (int p = 0; p < 2; ++p) a[bi][p] = *(const half8*)(as + ((bi * NCH + c) * 2 + p) * 1024);
        if (c > 0 && c == split_turn(NCH)) split_negate(acc);
        split_mfma(a, b[c & 1], acc);
        __builtin_amdgcn_sched_barrier(0);  // operands are read one chunk ahead, not further (registers)
      }
    } else {
      split_tile(Xf, nch, row0 / 32, col0 / 32, lds, wave, lane, acc);
    }

    // kappa on the tile's entries
    const bool est = fix && gauss_needs_fix(1.f, bmax[I], bmax[J], kp);
    const bool inside = J > I && col0 + kTile <= n;
    float cf[2];
#pragma unroll
    for (int bj = 0; bj < 2; ++bj) {
      cf[bj] = col_factor<KIND>(ci[bj], kp);
      if (KIND == GAUSS) cnj[bj] *= kp.neg_g_log2e;
    }
    unsigned mk[2];  // entries whose estimate calls for the differences: bit 31 - 2r - bj of mk[bi]
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
          const int il = wm * 64 + bi * 32 + 8 * q + 4 * h;
          const float4 s4 = *(const float4*)(rinv + il);
          float4 n4 = {0.f, 0.f, 0.f, 0.f};
          if (KIND == GAUSS) n4 = *(const float4*)(rcn + il);
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
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    kappa_pass<KIND>(est, kp, kpass);
    if (!inside) {  // the diagonal tile, the last tile: entries outside n x n are 0, the Gaussian diagonal 1
      const int nrows = (int)(n - row0 < kTile ? n - row0 : kTile);
      const int ncols = (int)(n - col0 < kTile ? n - col0 : kTile);
      // the lane's row and column are made opaque in the rare paths, so that
      // their per-entry index work is formed there and not hoisted out of the
      // sweep, where it would hold registers
      int rb = wm * 64 + 4 * h, jb = wn * 64 + l32;
      asm volatile("" : "+v"(rb), "+v"(jb));
#pragma unroll
      for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
          for (int bj = 0; bj < 2; ++bj) {
            const int il = rb + bi * 32 + 8 * (r >> 2) + (r & 3), jl = jb + bj * 32;
            float v = acc[bi][bj][r];
            if (KIND == GAUSS && J == I && il == jl) v = 1.f;
            if (il >= nrows || jl >= ncols) v = 0.f;
            acc[bi][bj][r] = v;
          }
    }
    if (KIND == GAUSS && est && __ballot((mk[0] | mk[1]) != 0u)) {
      int rb = wm * 64 + 4 * h, jb = wn * 64 + l32;
      asm volatile("" : "+v"(rb), "+v"(jb));
#pragma unroll
      for (int bi = 0; bi < 2; ++bi)
        for (unsigned m = mk[bi]; m; m &= m - 1u) {
          const int g = 31 - (__ffs(m) - 1), r = g >> 1, bj = g & 1;
          const int il = rb + bi * 32 + 8 * (r >> 2) + (r & 3), jl = jb + bj * 32;
          if (row0 + il >= n || col0 + jl >= n || (J == I && il == jl)) continue;
          const float w = gauss_direct(Xs + (row0 + il) * d_pad, Xs + (col0 + jl) * d_pad, d_pad, kp);
#pragma unroll
          for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int rr = 0; rr < 16; ++rr)
              if (q == bj && rr == r) acc[bi][q][rr] = w;
        }
    }

    const int64_t last = (col0 + kTile - 1 < n) ? col0 + kTile - 1 : n - 1;
    const int cfst = cs[col0], clst = cs[last];
    if (cfst == cur && clst == cur) {
#pragma unroll
      for (int bi = 0; bi < 2; ++bi)
#pragma unroll
        for (int r = 0; r < 16; ++r) rowacc[bi][r] += acc[bi][0][r] + acc[bi][1][r];
    } else {
      // the clusters are walked over the whole tile's columns, so both halves
      // write a partial, possibly zero, for every cluster the segment holds
      const int64_t q0 = col0 + wn * 64 + l32, q1 = q0 + 32;
      const int c0 = q0 < n ? cs[q0] : -1, c1 = q1 < n ? cs[q1] : -1;
      for (int c = cfst; c <= clst; ++c) {
        if (c != cur) {
          flush(cur);
          cur = c;
        }
#pragma unroll
        for (int bi = 0; bi < 2; ++bi)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            rowacc[bi][r] += (c0 == c ? acc[bi][0][r] : 0.f) + (c1 == c ? acc[bi][1][r] : 0.f);
      }
    }
    if (J > I) {
      if (nr == 1) {
        column_side(J, 0, true, 0, 0, acc);
      } else {
        for (int u = 0; u < nr; ++u) column_side(J, u, false, off[runA + u], off[runA + u + 1], acc);
      }
    }
    if constexpr (!kNarrow) __syncthreads();  // the sums' LDS is the next tile's buffer
  }
  flush(cur);
}

hipError_t launch_gather_split(const float* Xp, const float* nrm, const float* xinv, const unsigned* maxnrm_bits,
                               const IterBufs& b, const int* cl, int64_t n_pad, int d_pad, const KappaParams& kp,
                               half_t* Xf, float* xinv_s, float* Xs, float* nrm_s, int* cs, hipStream_t s) {
  if (n_pad % 32 || d_pad % 8) return hipErrorInvalidValue;
  hipLaunchKernelGGL(gather_split_kernel, dim3((unsigned)(n_pad / 32)), dim3(256), 0, s, Xp, nrm, xinv, maxnrm_bits,
                     b.perm, cl, b.n, d_pad, b.k, kp, Xf, xinv_s, Xs, nrm_s, cs);
  return hipGetLastError();
}

hipError_t launch_onthefly_split(const half_t* Xf, const float* xinv_s, const float* Xs, const float* nrm_s,
                                 const int* cs, const unsigned* maxnrm_bits, const IterBufs& b, int d_pad,
                                 const KappaParams& kp, const OtfTables& tb, float* Epart, float* Cpart,
                                 hipStream_t s) {
  const int nt = (int)((b.n + kTile - 1) / kTile), nseg = onthefly_segments(b.n), nch = (d_pad + 15) / 16;
  if (d_pad < kSplitMinDpad) return hipErrorInvalidValue;
  const bool narrow = onthefly_halves(d_pad) == 2;  // the reduction's layout of the partials
  int64_t items = 0;
  for (int q = 0; q < nseg; ++q) items += otf_seg_begin(q + 1, nt, nseg);
#define KKM_OTF_SPLIT(KIND, NCH)                                                                                 \
  hipLaunchKernelGGL((onthefly_split_kernel<KIND, NCH>), dim3((unsigned)items), dim3(256), 0, s, Xf, xinv_s, Xs,   \
                     nrm_s, cs, maxnrm_bits, b.off, tb.cA, tb.nruns, tb.cbase, tb.bmax, b.n, d_pad, b.ld, nt, nseg, \
                     b.k, kp, Epart, Cpart)
#define KKM_OTF_SPLIT_KIND(KIND)                  \
  switch (narrow ? nch : 0) {                     \
    case 0: KKM_OTF_SPLIT(KIND, 0); break;        \
    case 2: KKM_OTF_SPLIT(KIND, 2); break;        \
    case 3: KKM_OTF_SPLIT(KIND, 3); break;        \
    case 4: KKM_OTF_SPLIT(KIND, 4); break;        \
    default: return hipErrorInvalidValue;         \
  }
  switch (kp.kind) {
    case LINEAR: KKM_OTF_SPLIT_KIND(LINEAR); break;
    case POLY: KKM_OTF_SPLIT_KIND(POLY); break;
    default: KKM_OTF_SPLIT_KIND(GAUSS); break;
  }
#undef KKM_OTF_SPLIT_KIND
#undef KKM_OTF_SPLIT
  return hipGetLastError();
}

}  // namespace kkm

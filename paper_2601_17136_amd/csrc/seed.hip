// K-means++ seeding in the kernel's feature space: D^2 sampling of the
// centers among the points (Arthur and Vassilvitskii), the initialization
// the paper cites for its convergence properties (Section II-B) and leaves
// to future work (Section V).
//
// With centers c_0 .. c_{t-1} chosen, D(i) = min_s ||phi(x_i) - phi(x_cs)||^2
// where ||phi(x) - phi(y)||^2 = K(x,x) - 2 K(x,y) + K(y,y) (the kernel trick
// of Section II-B).  Center t is the first index i with P(i) > u_t * S
// (P the prefix sums of D in index order, S = P(n-1)), so i is drawn with
// probability D(i)/S; the uniforms u_t come from the caller.
//
// The entries of K are computed from the staged points, whatever the K
// storage mode, and the three entries of a distance by the same routine, so
// a point that coincides with a center has distance exactly 0.  One pass per
// center updates D and the nearest center (lowest position on ties) of the
// points and writes their fp64 sums of D per block.  Up to kSeedFusedBlk blocks
// it is one launch: every workgroup first walks the prefix sums of D to the
// drawn index (the same index in each: a fixed order over the same values).  D
// and its sums alternate between two buffers, so that no workgroup overwrites
// what another still draws from.  The sums are then read once per workgroup, 8
// (n / 64)^2 bytes per center, so beyond that one workgroup draws in a launch of
// its own.  Nothing returns to the host between centers.
#include "kkm.h"
#include "tile_mma.h"

namespace kkm {

namespace {

constexpr int kSeedThr = 256;               // threads per workgroup
constexpr int kSeedLanes = 16;              // lanes per point
constexpr int kSeedPer = 4;                 // points per group of lanes, their loads in flight together
constexpr int kSeedPts = kSeedThr / kSeedLanes * kSeedPer;  // points per workgroup (one block of D)

// Microseconds per center, drawn in the pass / by a launch before it: 50000
// points 9.5 / 10.4 (d = 8), 33.4 / 35.0 (d = 784); 100000 points 11.4 / 10.6,
// 16.1 / 16.5 (d = 128), 62.0 / 63.0; 200000 points 18.7 / 12.7, 25.6 / 24.0;
// 1000000 points 225 / 33, 301 / 104.  The sums come once per workgroup, so the
// first grows with n^2.
constexpr int kSeedFusedBlk = 1600;

// The dot products x_i . x_c (or, for the Gaussian, |x_i - x_c|^2) of
// kSeedPer rows over d_pad floats, by a group of 16 lanes: lane l takes the
// 16-byte chunks l, l + 16, ... in order, then a fixed shuffle tree adds the
// lanes.  The split depends on the column only, so identical rows give
// identical sums.
template <int KIND, int M>
__device__ inline void group_sums(const float* const (&xi)[M], const float* const (&xc)[M], int d4, int l,
                                  float (&s)[M]) {
#pragma unroll
  for (int m = 0; m < M; ++m) s[m] = 0.f;
  for (int c = l; c < d4; c += kSeedLanes) {
    float4 a[M], b[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
      a[m] = ((const float4*)xi[m])[c];
      b[m] = ((const float4*)xc[m])[c];
    }
#pragma unroll
    for (int m = 0; m < M; ++m) {
      if (KIND == GAUSS) {
        float t = a[m].x - b[m].x;
        s[m] = fmaf(t, t, s[m]);
        t = a[m].y - b[m].y;
        s[m] = fmaf(t, t, s[m]);
        t = a[m].z - b[m].z;
        s[m] = fmaf(t, t, s[m]);
        t = a[m].w - b[m].w;
        s[m] = fmaf(t, t, s[m]);
      } else {
        s[m] = fmaf(a[m].x, b[m].x, s[m]);
        s[m] = fmaf(a[m].y, b[m].y, s[m]);
        s[m] = fmaf(a[m].z, b[m].z, s[m]);
        s[m] = fmaf(a[m].w, b[m].w, s[m]);
      }
    }
  }
#pragma unroll
  for (int off = kSeedLanes / 2; off > 0; off >>= 1)
#pragma unroll
    for (int m = 0; m < M; ++m) s[m] += __shfl_xor(s[m], off, kSeedLanes);
}

// kappa from the group sum: the Gaussian takes the squared difference.
template <int KIND>
__device__ inline float kentry(float s, const KappaParams& kp) {
  if (KIND == GAUSS) return __builtin_amdgcn_exp2f(kp.neg_g_log2e * s);
  return kappa<KIND>(s, 0.f, 0.f, kp);
}

// LDS of a draw.
struct DrawLds {
  double wsum[kSeedThr / 64], val;
  int vote[kSeedThr / 64], index;
  unsigned char used[KKM_MAX_K];
};

// The lowest index not among centers[0 .. t-1]; it is at most t (< n).  All
// threads call.
__device__ inline int lowest_unused(const int* __restrict__ centers, int t, DrawLds& x) {
  const int tid = threadIdx.x;
  for (int i = tid; i < t; i += kSeedThr) x.used[i] = 0;
  if (tid == 0) x.index = t;
  __syncthreads();
  for (int i = tid; i < t; i += kSeedThr)
    if (centers[i] < t) x.used[centers[i]] = 1;
  __syncthreads();
  for (int i = tid; i < t; i += kSeedThr)
    if (!x.used[i]) atomicMin(&x.index, i);
  __syncthreads();
  return x.index;
}

// Inclusive prefix sums of v over the workgroup's threads: a fixed shuffle
// tree per wavefront, then the wavefronts' totals in order.
__device__ inline double block_scan(double v, DrawLds& x) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const double o = __shfl_up(v, off, 64);
    if (lane >= off) v += o;
  }
  if (lane == 63) x.wsum[w] = v;
  __syncthreads();
  double before = 0.0;
  for (int u = 0; u < w; ++u) before += x.wsum[u];
  __syncthreads();
  return before + v;
}

// The lowest (or highest) thread whose flag is set, -1 if none; all threads call.
__device__ inline int block_vote(bool f, bool lowest, DrawLds& x) {
  const int w = threadIdx.x >> 6;
  const unsigned long long m = __ballot(f);
  if ((threadIdx.x & 63) == 0)
    x.vote[w] = !m ? -1 : w * 64 + (lowest ? __ffsll(m) - 1 : 63 - __clzll((long long)m));
  __syncthreads();
  int r = -1;
  for (int u = 0; u < kSeedThr / 64; ++u) {
    const int v = x.vote[u];
    if (v >= 0 && (r < 0 || !lowest)) r = v;
  }
  __syncthreads();
  return r;
}

__device__ inline double block_bcast(double v, int src, DrawLds& x) {
  if ((int)threadIdx.x == src) x.val = v;
  __syncthreads();
  const double r = x.val;
  __syncthreads();
  return r;
}

// Draws center t from D with the uniform ut: the first index whose prefix
// sum exceeds ut * S, with D(i) > 0.  Three levels, each prefix-summed in
// parallel by a fixed tree: runs of block sums (one per thread), the blocks
// of the run holding the target, the points of the block holding it; at each
// level the lowest qualifying entry wins.  The levels' sums are associated
// differently, so rounding can leave a level short of the target: then its
// last entry with a positive weight is taken.  If S = 0, the lowest index not
// yet chosen.  Every thread returns the index.
__device__ inline int draw_center(const float* __restrict__ D, const double* __restrict__ bsum, int nblk, int64_t n,
                                  double ut, const int* __restrict__ centers, int t, DrawLds& x) {
  const int tid = threadIdx.x;
  // level 1: runs of `per` block sums, one per thread, added in order
  const int per = (nblk + kSeedThr - 1) / kSeedThr;
  const int b0 = tid * per, b1 = min(nblk, b0 + per);
  double r = 0.0;
  for (int b = b0; b < b1; b += 8) {  // eight loads in flight
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = bsum[min(b + u, nblk - 1)];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (b + u < b1) r += v[u];
  }
  const double P1 = block_scan(r, x);
  const double S = block_bcast(P1, kSeedThr - 1, x);
  int index = -1;  // (uniform branches from here on)
  if (S > 0.0) {
    const double target = ut * S;
    int j = block_vote(r > 0.0 && P1 > target, true, x);
    if (j < 0) j = block_vote(r > 0.0, false, x);
    double base = block_bcast(P1 - r, j, x);

    // level 2: the blocks of run j, kSeedThr at a time
    const int m_lo = j * per, m_hi = min(nblk, m_lo + per);
    int blk = -1, fb_blk = -1;
    double fb_base = 0.0;
    for (int m0 = m_lo; m0 < m_hi && blk < 0; m0 += kSeedThr) {
      const int m = m0 + tid;
      const double v = m < m_hi ? bsum[m] : 0.0;
      const double P2 = base + block_scan(v, x);
      const int f = block_vote(v > 0.0 && P2 > target, true, x);
      if (f >= 0) {
        blk = m0 + f;
        base = block_bcast(P2 - v, f, x);
      } else {
        const int lp = block_vote(v > 0.0, false, x);
        if (lp >= 0) {
          fb_blk = m0 + lp;
          fb_base = block_bcast(P2 - v, lp, x);
        }
        base = block_bcast(P2, kSeedThr - 1, x);
      }
    }
    if (blk < 0) {
      blk = fb_blk;
      base = fb_base;
    }

    // level 3: the points of block blk
    const int64_t i0 = (int64_t)blk * kSeedPts;
    const float d = (tid < kSeedPts && i0 + tid < n) ? D[i0 + tid] : 0.f;
    const double P3 = base + block_scan((double)d, x);
    int f = block_vote(d > 0.f && P3 > target, true, x);
    if (f < 0) f = block_vote(d > 0.f, false, x);
    if (f >= 0) index = (int)(i0 + f);
  }
  return index < 0 ? lowest_unused(centers, t, x) : index;
}

// The draw of center t in a launch of its own.
__global__ __launch_bounds__(kSeedThr) void kpp_draw_kernel(const float* __restrict__ D, const double* __restrict__ bsum,
                                                           int nblk, int64_t n, double ut, int* __restrict__ centers,
                                                           int t) {
  __shared__ DrawLds x;
  const int c = draw_center(D, bsum, nblk, n, ut, centers, t, x);
  if (threadIdx.x == 0) centers[t] = c;
}

// Bound by latency and the read of the points (in the last-level cache up to
// some 200 MB).  n = 100000, d = 128, 64 centers: 1.55 -> 0.94 ms with the draw
// in the pass (a launch per center instead of two) and four points' loads in
// flight per group.
//
// Center t (c_first when t = 0, else drawn with ut from D_in and bsum_in, here or,
// drawn set, before this launch):
// D_out = min(D_in, distance), the nearest centers, the block's fp64 sum of
// D_out (fixed order).  kd[i] = K(i,i) by the same routine (written when t =
// 0).  V, when not null, receives each point's nearest center (the last pass).
template <int KIND>
__global__ __launch_bounds__(kSeedThr) void kpp_pass_kernel(const float* __restrict__ Xp, int64_t n, int d_pad,
                                                           KappaParams kp, int* __restrict__ centers, int t,
                                                           int c_first, double ut, int nblk, bool drawn,
                                                           const float* __restrict__ D_in,
                                                           const double* __restrict__ bsum_in,
                                                           float* __restrict__ kd, float* __restrict__ D_out,
                                                           int* __restrict__ bestc, double* __restrict__ bsum_out,
                                                           int* __restrict__ V) {
  __shared__ DrawLds x;
  __shared__ float dpt[kSeedPts];
  const int tid = threadIdx.x, l = tid % kSeedLanes, p = tid / kSeedLanes;
  const int c = t == 0 ? c_first : drawn ? centers[t] : draw_center(D_in, bsum_in, nblk, n, ut, centers, t, x);
  if (!drawn && blockIdx.x == 0 && tid == 0) centers[t] = c;
  const int d4 = d_pad / 4;
  const int64_t i0 = (int64_t)blockIdx.x * kSeedPts + p * kSeedPer;
  const float *xi[kSeedPer], *xc[kSeedPer];
#pragma unroll
  for (int m = 0; m < kSeedPer; ++m) {
    xi[m] = Xp + (i0 + m < n ? i0 + m : c) * d_pad;  // rows past n read the center's (unused)
    xc[m] = Xp + (int64_t)c * d_pad;
  }
  float sic[kSeedPer], kii[kSeedPer];
  group_sums<KIND, kSeedPer>(xi, xc, d4, l, sic);
  float kcc = 1.f;
  if (t == 0 && KIND != GAUSS) {
    float s2[kSeedPer];
    group_sums<KIND, kSeedPer>(xi, xi, d4, l, s2);
#pragma unroll
    for (int m = 0; m < kSeedPer; ++m) kii[m] = kentry<KIND>(s2[m], kp);
    group_sums<KIND, kSeedPer>(xc, xc, d4, l, s2);
    kcc = kentry<KIND>(s2[0], kp);
  }
  // lane m of a group finishes point m
  if (l < kSeedPer) {
    float s = 0.f, k0 = 1.f;
#pragma unroll
    for (int m = 0; m < kSeedPer; ++m)
      if (l == m) {
        s = sic[m];
        if (t == 0 && KIND != GAUSS) k0 = kii[m];
      }
    const int64_t i = i0 + l;
    float dv = 0.f;
    if (i < n) {
      const float kic = kentry<KIND>(s, kp);
      if (t == 0) {
        kd[i] = k0;
      } else if (KIND != GAUSS) {
        k0 = kd[i];
        kcc = kd[c];
      }
      const float d2 = i == c ? 0.f : fmaxf((k0 + kcc) - 2.f * kic, 0.f);
      dv = d2;
      int bc = t;
      if (t > 0) {
        const float b0 = D_in[i];
        if (!(d2 < b0)) {
          dv = b0;
          bc = bestc[i];
        }
      }
      D_out[i] = dv;
      bestc[i] = bc;
      if (V) V[i] = bc;
    }
    dpt[p * kSeedPer + l] = dv;
  }
  __syncthreads();
  if (tid < 64) {
    static_assert(kSeedPts == 64, "one wavefront adds a block");
    double v = (double)dpt[tid];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if (tid == 0) bsum_out[blockIdx.x] = v;
  }
}

}  // namespace

int seed_blocks(int64_t n) { return (int)((n + kSeedPts - 1) / kSeedPts); }

hipError_t launch_kpp_pass(const float* Xp, int64_t n, int d_pad, const KappaParams& kp, int* centers, int t,
                           int c_first, double ut, const float* D_in, const double* bsum_in, float* kd, float* D_out,
                           int* bestc, double* bsum_out, int* V, hipStream_t s) {
  const int nblk = seed_blocks(n);
  const dim3 grid((unsigned)nblk), block(kSeedThr);
  const bool drawn = t > 0 && nblk > kSeedFusedBlk;
  if (drawn) {
    hipLaunchKernelGGL(kpp_draw_kernel, dim3(1), block, 0, s, D_in, bsum_in, nblk, n, ut, centers, t);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
#define KKM_KPP(KIND)                                                                                             \
  hipLaunchKernelGGL(kpp_pass_kernel<KIND>, grid, block, 0, s, Xp, n, d_pad, kp, centers, t, c_first, ut, nblk, drawn, D_in, \
                     bsum_in, kd, D_out, bestc, bsum_out, V)
  switch (kp.kind) {
    case LINEAR: KKM_KPP(LINEAR); break;
    case POLY: KKM_KPP(POLY); break;
    default: KKM_KPP(GAUSS); break;
  }
#undef KKM_KPP
  return hipGetLastError();
}

}  // namespace kkm

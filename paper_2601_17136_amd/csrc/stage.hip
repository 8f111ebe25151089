// Staging of the points and small helpers.
//
// The points X (n x d, fp32, row-major; the paper's P of Section II-B) are
// copied into a zero-padded n_pad x d_pad buffer so the K-build tiles never
// need bounds checks along k; zero columns leave every dot product, and so
// Eq. 1, unchanged.  The squared row norms |x_i|^2 are taken in the same pass
// (the Gaussian kernel's expansion |x|^2 + |y|^2 - 2 x.y needs them).
#include "split_mma.h"

namespace kkm {

// A workgroup stages kStageBlk rows, each wavefront kStageRows at once (their
// loads in flight together); per row, lane l sums the squares of columns l,
// l+64, ... in order and a fixed shuffle tree adds the lanes, so the norm is
// deterministic.  stat (kStatWords words, zero on entry) receives the largest
// norm as its IEEE bits (non-negative floats order like their bit patterns); a
// workgroup takes the max of its rows in LDS and updates the word only when its
// max is larger than what the word already holds.  A stale read only costs a
// redundant atomic.
//
// xinv (may be null): xinv[i] = 1 / s_i, the power of two that undoes row i's
// scale in the split points (split_mma.h); Xf (may be null): those points in
// operand order, zero past n.  The rows' largest coordinates come from the
// same pass as the norms, and the second pass reads the staged rows back from
// cache.  With xinv, stat also receives the range of the rows' largest
// coordinates, and with ranges (and xinv) what split_runs asks about each row's
// own: a row has many coordinates that the split holds to fewer bits if they
// are more than a sixteenth of its nonzero ones and at least three, or half.
constexpr int kStageRows = 4;
constexpr int kStageWaves = 8;  // (a block's rows at once: two turns of 4 wavefronts took a small build 2-4 us longer)
constexpr int kStageBlk = 32;

__device__ inline void raise_to(unsigned* word, unsigned bits) {
  if (__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < bits) atomicMax(word, bits);
}

__global__ __launch_bounds__(64 * kStageWaves) void stage_kernel(const float* __restrict__ X, int64_t n,
                                                                 int d, int d_pad, int64_t n_pad,
                                                                 float* __restrict__ Xp,
                                                                 float* __restrict__ nrm,
                                                                 unsigned* __restrict__ stat,
                                                                 half_t* __restrict__ Xf,
                                                                 float* __restrict__ xinv, bool ranges) {
  __shared__ float wmax[kStageWaves], whigh[kStageWaves], wlow[kStageWaves];
  __shared__ int nnz[kStageBlk], nlost[kStageBlk];
  __shared__ float scl[kStageBlk];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t b0 = (int64_t)blockIdx.x * kStageBlk;
  if (threadIdx.x < kStageBlk) nnz[threadIdx.x] = nlost[threadIdx.x] = 0;
  float m = 0.f, high = 0.f, low = INFINITY;
  for (int g = 0; g < kStageBlk / (kStageRows * kStageWaves); ++g) {
    const int64_t i0 = b0 + (g * kStageWaves + w) * kStageRows;
    float s[kStageRows], mx[kStageRows];
#pragma unroll
    for (int r = 0; r < kStageRows; ++r) s[r] = mx[r] = 0.f;
    for (int c = lane; c < d_pad; c += 64) {
      float v[kStageRows];
#pragma unroll
      for (int r = 0; r < kStageRows; ++r) {
        const int64_t i = i0 + r;
        v[r] = (i < n && c < d) ? X[i * d + c] : 0.f;
      }
#pragma unroll
      for (int r = 0; r < kStageRows; ++r) {
        const int64_t i = i0 + r;
        if (i < n_pad) Xp[i * d_pad + c] = v[r];
        s[r] = fmaf(v[r], v[r], s[r]);
        mx[r] = fmaxf(mx[r], fabsf(v[r]));
      }
    }
#pragma unroll
    for (int r = 0; r < kStageRows; ++r) {
      for (int off = 32; off > 0; off >>= 1) {
        s[r] += __shfl_xor(s[r], off, 64);
        mx[r] = fmaxf(mx[r], __shfl_xor(mx[r], off, 64));
      }
      if (lane == r && i0 + r < n_pad) nrm[i0 + r] = s[r];
      if (lane == r && xinv) {
        // s_i = 2^(14 - e) for a largest coordinate in [2^e, 2^(e+1)), at most
        // 2^126; 1 for a zero row and for one that holds an infinity
        const int e = max((int)(__float_as_uint(mx[r]) >> 23), 1) - 127;
        const int p = mx[r] > 0.f && mx[r] < INFINITY ? min(14 - e, 126) : 0;
        scl[i0 + r - b0] = __uint_as_float((unsigned)(127 + p) << 23);
        xinv[i0 + r] = __uint_as_float((unsigned)(127 - p) << 23);
      }
      m = fmaxf(m, s[r]);
      high = fmaxf(high, mx[r]);
      if (mx[r] > 0.f) low = fminf(low, mx[r]);
    }
  }
  if (lane == 0) {
    wmax[w] = m;
    whigh[w] = high;
    wlow[w] = low;
  }
  __syncthreads();
  // (a thread per word: one after the other their loads took 23 us more at
  // 50000 points; the coordinates in whole binades, which few workgroups raise)
  if (threadIdx.x == 0) {
    for (int q = 1; q < kStageWaves; ++q) m = fmaxf(m, wmax[q]);
    raise_to(stat + kStatNorm, __float_as_uint(m));
  } else if (threadIdx.x == 64 && xinv) {
    high = whigh[0];
    for (int q = 1; q < kStageWaves; ++q) high = fmaxf(high, whigh[q]);
    if (high > 0.f) raise_to(stat + kStatHigh, __float_as_uint(high) | 0x7fffffu);
  } else if (threadIdx.x == 128 && xinv) {
    low = wlow[0];
    for (int q = 1; q < kStageWaves; ++q) low = fminf(low, wlow[q]);
    if (low < INFINITY) raise_to(stat + kStatLow, ~(__float_as_uint(low) & 0x7f800000u));
  }
  if (!Xf && !ranges) return;
  const int nch = (d_pad + 15) / 16, l = lane & 31, h = lane >> 5;
  const float sc = scl[l];
  const float* row = Xp + (b0 + l) * d_pad + 8 * h;
  int nz = 0, lost = 0;
  for (int c = w; c < nch; c += kStageWaves) {
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (16 * c + 8 * h < d_pad) {  // (a multiple of 8)
      const float4 x0 = *(const float4*)(row + 16 * c), x1 = *(const float4*)(row + 16 * c + 4);
      v[0] = x0.x, v[1] = x0.y, v[2] = x0.z, v[3] = x0.w;
      v[4] = x1.x, v[5] = x1.y, v[6] = x1.z, v[7] = x1.w;
    }
    if (ranges) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        nz += v[e] != 0.f ? 1 : 0;
        lost += v[e] != 0.f && fabsf(v[e] * sc) < 0x1p-3f ? 1 : 0;
      }
    }
    if (Xf) split_store(v, sc, Xf + split_unit(blockIdx.x, nch, c, 0) * kUnit + lane * 8);
  }
  if (!ranges) return;
  atomicAdd(&nnz[l], nz);
  atomicAdd(&nlost[l], lost);
  __syncthreads();
  if (threadIdx.x < kStageBlk) {
    nz = nnz[l];
    lost = nlost[l];
    const unsigned any = __ballot(lost > 0) != 0 ? kLostAny : 0u;
    const bool many = lost > nz / 16 && (lost >= 3 || 2 * lost >= nz);
    const unsigned bits = any | (__ballot(lost > 0 && many) != 0 ? kLostShare : 0u);
    if (threadIdx.x == 0 && (bits & ~__hip_atomic_load(stat + kStatLost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)))
      atomicOr(stat + kStatLost, bits);
  }
}

hipError_t launch_stage(const float* X, int64_t n, int d, int d_pad, int64_t n_pad, float* Xp, float* nrm,
                        unsigned* maxnrm_bits, half_t* Xf, float* xinv, bool ranges,
                        hipStream_t s) {
  if (n_pad % kStageBlk || d_pad % 8 || ((Xf || ranges) && !xinv)) return hipErrorInvalidValue;
  dim3 grid((unsigned)(n_pad / kStageBlk));
  hipLaunchKernelGGL(stage_kernel, grid, dim3(64 * kStageWaves), 0, s, X, n, d, d_pad, n_pad, Xp, nrm,
                     maxnrm_bits, Xf, xinv, ranges);
  return hipGetLastError();
}

// tr K in fp64 with a fixed reduction order (one workgroup, sixteen loads in
// flight per thread); ones: every entry is 1 (the Gaussian's), so nothing is
// read (one CU reads a few GB/s: 41 us at 120000 points).
__global__ __launch_bounds__(1024) void trace_kernel(const float* __restrict__ diagK, int64_t n, bool ones,
                                                     double* __restrict__ out) {
  __shared__ double part[1024];
  if (ones) {
    if (threadIdx.x == 0) *out = (double)n;
    return;
  }
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += 16 * 1024) {
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = i + 1024 * u < n ? diagK[i + 1024 * u] : 0.f;
#pragma unroll
    for (int u = 0; u < 16; ++u) s += (double)v[u];  // in order
  }
  part[threadIdx.x] = s;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = part[0];
}

hipError_t launch_trace(const float* diagK, int64_t n, bool ones, double* trK, hipStream_t s) {
  hipLaunchKernelGGL(trace_kernel, dim3(1), dim3(ones ? 64 : 1024), 0, s, diagK, n, ones, trK);
  return hipGetLastError();
}

__global__ void fill_kernel(float* __restrict__ p, int64_t count, float v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = v;
}

hipError_t launch_fill_diag(float* diagK, int64_t n, float v, hipStream_t s) {
  hipLaunchKernelGGL(fill_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, diagK, n, v);
  return hipGetLastError();
}

__global__ void zero_ints_kernel(int* __restrict__ p, int64_t count, int* __restrict__ q, int64_t qcount) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = 0;
  if (i < qcount) q[i] = 0;
}

// A fill kernel rather than hipMemsetAsync, so a captured graph replays it safely.
hipError_t launch_zero_ints(int* p, int64_t count, hipStream_t s, int* q, int64_t qcount) {
  const int64_t most = std::max(count, qcount);
  if (most <= 0) return hipSuccess;
  hipLaunchKernelGGL(zero_ints_kernel, dim3((unsigned)((most + 255) / 256)), dim3(256), 0, s, p, count, q, qcount);
  return hipGetLastError();
}

}  // namespace kkm

// E = K V^T for problems small enough to be bound by launches and latency
// (IterBufs.small): one kernel in place of the sort, the SpMM over sorted
// chunks and its two reductions.
//
// A workgroup owns 16 rows and reads each of them whole, the part left of a
// packed row's first stored column by symmetry from the rows above (a packed K
// of this size sits in cache, so reading both triangles costs little).  The
// per-label sums are a product with the one-hot matrix of the column labels on
// v_mfma_f32_16x16x4_f32: every product is 0 or the entry itself, the sums are
// fp32, in a fixed order.  Nothing needs the points sorted, and nothing is
// left to reduce but the workgroups' parts of the self-terms, which the assign
// step adds.  An infinite or NaN entry must not reach the other labels as 0
// times itself: a wavefront whose sums come out not finite takes its entries
// once more with those set aside and added to their own label.
#include "kkm_internal.h"

namespace kkm {

typedef float f4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int kSmallThreads = 512, kSmallWaves = 8;

// Workgroup w: rows 16 w .. 16 w + 15.  NB blocks of 16 labels.  FULL: all of K
// is stored.  Wavefront v takes the 64-column batches v, v + 8, ...; lane (l, q)
// = (lane % 16, lane / 16) holds row l's entries at columns 16 g + 4 q .. + 3 of
// each 16-column group g, and instruction e takes entry e of every lane: its k
// slot q is column 16 g + 4 q + e.
// Bound by latency: one round trip for the ids, a few for the rows.  n = 2000,
// k = 8: 15.5 us per update with the assign step, before it 25 (packed) and 50
// (full).
template <int NB, bool FULL>
__global__ __launch_bounds__(kSmallThreads) void spmm_small_kernel(const float* __restrict__ K, IterBufs b,
                                                                   const int* __restrict__ cl,
                                                                   int* __restrict__ counts,
                                                                   int* __restrict__ zero_changed, bool check) {
  __shared__ __attribute__((aligned(16))) unsigned char lab[kSmallN];
  __shared__ f4 part[kSmallWaves][NB][64];
  __shared__ float esum[16 * NB][17];
  __shared__ float extra[16 * NB][17];  // infinite and NaN entries, by label and row
  __shared__ int hist[16 * NB];
  __shared__ int own[16];
  __shared__ int bad, any_extra;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, l16 = lane & 15, q = lane >> 4;
  const int n = (int)b.n, k = b.k, ld = (int)b.ld;
  const int r0 = (int)blockIdx.x * 16;
  const bool first = blockIdx.x == 0;  // this workgroup also counts the sizes (and checks the ids)
  if (first && tid < 16 * NB) hist[tid] = 0;
  if (tid == 0) bad = any_extra = 0;
  for (int x = tid; x < 16 * NB * 17; x += kSmallThreads) (&extra[0][0])[x] = 0.f;
  if (tid < 16) own[tid] = -1;
  __syncthreads();
  int wrong = 0;
  for (int i = tid; i < ld; i += kSmallThreads) {
    int c = i < n ? cl[i] : 255;  // columns past n hold zeros and match no label
    if (i < n) {
      if (c < 0 || c >= k) {
        wrong = 1;
        c = c < 0 ? 0 : k - 1;
      }
      if (first) atomicAdd(&hist[c], 1);
    }
    lab[i] = (unsigned char)c;
    if (i >= r0 && i < r0 + 16 && i < n) own[i - r0] = c;
  }
  if (first && wrong) bad = 1;
  __syncthreads();
  if (first) {
    if (tid < k) counts[tid] = hist[tid];
    if (tid == 0) {
      if (zero_changed) *zero_changed = 0;
      if (check) *b.status = bad;
    }
  }

  const int row = min(r0 + l16, n - 1);
  const float* rowp = K + (FULL ? (int64_t)row * ld : packed_row(row, ld));
  const int c0 = FULL ? 0 : r0 / kTile * kTile;  // first stored column of the rows
  f4 D[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) D[nb] = f4{0.f, 0.f, 0.f, 0.f};
  const int nbatch = ld / 64;
  auto load = [&](int t, f4(&v)[4]) {  // batch t: columns 64 t .. 64 t + 63
    const int cb = 64 * t;
    if (cb >= c0) {
#pragma unroll
      for (int g = 0; g < 4; ++g) v[g] = *(const f4*)(rowp + cb + 16 * g + 4 * q);
    } else {  // K(row, c) = K(c, row), stored in row c
      const int64_t S = ld - cb / kTile * kTile;
      const float* p = K + packed_row(cb, ld) + (int64_t)(4 * q) * S + row;
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[g][e] = p[(16 * g + e) * S];
    }
  };
  auto fold = [&](int t, const f4(&v)[4]) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const unsigned m = *(const unsigned*)(lab + 64 * t + 16 * g + 4 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = (int)((m >> (8 * e)) & 255u);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          D[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(c == 16 * nb + l16 ? 1.f : 0.f, v[g][e], D[nb], 0, 0, 0);
      }
    }
  };
  f4 v0[4], v1[4];  // two batches in flight
  int t = w;
  if (t < nbatch) load(t, v0);
  for (; t < nbatch; t += 2 * kSmallWaves) {
    if (t + kSmallWaves < nbatch) load(t + kSmallWaves, v1);
    fold(t, v0);
    if (t + 2 * kSmallWaves < nbatch) load(t + 2 * kSmallWaves, v0);
    if (t + kSmallWaves < nbatch) fold(t + kSmallWaves, v1);
  }
  bool finite = true;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 4; ++r) finite &= fabsf(D[nb][r]) < INFINITY;
  if (__ballot(!finite)) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) D[nb] = f4{0.f, 0.f, 0.f, 0.f};
    for (t = w; t < nbatch; t += kSmallWaves) {
      load(t, v0);
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x = v0[g][e];
          if (fabsf(x) < INFINITY) continue;
          // (columns past n hold zeros; which sum of infinities and NaN comes
          // out does not depend on their order)
          atomicAdd(&extra[min((int)lab[64 * t + 16 * g + 4 * q + e], k - 1)][l16], x);
          any_extra = 1;
          v0[g][e] = 0.f;
        }
      fold(t, v0);
    }
  }

  // the wavefronts' sums, in order: D[nb][r] is label 16 nb + 4 q + r of row l16
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) part[w][nb][lane] = D[nb];
  __syncthreads();
  for (int x = tid; x < NB * 64; x += kSmallThreads) {
    const int nb = x >> 6, ln = x & 63;
    f4 s = part[0][nb][ln];
#pragma unroll
    for (int ww = 1; ww < kSmallWaves; ++ww) s += part[ww][nb][ln];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = 16 * nb + 4 * (ln >> 4) + r, i = ln & 15;
      esum[j][i] = any_extra ? s[r] + extra[j][i] : s[r];
    }
  }
  __syncthreads();
  for (int x = tid; x < k * 16; x += kSmallThreads) {
    const int j = x >> 4, i = r0 + (x & 15);
    if (i < n) b.Et[(int64_t)j * ld + i] = esum[j][x & 15];
  }
  if (tid < k) {  // the rows' part of sum_{i in L_j} E(i, j)
    double zs = 0.0;
    for (int i = 0; i < 16; ++i)
      if (own[i] == tid) zs += (double)esum[tid][i];
    b.zpart[(int64_t)tid * b.nzpart + blockIdx.x] = zs;
  }
}

}  // namespace

hipError_t launch_spmm_small(const float* K, bool full, const IterBufs& b, const int* cl, int* counts,
                             int* zero_changed, bool check, hipStream_t s) {
  const int wgs = small_wgs(b.n), nb = (b.k + 15) / 16;
  if (b.n > kSmallN || b.ld > kSmallN || b.ld % 64 || b.nzpart != wgs || b.k > kSmallMaxK) return hipErrorInvalidValue;
#define KKM_SMALL(NB)                                                                                          \
  do {                                                                                                         \
    if (full)                                                                                                  \
      hipLaunchKernelGGL((spmm_small_kernel<NB, true>), dim3(wgs), dim3(kSmallThreads), 0, s, K, b, cl, counts,  \
                         zero_changed, check);                                                                 \
    else                                                                                                       \
      hipLaunchKernelGGL((spmm_small_kernel<NB, false>), dim3(wgs), dim3(kSmallThreads), 0, s, K, b, cl, counts, \
                         zero_changed, check);                                                                 \
  } while (0)
  switch (nb) {
    case 1: KKM_SMALL(1); break;
    case 2: KKM_SMALL(2); break;
    case 3: KKM_SMALL(3); break;
    default: KKM_SMALL(4); break;
  }
#undef KKM_SMALL
  return hipGetLastError();
}

}  // namespace kkm

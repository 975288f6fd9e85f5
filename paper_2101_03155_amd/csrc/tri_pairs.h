// Pairs i <= j in row-major order over the upper triangle, and their ordered
// compaction.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace ace {

// Pair t -> (i, j).  Row i starts at i n - i (i - 1) / 2.
__device__ __forceinline__ void tri_ij(int64_t t, int n, int& i, int& j) {
  const double a = 2.0 * n + 1.0;
  i = int((a - sqrt(a * a - 8.0 * double(t))) * 0.5);
  while (i > 0 && int64_t(i) * n - int64_t(i) * (i - 1) / 2 > t) --i;
  while (int64_t(i + 1) * n - int64_t(i + 1) * i / 2 <= t) ++i;
  j = i + int(t - (int64_t(i) * n - int64_t(i) * (i - 1) / 2));
}

// Calls put(p, i, j) for the p-th pair in order that keep(t, i, j) holds for, and
// writes the number of these.  One workgroup of CNT threads: each wave owns one
// stretch of the triangle, counts it, and after one barrier goes through it again
// with its first position known.  (Chunks of 1024 pairs in turn, with three
// barriers each, took 60 us for 32896 pairs; now 23.)
constexpr int CNT = 1024;
template <typename Keep, typename Put>
__device__ __forceinline__ void compact_tri(int n, Keep keep, Put put, int64_t* __restrict__ count) {
  __shared__ int64_t wsum[CNT / 64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t np = int64_t(n) * (n + 1) / 2;
  const int64_t len = ((np + CNT - 1) / CNT) * 64;
  const int64_t t0 = wv * len + lane, t1 = t0 - lane + len < np ? t0 - lane + len : np;
  int i0 = 0, j0 = 0;
  if (t0 < t1) tri_ij(t0, n, i0, j0);
  // 64 pairs further: the rows i0, i0 + 1, ... have n - i0, n - i0 - 1, ... pairs
  const auto next = [&](int& i, int& j) {
    j += 64;
    while (j >= n && i < n - 1) {
      ++i;
      j -= n - i;
    }
  };
  int64_t c = 0;
  {
    int i = i0, j = j0;
#pragma unroll 4
    for (int64_t t = t0; t < t1; t += 64) {
      c += keep(t, i, j) ? 1 : 0;
      next(i, j);
    }
  }
  for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off, 64);
  if (lane == 0) wsum[wv] = c;
  __syncthreads();
  int64_t off = 0;
  for (int w = 0; w < wv; ++w) off += wsum[w];
  if (threadIdx.x == CNT - 1) count[0] = off + wsum[wv];
  int i = i0, j = j0;
#pragma unroll 4
  for (int64_t g = t0 - lane; g < t1; g += 64) {
    const bool k = g + lane < t1 && keep(g + lane, i, j);
    const unsigned long long m = __ballot(k);
    if (k) put(off + __popcll(m & ((1ull << lane) - 1ull)), i, j);
    off += __popcll(m);
    next(i, j);
  }
}

}  // namespace ace

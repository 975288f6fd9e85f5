// A 16 x 16 tile of a small product on four waves.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace ace {

typedef double tiny_d4 __attribute__((ext_vector_type(4)));

// sum_{k < kend} (ss S(m, k)) (bs B(k, r)) over the tile of rows m0 .. m0 + 15 < M and
// columns r0 .. r0 + 15 < R; S(m, k) = TRANS ? S[k][m] : S[m][k],
// B(k, r) = BT ? B[r][k] : B[k][r], kend <= K.
// 256 threads: each wave takes a quarter of k with four steps' loads in flight,
// the sums meet in LDS, and wave 0 returns the tile (element q of lane l: row
// l / 16 + 4 q, column l % 16).  Operands come straight from global memory.
// Bound by latency: one wave per tile, a step at a time, took 13.7 us for
// 128^3 and 23.9 us for 256^3, this takes 3.8 and 5.1.
template <typename TB, bool TRANS, bool BT = false>
__device__ __forceinline__ tiny_d4 tiny_tile(const double* __restrict__ S, int lds, const TB* __restrict__ B,
                                             int64_t ldb, int m0, int64_t r0, int M, int K, int64_t R, int kend,
                                             double ss = 1.0, double bs = 1.0) {
  __shared__ double part[3][256];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
  const int ks = (kend + 15) / 16 * 4, kb = w * ks, ke = kb + ks < kend ? kb + ks : kend;
  // rows and columns past the edge repeat the last one and count as zero
  const bool mok = m0 + li < M, rok = r0 + li < R;
  const int m = mok ? m0 + li : M - 1;
  const int64_t r = rok ? r0 + li : R - 1;
  tiny_d4 acc = tiny_d4{0, 0, 0, 0};
  for (int k0 = kb; k0 < ke; k0 += 16) {
    double a[4], b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int k = k0 + 4 * u + lk, kc = k < K ? k : K - 1;
      a[u] = TRANS ? S[int64_t(kc) * lds + m] : S[int64_t(m) * lds + kc];
      b[u] = double(BT ? B[r * ldb + kc] : B[int64_t(kc) * ldb + r]);
      a[u] = k < ke && mok ? ss * a[u] : 0.0;
      b[u] = k < ke && rok ? bs * b[u] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[u], acc, 0, 0, 0);
  }
  if (w > 0)
#pragma unroll
    for (int q = 0; q < 4; ++q) part[w - 1][q * 64 + lane] = acc[q];
  __syncthreads();
  if (w == 0)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] += part[0][q * 64 + lane] + part[1][q * 64 + lane] + part[2][q * 64 + lane];
  return acc;
}

}  // namespace ace

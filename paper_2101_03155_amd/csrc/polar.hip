// Loewdin rotation U = A_C (A_C^T A_C)^-1/2: the polar factor of the norb x norb
// matrix A_C by the Newton-Schulz iteration X <- X (3 I - X^T X) / 2 from X = A_C
// scaled so that every singular value is at most 1 (divided by the square root
// of the largest absolute row sum of A_C^T A_C).
//
// Up to 64 orbitals the iteration runs in one workgroup with X and G = X^T X in
// LDS, from the gather of A_C to the check of the result; beyond, an iteration
// is two launches over 16 x 16 tiles.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "ace_internal.h"
#include "tiny_tile.h"

namespace ace {

// The larger of two deviations; one that is not a number counts as infinite.
__device__ __forceinline__ double worst(double m, double d) { return d <= m ? m : d < INFINITY ? d : INFINITY; }

// ---------------------------------------------------------------- one workgroup
// The matrix is padded to 64 x 64 with zeros, so the products run on the FP64
// matrix cores without edges: wave w owns tile (w / 4, w % 4).  The pitch of 65
// leaves two-way bank conflicts in both operand reads (rows and columns).
// stat: 0 converged, 1 a value that is not finite, 2 not converged.  As in the
// tiled iteration max|X^T X - I| is tested on every second iteration from the
// fourth on, and two more follow once it is below 1e-11.
// Bound by the chain of barriers and MFMAs of its iterations: 12 us at 8
// orbitals, where some 35 launches and two or three waits of the host took 200.
constexpr int PN = 64, PP = PN + 1;
__global__ __launch_bounds__(1024) void k_polar_small(const double* __restrict__ psi, int n, int64_t ng,
                                                      const int32_t* __restrict__ piv, double* __restrict__ X,
                                                      double* __restrict__ U, double* __restrict__ stat) {
  __shared__ double Xs[PN * PP], Gs[PN * PP];
  __shared__ double sdev[16], snorm;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, li = lane & 15, lk = lane >> 4;
  const int nt = (n + 15) / 16, m0 = (w >> 2) * 16, r0 = (w & 3) * 16;
  const bool mine = m0 < n && r0 < n;
  for (int e = tid; e < PN * PN; e += 1024) {
    const int i = e / PN, k = e % PN;
    Xs[i * PP + k] = i < n && k < n ? psi[int64_t(i) * ng + piv[k]] : 0.0;
  }
  __syncthreads();
  const auto product = [&](const double* S, bool trans, const double* B) {
    tiny_d4 acc = tiny_d4{0, 0, 0, 0};
    if (mine)
      for (int k0 = 0; k0 < nt * 16; k0 += 16)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = k0 + 4 * u + lk;
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(trans ? S[k * PP + m0 + li] : S[(m0 + li) * PP + k],
                                                     B[k * PP + r0 + li], acc, 0, 0, 0);
        }
    return acc;
  };
  {
    const tiny_d4 g = product(Xs, true, Xs);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (mine) Gs[(m0 + lk + 4 * q) * PP + r0 + li] = g[q];
  }
  __syncthreads();
  if (w == 0) {
    double s = 0.0;
    if (lane < n)
      for (int j = 0; j < n; ++j) s += fabs(Gs[lane * PP + j]);
    for (int off = 32; off > 0; off >>= 1) s = fmax(s, __shfl_xor(s, off, 64));
    if (lane == 0) snorm = s;
  }
  __syncthreads();
  const double inv = 1.0 / sqrt(snorm);
  for (int e = tid; e < PN * PN; e += 1024) {
    const int i = e / PN, k = e % PN;
    if (i < n && k < n) Xs[i * PP + k] *= inv;
  }
  __syncthreads();
  int left = -1;  // iterations still to do once converged
  for (int it = 0; it < 200 || left > 0; ++it) {
    const tiny_d4 g = product(Xs, true, Xs);
    const bool test = left < 0 && it >= 4 && it % 2 == 0;
    double dev = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = m0 + lk + 4 * q, j = r0 + li;
      if (mine) Gs[i * PP + j] = g[q];
      const double d = i < n && j < n ? fabs(g[q] - (i == j ? 1.0 : 0.0)) : 0.0;
      dev = worst(dev, d);
    }
    if (test) {
      for (int off = 32; off > 0; off >>= 1) dev = fmax(dev, __shfl_xor(dev, off, 64));
      if (lane == 0) sdev[w] = dev;
    }
    __syncthreads();
    if (test) {
      double h = sdev[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) h = fmax(h, sdev[i]);
      if (!isfinite(h)) {  // (the same in every thread)
        if (tid == 0) *stat = 1.0;
        return;
      }
      if (h < 1e-11) left = 2;
    }
    const tiny_d4 z = product(Xs, false, Gs);
    tiny_d4 x;
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = 1.5 * Xs[(m0 + lk + 4 * q) * PP + r0 + li] - 0.5 * z[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (mine) Xs[(m0 + lk + 4 * q) * PP + r0 + li] = x[q];
    __syncthreads();
    if (left > 0 && --left == 0) break;
  }
  for (int e = tid; e < n * n; e += 1024) {
    const double v = Xs[e / n * PP + e % n];
    X[e] = v;
    if (U) U[e] = v;
  }
  if (tid == 0) *stat = left == 0 ? 0.0 : 2.0;
}

// ---------------------------------------------------------------- tiles
// G = X^T X; dev[tile] = max |G - I| over the tile.
__global__ __launch_bounds__(256) void k_ns_gram(const double* __restrict__ X, int n, double* __restrict__ G,
                                                 double* __restrict__ dev) {
  const int m0 = blockIdx.y * 16, r0 = blockIdx.x * 16, lane = threadIdx.x;
  const tiny_d4 g = tiny_tile<double, true>(X, n, X, n, m0, r0, n, n, n, n);
  if (lane >= 64) return;
  double m = 0.0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = m0 + lane / 16 + 4 * q, j = r0 + lane % 16;
    if (i >= n || j >= n) continue;
    G[int64_t(i) * n + j] = g[q];
    const double d = fabs(g[q] - (i == j ? 1.0 : 0.0));
    m = worst(m, d);
  }
  for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_down(m, off, 64));
  if (lane == 0) dev[blockIdx.y * gridDim.x + blockIdx.x] = m;
}

// rows[i] = sum_j |G[i][j]|, one wave per row
__global__ __launch_bounds__(256) void k_row_abs(const double* __restrict__ G, int n, double* __restrict__ rows) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (i >= n) return;
  double s = 0.0;
  for (int j = lane; j < n; j += 64) s += fabs(G[int64_t(i) * n + j]);
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if (lane == 0) rows[i] = s;
}

// Y = 1.5 X - 0.5 X G.  With rows (the first iteration) X and G stand for the
// scaled X / sqrt(s) and its G / s, s the largest of the n row sums; both are
// scaled before they are multiplied, so that only squares need be in range.
__global__ __launch_bounds__(256) void k_ns_step(const double* __restrict__ X, const double* __restrict__ G,
                                                 const double* __restrict__ rows, int n, double* __restrict__ Y) {
  const int m0 = blockIdx.y * 16, r0 = blockIdx.x * 16, lane = threadIdx.x & 63;
  double inv = 1.0, invs = 1.0;
  if (rows) {
    double s = 0.0;
    for (int j = lane; j < n; j += 64) s = fmax(s, rows[j]);
    for (int off = 32; off > 0; off >>= 1) s = fmax(s, __shfl_xor(s, off, 64));
    inv = 1.0 / sqrt(s);
    invs = 1.0 / s;
  }
  const tiny_d4 z = tiny_tile<double, false>(X, n, G, n, m0, r0, n, n, n, n, inv, invs);
  if (threadIdx.x >= 64) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = m0 + lane / 16 + 4 * q, j = r0 + lane % 16;
    if (i < n && j < n) Y[int64_t(i) * n + j] = 1.5 * (inv * X[int64_t(i) * n + j]) - 0.5 * z[q];
  }
}

// dg = {max_k A_kk, min_k A_kk, *info}
__global__ __launch_bounds__(64) void k_diag_range(const double* __restrict__ A, int n, const int* __restrict__ info,
                                                   double* __restrict__ dg) {
  double mx = 0.0, mn = INFINITY;
  for (int k = threadIdx.x; k < n; k += 64) {
    const double d = A[int64_t(k) * n + k];
    mx = fmax(mx, d);
    mn = fmin(mn, d);
  }
  for (int off = 32; off > 0; off >>= 1) {
    mx = fmax(mx, __shfl_down(mx, off, 64));
    mn = fmin(mn, __shfl_down(mn, off, 64));
  }
  if (threadIdx.x == 0) {
    dg[0] = mx;
    dg[1] = mn;
    dg[2] = double(*info);
  }
}

// ---------------------------------------------------------------- launchers
bool polar_fits_one(int n) { return n <= PN; }
int polar_tiles(int n) { return ((n + 15) / 16) * ((n + 15) / 16); }
void launch_polar_small(const double* psi, int n, int64_t ng, const int32_t* piv, double* X, double* U, double* stat,
                        hipStream_t s) {
  hipLaunchKernelGGL(k_polar_small, dim3(1), dim3(1024), 0, s, psi, n, ng, piv, X, U, stat);
}
void launch_ns_gram(const double* X, int n, double* G, double* dev, hipStream_t s) {
  const unsigned nt = unsigned((n + 15) / 16);
  hipLaunchKernelGGL(k_ns_gram, dim3(nt, nt), dim3(256), 0, s, X, n, G, dev);
}
void launch_row_abs(const double* G, int n, double* rows, hipStream_t s) {
  hipLaunchKernelGGL(k_row_abs, dim3(unsigned((n + 3) / 4)), dim3(256), 0, s, G, n, rows);
}
void launch_ns_step(const double* X, const double* G, const double* rows, int n, double* Y, hipStream_t s) {
  const unsigned nt = unsigned((n + 15) / 16);
  hipLaunchKernelGGL(k_ns_step, dim3(nt, nt), dim3(256), 0, s, X, G, rows, n, Y);
}
void launch_diag_range(const double* A, int n, const int* info, double* dg, hipStream_t s) {
  hipLaunchKernelGGL(k_diag_range, dim3(1), dim3(64), 0, s, A, n, info, dg);
}

}  // namespace ace

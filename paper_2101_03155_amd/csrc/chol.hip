// FP64 Cholesky factorization A = L L^T and X = L^-1 of the norb x norb matrices
// (n <= 512).  Up to 128 columns one workgroup does both in LDS; larger matrices
// take 128-column blocks: a block's factor and inverse, the rows below it
// (L21 = A21 X11^T with one correction), the trailing update, and at the end the block rows of X,
// products of 16 x 16 tiles.
//
// info = k + 1 when the pivot of column k is not positive, -(k + 1) when it is
// not finite; every kernel returns at once when info is already set.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "ace_internal.h"
#include "tiny_tile.h"

namespace ace {

// ---------------------------------------------------------------- one block
// The block sits in LDS with a pitch of 129: L in the lower triangle, and X in
// what is left, element (i, j) at (j, i + 1).  Columns go by panels of 16.  Wave 0
// factors the panel's diagonal block and inverts it in registers, a row per lane
// (four copies of the block) with broadcasts in rows of 16 lanes; the rows below
// are multiplied by that inverse, corrected once for what its rounding leaves of
// A21, and the trailing matrix is updated by 16 x 16 tiles on the FP64 matrix
// cores, as are the block rows of X: X_IJ = -X_II Y, Y = sum_K L_IK X_KJ, corrected
// once by the residual of L_II X_IJ = -Y.  A tile's accumulators are directly the
// right operand of the next product (step u takes the k's lk + 4 u).  The
// corrections make up for the explicit inverses: without them 64 columns of
// which every fifth repeats its neighbour to 1e-6 are taken for not positive
// definite (condition 1e13), and for 130 such to 1e-5 X^T X times the matrix is
// off by 4e-7 instead of 1e-11.  Rows and columns past n are those of the
// identity, so there are no edges.
// Bound by the chain of the diagonal blocks (sixteen dependent pivots each):
// 128 columns with the inverse take 71 us, 64 31, 8 9 (a scalar trailing update
// and pivots passed through LDS took 172, 73 and 11; 256 columns by blocks of 64
// and a wave per column of the inverse 620, now 187, of which the corrections'
// launches are 20).  512 threads, as wave 0
// needs 185 registers: with 1024 it spilled and took 115.
constexpr int CBN = 128, CP = CBN + 1, CNT = 512, CW = CNT / 64, CR = CNT / CBN;

// Lane L of each row of 16 lanes to the whole row.
template <int L>
__device__ __forceinline__ double row_lane(double v) {
  return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), 0x150 + L, 0xf, 0xf, false),
                          __builtin_amdgcn_mov_dpp(__double2loint(v), 0x150 + L, 0xf, 0xf, false));
}
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// A (n x n at pitch lda, lower triangle read) becomes L with zeros above it; with
// X (pitch ldx) also the inverse, and zeros in the `rest` columns right of it.
// col0 is the global index of the first column.
__global__ __launch_bounds__(CNT) void k_chol_block(double* __restrict__ A, int lda, int n, int col0,
                                                     int* __restrict__ info, double* __restrict__ X, int ldx,
                                                     int rest) {
  __shared__ double S[CBN * CP];
  __shared__ int sbad;
  if (*info) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, li = lane & 15, lk = lane >> 4;
  const int nb = (n + 15) / 16, np = nb * 16;
  if (tid == 0) sbad = 0;
  // rows i0, i0 + CR, ... of column tid % 128, all loads in flight
  const int j0 = tid & (CBN - 1), i0 = tid / CBN;
  {
    double v[CBN / CR];
#pragma unroll
    for (int t = 0; t < CBN / CR; ++t) {
      const int i = i0 + CR * t;
      v[t] = i == j0 ? 1.0 : 0.0;
      if (i < n && j0 <= i) v[t] = A[int64_t(i) * lda + j0];
    }
#pragma unroll
    for (int t = 0; t < CBN / CR; ++t) {
      const int i = i0 + CR * t;
      if (j0 <= i) S[i * CP + j0] = v[t];
    }
  }
  __syncthreads();
  for (int b = 0; b < nb; ++b) {
    const int k0 = 16 * b;
    if (w == 0) {
      int lr = li;  // opaque: masks of all rows kept from panel to panel would spill
      asm volatile("" : "+v"(lr));
      // row lr of the block and of its inverse, which starts as the identity:
      // both are eliminated together
      double v[16], x[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        v[j] = j <= lr ? S[(k0 + lr) * CP + k0 + j] : 0.0;
        x[j] = j == lr ? 1.0 : 0.0;
      }
      int bad = 0;  // (the same in all lanes; past a bad pivot the values are not used)
      static_for<0, 16>([&](auto kc) {
        constexpr int k = kc();
        const double d = row_lane<k>(v[k]);
        if (bad == 0 && !isfinite(d)) bad = -(col0 + k0 + k + 1);
        if (bad == 0 && !(d > 0.0)) bad = col0 + k0 + k + 1;
        // 1 / sqrt(d): the hardware's approximation y (about 26 bits) times the
        // binomial series of (1 - e)^(-1/2) = 1 + e / 2 + 3 e^2 / 8 + ..., e = 1 -
        // d y^2, to second order; sqrt(d) from it with a Newton correction
        double y = __builtin_amdgcn_rsq(d);
        const double e = fma(-(d * y), y, 1.0);
        y = fma(y * e, fma(0.375, e, 0.5), y);
        double r = d * y;
        r = fma(fma(-r, r, d), 0.5 * y, r);
        const double l = lr > k ? v[k] * y : 0.0;
        v[k] = lr == k ? r : l;
        static_for<k + 1, 16>([&](auto jc) { v[jc()] = fma(-l, row_lane<jc()>(l), v[jc()]); });
        static_for<0, k + 1>([&](auto cc) {
          const double xk = row_lane<k>(x[cc()]) * y;
          x[cc()] = lr == k ? xk : fma(-l, xk, x[cc()]);
        });
        __builtin_amdgcn_sched_barrier(0);  // (else the broadcasts of several pivots are live and spill)
      });
      if (lane < 16) {
        if (bad) {
          if (lane == 0) sbad = bad;
        } else {
#pragma unroll
          for (int j = 0; j < 16; ++j)
            if (j <= lr) {
              S[(k0 + lr) * CP + k0 + j] = v[j];
              S[(k0 + j) * CP + k0 + lr + 1] = x[j];
            }
        }
      }
    }
    __syncthreads();
    if (sbad) break;
    // rows below: L21^T = X11 A21^T and one correction, L21^T += X11 (A21^T - L11
    // L21^T), a wave per 16 rows; each product's accumulators are the right
    // operand of the next
    for (int rb = b + 1 + w; rb < nb; rb += CW) {
      const double* a21 = S + (16 * rb + li) * CP + k0;
      double x11[4], l11[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = lk + 4 * u;
        x11[u] = k <= li ? S[(k0 + k) * CP + k0 + li + 1] : 0.0;
        l11[u] = k <= li ? S[(k0 + li) * CP + k0 + k] : 0.0;
      }
      tiny_d4 t = tiny_d4{0, 0, 0, 0}, p = tiny_d4{0, 0, 0, 0};
#pragma unroll
      for (int u = 0; u < 4; ++u) t = __builtin_amdgcn_mfma_f64_16x16x4f64(x11[u], a21[lk + 4 * u], t, 0, 0, 0);
#pragma unroll
      for (int u = 0; u < 4; ++u) p = __builtin_amdgcn_mfma_f64_16x16x4f64(l11[u], t[u], p, 0, 0, 0);
#pragma unroll
      for (int u = 0; u < 4; ++u)
        t = __builtin_amdgcn_mfma_f64_16x16x4f64(x11[u], a21[lk + 4 * u] - p[u], t, 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q) S[(16 * rb + li) * CP + k0 + lk + 4 * q] = t[q];
    }
    __syncthreads();
    // trailing update of the tiles (bi, bj), b < bj <= bi < nb
    const int m = nb - 1 - b;
    for (int t = w; t < m * (m + 1) / 2; t += CW) {
      int bi = 0, bj = t;
      while (bj > bi) bj -= ++bi;
      bi += b + 1;
      bj += b + 1;
      tiny_d4 acc = tiny_d4{0, 0, 0, 0};
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = k0 + lk + 4 * u;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(S[(16 * bi + li) * CP + k], S[(16 * bj + li) * CP + k], acc, 0, 0,
                                                   0);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = 16 * bi + lk + 4 * q, j = 16 * bj + li;
        if (j <= i) S[i * CP + j] -= acc[q];
      }
    }
    __syncthreads();
  }
  if (sbad) {
    if (tid == 0) *info = sbad;
    return;
  }
  if (j0 < n)
    for (int i = i0; i < n; i += CR) A[int64_t(i) * lda + j0] = j0 <= i ? S[i * CP + j0] : 0.0;
  if (!X) return;
  for (int I = 1; I < nb; ++I) {
    for (int J = w; J < I; J += CW) {
      tiny_d4 y = tiny_d4{0, 0, 0, 0}, z = tiny_d4{0, 0, 0, 0}, p = tiny_d4{0, 0, 0, 0};
      for (int K = J; K < I; ++K)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int k = lk + 4 * u;
          y = __builtin_amdgcn_mfma_f64_16x16x4f64(
              S[(16 * I + li) * CP + 16 * K + k],
              K > J || li <= k ? S[(16 * J + li) * CP + 16 * K + k + 1] : 0.0, y, 0, 0, 0);
        }
      double xii[4], lii[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = lk + 4 * u;
        xii[u] = k <= li ? S[(16 * I + k) * CP + 16 * I + li + 1] : 0.0;
        lii[u] = k <= li ? S[(16 * I + li) * CP + 16 * I + k] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) z = __builtin_amdgcn_mfma_f64_16x16x4f64(xii[u], y[u], z, 0, 0, 0);
#pragma unroll
      for (int u = 0; u < 4; ++u) p = __builtin_amdgcn_mfma_f64_16x16x4f64(lii[u], z[u], p, 0, 0, 0);
#pragma unroll
      for (int u = 0; u < 4; ++u) z = __builtin_amdgcn_mfma_f64_16x16x4f64(xii[u], y[u] - p[u], z, 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q) S[(16 * J + li) * CP + 16 * I + lk + 4 * q + 1] = -z[q];
    }
    __syncthreads();
  }
  if (j0 < n)
    for (int i = i0; i < n; i += CR) X[int64_t(i) * ldx + j0] = j0 <= i ? S[j0 * CP + i + 1] : 0.0;
  for (int e = tid; e < n * rest; e += CNT) X[int64_t(e / rest) * ldx + n + e % rest] = 0.0;
}

// ---------------------------------------------------------------- between blocks
// C(m, r) = beta C(m, r) + alpha sum_k S[m][k] B(k, r) over 16 x 16 tiles, every
// matrix at pitch ld, B(k, r) = BT ? B[r][k] : B[k][r].  LOWER: tiles with
// columns beyond their rows are left alone.
template <bool BT, bool LOWER>
__global__ __launch_bounds__(256) void k_chol_tile(const double* __restrict__ S, const double* __restrict__ B,
                                                   double* __restrict__ C, int ld, int M, int K, int R, double alpha,
                                                   double beta, const int* __restrict__ info) {
  const int m0 = blockIdx.y * 16, r0 = blockIdx.x * 16, lane = threadIdx.x;
  if (*info || (LOWER && r0 > m0)) return;
  const tiny_d4 acc = tiny_tile<double, false, BT>(S, ld, B, ld, m0, r0, M, K, R, K);
  if (lane >= 64) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = m0 + lane / 16 + 4 * q, j = r0 + lane % 16;
    if (i >= M || j >= R) continue;
    double* p = C + int64_t(i) * ld + j;
    *p = beta == 0.0 ? alpha * acc[q] : beta * *p + alpha * acc[q];
  }
}

// ---------------------------------------------------------------- launchers
static dim3 tiles(int M, int R) { return dim3(unsigned((R + 15) / 16), unsigned((M + 15) / 16)); }

// L in A for n <= 128.  Else A receives the diagonal blocks of L, X (n x n) their
// inverses and the blocks of L below them; A's blocks there end as residuals.
void launch_cholesky(double* A, int n, int* info, double* X, hipStream_t s) {
  if (n <= CBN) {
    hipLaunchKernelGGL(k_chol_block, dim3(1), dim3(CNT), 0, s, A, n, n, 0, info, (double*)nullptr, n, 0);
    return;
  }
  for (int k0 = 0; k0 < n; k0 += CBN) {
    const int b = n - k0 < CBN ? n - k0 : CBN, rest = n - k0 - b;
    const int64_t d = int64_t(k0) * n + k0, below = d + int64_t(b) * n;
    hipLaunchKernelGGL(k_chol_block, dim3(1), dim3(CNT), 0, s, A + d, n, b, k0, info, X + d, n, rest);
    if (rest == 0) break;
    // L21 = A21 X11^T, then A21 -= L21 L11^T and L21 += A21 X11^T: one correction
    const auto product = [&](const double* S, const double* B, double* C, double alpha, double beta) {
      hipLaunchKernelGGL((k_chol_tile<true, false>), tiles(rest, b), dim3(256), 0, s, S, B, C, n, rest, b, b, alpha,
                         beta, info);
    };
    product(A + below, X + d, X + below, 1.0, 0.0);
    product(X + below, A + d, A + below, -1.0, 1.0);
    product(A + below, X + d, X + below, 1.0, 1.0);
    hipLaunchKernelGGL((k_chol_tile<true, true>), tiles(rest, rest), dim3(256), 0, s, X + below, X + below,
                       A + below + b, n, rest, b, rest, -1.0, 1.0, info);
  }
}

void launch_chol_inv(double* A, int n, int* info, double* X, hipStream_t s) {
  if (n <= CBN) {
    hipLaunchKernelGGL(k_chol_block, dim3(1), dim3(CNT), 0, s, A, n, n, 0, info, X, n, 0);
    return;
  }
  launch_cholesky(A, n, info, X, s);
  // block row I of X: Y_IJ = sum_K L_IK X_KJ into A, X_IJ = -X_II Y_IJ, and one
  // correction: Y_IJ += L_II X_IJ, X_IJ -= X_II Y_IJ
  for (int i0 = CBN; i0 < n; i0 += CBN) {
    const int b = n - i0 < CBN ? n - i0 : CBN;
    const int64_t row = int64_t(i0) * n;
    const auto product = [&](const double* S, const double* B, double* C, int K, double alpha, double beta) {
      hipLaunchKernelGGL((k_chol_tile<false, false>), tiles(b, i0), dim3(256), 0, s, S, B, C, n, b, K, i0, alpha, beta,
                         info);
    };
    product(X + row, X, A + row, i0, 1.0, 0.0);
    product(X + row + i0, A + row, X + row, b, -1.0, 0.0);
    product(A + row + i0, X + row, A + row, b, 1.0, 1.0);
    product(X + row + i0, A + row, X + row, b, -1.0, 1.0);
  }
}

}  // namespace ace

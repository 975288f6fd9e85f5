// Small dense kernels around the ACE build and the localization:
//   * symmetrization, trace and sign flip of M (Appendix A: -M = L L^T);
//   * the column-pivoted QR pivot search of the SCDM localization;
//   * screening-pair compaction; pair-energy reduction; conversions.
#include <hip/hip_runtime.h>
#include <cstdint>
#include "ace_internal.h"
#include "tri_pairs.h"

namespace ace {

// ---------------------------------------------------------------- M handling
// Msym = (M + M^T)/2 -> out (nullable); negM = -Msym; ex = trace(M).
__global__ void k_symmetrize(const double* __restrict__ M, int n, double* __restrict__ out,
                             double* __restrict__ negM, double* __restrict__ ex, double* __restrict__ asym) {
  __shared__ double red[2][256];
  double tr = 0.0, am = 0.0;
  for (int e = threadIdx.x; e < n * n; e += blockDim.x) {
    const int i = e / n, j = e % n;
    const double a = M[e], b = M[j * n + i];
    const double v = 0.5 * (a + b);
    if (out) out[e] = v;
    negM[e] = -v;
    if (i == j) tr += a;
    const double d = fabs(a - b);
    am = d > am ? d : am;
  }
  red[0][threadIdx.x] = tr;
  red[1][threadIdx.x] = am;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      red[0][threadIdx.x] += red[0][threadIdx.x + s];
      red[1][threadIdx.x] = fmax(red[1][threadIdx.x], red[1][threadIdx.x + s]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    if (ex) ex[0] = red[0][0];
    if (asym) asym[0] = red[1][0];
  }
}


// ---------------------------------------------------------------- SCDM pivot search
// Residual column norms res[r] = sum_i A[i][r]^2, A = psi [n][ng].
__global__ void k_colnorm(const double* __restrict__ A, int n, int64_t ng, double* __restrict__ res) {
  for (int64_t r = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; r < ng; r += int64_t(gridDim.x) * blockDim.x) {
    double s = 0.0;
    for (int i = 0; i < n; ++i) {
      const double a = A[int64_t(i) * ng + r];
      s += a * a;
    }
    res[r] = s;
  }
}

constexpr int TOPK = 8;

// Is (v, i) ranked before (w, j)?  Larger value first; ties to smaller index.
__device__ __forceinline__ bool ranks_before(double v, int64_t i, double w, int64_t j) {
  return v > w || (v == w && i < j);
}

template <int NT>
__device__ void block_topk(double (&tv)[TOPK], int64_t (&ti)[TOPK], double* outv, int64_t* outi) {
  // repeated block-wide extraction of the best remaining head
  __shared__ double sv[NT / 64];
  __shared__ int64_t si[NT / 64];
  __shared__ int st[NT / 64];
  int head = 0;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int round = 0; round < TOPK; ++round) {
    double v = head < TOPK ? tv[0] : -INFINITY;
    int64_t idx = head < TOPK ? ti[0] : INT64_MAX;
    // (tv[0], ti[0]) always holds the current head: the list is shifted on pop
    int who = threadIdx.x;
    for (int off = 32; off > 0; off >>= 1) {
      const double ov = __shfl_down(v, off, 64);
      const int64_t oi = __shfl_down(idx, off, 64);
      const int ow = __shfl_down(who, off, 64);
      if (ranks_before(ov, oi, v, idx)) { v = ov; idx = oi; who = ow; }
    }
    if (lane == 0) { sv[wv] = v; si[wv] = idx; st[wv] = who; }
    __syncthreads();
    if (threadIdx.x == 0) {
      double bv = sv[0]; int64_t bi = si[0]; int bw = st[0];
      for (int w = 1; w < NT / 64; ++w)
        if (ranks_before(sv[w], si[w], bv, bi)) { bv = sv[w]; bi = si[w]; bw = st[w]; }
      outv[round] = bv; outi[round] = bi;
      st[0] = bw;
    }
    __syncthreads();
    const int winner = st[0];
    __syncthreads();
    if (threadIdx.x == winner) {
#pragma unroll
      for (int q = 0; q < TOPK - 1; ++q) { tv[q] = tv[q + 1]; ti[q] = ti[q + 1]; }
      tv[TOPK - 1] = -INFINITY; ti[TOPK - 1] = INT64_MAX;
      ++head;
    }
  }
}

__device__ __forceinline__ void topk_insert(double (&tv)[TOPK], int64_t (&ti)[TOPK], double v, int64_t i) {
  if (!ranks_before(v, i, tv[TOPK - 1], ti[TOPK - 1])) return;
  tv[TOPK - 1] = v; ti[TOPK - 1] = i;
#pragma unroll
  for (int q = TOPK - 1; q > 0; --q) {
    if (ranks_before(tv[q], ti[q], tv[q - 1], ti[q - 1])) {
      const double a = tv[q]; tv[q] = tv[q - 1]; tv[q - 1] = a;
      const int64_t b = ti[q]; ti[q] = ti[q - 1]; ti[q - 1] = b;
    }
  }
}

// One pivot step, bulk part: ell[r] = q . A[:, r]; res[r] -= ell^2 (if q given);
// then per-block top-8 of res into pv/pi [block][8].  A is [n][ng]: either
// the orbitals themselves or a compact pool of candidate columns.  A set stop
// flag turns the launch into a no-op.
template <int NT>
__global__ __launch_bounds__(NT) void k_qrcp_update(const double* __restrict__ A, int n, int64_t ng,
                                                    const double* __restrict__ q, double* __restrict__ res,
                                                    double* __restrict__ pv, int64_t* __restrict__ pi,
                                                    const int* __restrict__ stop) {
  if (stop && *stop) return;
  __shared__ double qs[1024];
  const bool upd = q != nullptr;
  if (upd)
    for (int i = threadIdx.x; i < n; i += NT) qs[i] = q[i];
  __syncthreads();
  double tv[TOPK];
  int64_t ti[TOPK];
#pragma unroll
  for (int t = 0; t < TOPK; ++t) { tv[t] = -INFINITY; ti[t] = INT64_MAX; }
  for (int64_t r = blockIdx.x * int64_t(NT) + threadIdx.x; r < ng; r += int64_t(gridDim.x) * NT) {
    double v = res[r];
    if (upd) {
      double l = 0.0;
      for (int i = 0; i < n; ++i) l += qs[i] * A[int64_t(i) * ng + r];
      v -= l * l;
      res[r] = v;
    }
    topk_insert(tv, ti, v, r);
  }
  block_topk<NT>(tv, ti, pv + blockIdx.x * TOPK, pi + blockIdx.x * TOPK);
}

// One pivot step, selection part (single workgroup of NT threads):
// merge block candidates -> global top-8; recompute their residuals by
// explicit double projection against Q[0..k); pick the best (ties: smaller
// column index); append q_k = residual / |residual| to Q; record the pivot and
// retire the column (res = -1).
//
// k is read from and advanced in device memory.  With a candidate pool
// (pool != nullptr, columns sorted by grid index), the pick is accepted only
// if its exact residual is at least t_out, an upper bound of every residual
// outside the pool; otherwise the stop flag is raised and the host refreshes
// the pool.  A raised stop flag turns the launch into a no-op.
template <int NT>
__global__ __launch_bounds__(NT) void k_qrcp_select(const double* __restrict__ A, int n, int64_t ng,
                                                    int* __restrict__ kdev, const double* __restrict__ pv,
                                                    const int64_t* __restrict__ pi, int nblk, double* __restrict__ Q,
                                                    double* __restrict__ res, int32_t* __restrict__ piv,
                                                    double* __restrict__ qout, const int32_t* __restrict__ pool,
                                                    const double* __restrict__ t_out, int* __restrict__ stop) {
  if (*stop) return;
  __shared__ double cv[TOPK];
  __shared__ int64_t ci[TOPK];
  __shared__ double vec[TOPK][512];
  __shared__ double dots[TOPK][512];
  __shared__ double part[TOPK * NT];
  constexpr int QCH = 4096;
  __shared__ double Qs[QCH];
  __shared__ double r2[TOPK];
  __shared__ int best, accept;
  const int k = *kdev;
  {
    double tv[TOPK];
    int64_t ti[TOPK];
#pragma unroll
    for (int t = 0; t < TOPK; ++t) { tv[t] = -INFINITY; ti[t] = INT64_MAX; }
    for (int e = threadIdx.x; e < nblk * TOPK; e += NT) topk_insert(tv, ti, pv[e], pi[e]);
    block_topk<NT>(tv, ti, cv, ci);
  }
  __syncthreads();
  // valid candidates: real columns that are not retired (res = -1)
  int nc = 0;
  for (int t = 0; t < TOPK; ++t)
    if (ci[t] != INT64_MAX && ci[t] < ng && cv[t] > -0.5) nc = t + 1;
  if (nc == 0) {
    if (threadIdx.x == 0) *stop = 1;
    return;
  }
  for (int e = threadIdx.x; e < TOPK * n; e += NT) {
    const int c = e / n, i = e % n;
    vec[c][i] = c < nc ? A[int64_t(i) * ng + ci[c]] : 0.0;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  constexpr int NW = NT / 64;
  // Q is read in chunks of mc rows staged through LDS (coalesced bulk loads)
  const int mc = QCH / n;
  const int G = NT / n;
  const int g = threadIdx.x / n, gi = threadIdx.x % n;
  for (int pass = 0; pass < 2; ++pass) {
    // dots[c][m] = Q[m] . vec[c]: one wave per row, lanes across i
    for (int m0 = 0; m0 < k; m0 += mc) {
      const int rows = (k - m0 < mc) ? k - m0 : mc;
      for (int e = threadIdx.x; e < rows * n; e += NT) Qs[e] = Q[int64_t(m0) * n + e];
      __syncthreads();
      for (int r = wv; r < rows; r += NW) {
        double acc[TOPK];
#pragma unroll
        for (int c = 0; c < TOPK; ++c) acc[c] = 0.0;
        for (int i = lane; i < n; i += 64) {
          const double qv = Qs[r * n + i];
#pragma unroll
          for (int c = 0; c < TOPK; ++c) acc[c] += qv * vec[c][i];
        }
#pragma unroll
        for (int c = 0; c < TOPK; ++c) {
          double v = acc[c];
          for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
          if (lane == 0) dots[c][m0 + r] = v;
        }
      }
      __syncthreads();
    }
    // vec[c][i] -= sum_m dots[c][m] Q[m][i]: G thread groups split the rows,
    // their partial sums meet in LDS
    double acc[TOPK];
#pragma unroll
    for (int c = 0; c < TOPK; ++c) acc[c] = 0.0;
    for (int m0 = 0; m0 < k; m0 += mc) {
      const int rows = (k - m0 < mc) ? k - m0 : mc;
      for (int e = threadIdx.x; e < rows * n; e += NT) Qs[e] = Q[int64_t(m0) * n + e];
      __syncthreads();
      if (g < G)
        for (int r = g; r < rows; r += G) {
          const double qv = Qs[r * n + gi];
#pragma unroll
          for (int c = 0; c < TOPK; ++c) acc[c] += dots[c][m0 + r] * qv;
        }
      __syncthreads();
    }
    if (g < G) {
#pragma unroll
      for (int c = 0; c < TOPK; ++c) part[(g * TOPK + c) * n + gi] = acc[c];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < TOPK * n; e += NT) {
      const int c = e / n, ii = e % n;
      double sum = 0.0;
      for (int gg = 0; gg < G; ++gg) sum += part[(gg * TOPK + c) * n + ii];
      vec[c][ii] -= sum;
    }
    __syncthreads();
  }
  // squared residual norms: one wave per candidate
  for (int c = wv; c < TOPK; c += NW) {
    double v = 0.0;
    for (int i = lane; i < n; i += 64) v += vec[c][i] * vec[c][i];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if (lane == 0) r2[c] = v;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int b = 0;
    for (int c = 1; c < nc; ++c)
      if (ranks_before(r2[c], ci[c], r2[b], ci[b])) b = c;
    best = b;
    const bool ok = (t_out == nullptr) || (r2[b] >= *t_out);
    accept = ok ? 1 : 0;
    if (ok) {
      piv[k] = pool ? pool[ci[b]] : int32_t(ci[b]);
      res[ci[b]] = -1.0;
    } else {
      *stop = 1;
    }
  }
  __syncthreads();
  if (!accept) return;
  const double inv = 1.0 / sqrt(r2[best]);
  for (int i = threadIdx.x; i < n; i += NT) {
    const double v = vec[best][i] * inv;
    Q[int64_t(k) * n + i] = v;
    qout[i] = v;
  }
  __syncthreads();
  if (threadIdx.x == 0) *kdev = k + 1;
}

// ---------------------------------------------------------------- pool steps on explicit residuals
// On a candidate pool the residual columns are kept explicitly,
// R = (I - Q^T Q) A_pool ([n][P], row-major), so every step's norms are exact
// and no re-ranking against Q is needed: with the new direction q,
// l_c = q . R[:,c], R[:,c] -= q l_c, res_c = |R[:,c]|^2.

// Best (value, index) of the block, ties to the smaller index; result in
// out[0], idx_out[0] (shared) for every thread after the call.
template <int NT>
__device__ void block_top1(double v, int64_t idx, double* outv, int64_t* outi) {
  __shared__ double sv[NT / 64];
  __shared__ int64_t si[NT / 64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int off = 32; off > 0; off >>= 1) {
    const double ov = __shfl_down(v, off, 64);
    const int64_t oi = __shfl_down(idx, off, 64);
    if (ranks_before(ov, oi, v, idx)) { v = ov; idx = oi; }
  }
  if (lane == 0) { sv[wv] = v; si[wv] = idx; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double bv = sv[0];
    int64_t bi = si[0];
    for (int w = 1; w < NT / 64; ++w)
      if (ranks_before(sv[w], si[w], bv, bi)) { bv = sv[w]; bi = si[w]; }
    *outv = bv;
    *outi = bi;
  }
  __syncthreads();
}

// One update of the pool residuals (q == nullptr: only the norms).  A block
// covers CW columns with NT/CW row groups (a wave reads CW-column row
// segments); partial sums meet in LDS in a fixed order.  Retired columns
// (res = -1) are skipped.  Writes the block's best live column to
// pv[blockIdx.x], pi[blockIdx.x].
template <int NT, int CW>
__global__ __launch_bounds__(NT) void k_qrcp_update_r(double* __restrict__ R, int n, int P,
                                                      const double* __restrict__ q, double* __restrict__ res,
                                                      double* __restrict__ pv, int64_t* __restrict__ pi,
                                                      const int* __restrict__ stop) {
  if (*stop) return;
  constexpr int RG = NT / CW;
  __shared__ double qs[1024];
  __shared__ double red[RG][CW];
  __shared__ double bv;
  __shared__ int64_t bi;
  const int lane = threadIdx.x % CW, g = threadIdx.x / CW;
  const int c = blockIdx.x * CW + lane;
  const bool upd = q != nullptr;
  if (upd)
    for (int i = threadIdx.x; i < n; i += NT) qs[i] = q[i];
  const bool live = c < P && res[c] > -0.5;
  __syncthreads();
  double* col = R + c;
  double l = 0.0;
  if (upd) {
    if (live) {
      double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
      int i = g;
      for (; i + 3 * RG < n; i += 4 * RG) {
        a0 += qs[i] * col[int64_t(i) * P];
        a1 += qs[i + RG] * col[int64_t(i + RG) * P];
        a2 += qs[i + 2 * RG] * col[int64_t(i + 2 * RG) * P];
        a3 += qs[i + 3 * RG] * col[int64_t(i + 3 * RG) * P];
      }
      for (; i < n; i += RG) a0 += qs[i] * col[int64_t(i) * P];
      l = (a0 + a1) + (a2 + a3);
    }
    red[g][lane] = l;
    __syncthreads();
    l = 0.0;
#pragma unroll
    for (int h = 0; h < RG; ++h) l += red[h][lane];
    __syncthreads();
  }
  double v = 0.0;
  if (live) {
    double v0 = 0.0, v1 = 0.0;
    int i = g;
    for (; i + RG < n; i += 2 * RG) {
      double x0 = col[int64_t(i) * P], x1 = col[int64_t(i + RG) * P];
      if (upd) {
        x0 -= qs[i] * l;
        x1 -= qs[i + RG] * l;
        col[int64_t(i) * P] = x0;
        col[int64_t(i + RG) * P] = x1;
      }
      v0 += x0 * x0;
      v1 += x1 * x1;
    }
    for (; i < n; i += RG) {
      double x = col[int64_t(i) * P];
      if (upd) {
        x -= qs[i] * l;
        col[int64_t(i) * P] = x;
      }
      v0 += x * x;
    }
    v = v0 + v1;
  }
  red[g][lane] = v;
  __syncthreads();
  double cand = -INFINITY;
  int64_t cidx = INT64_MAX;
  if (g == 0) {
    v = 0.0;
#pragma unroll
    for (int h = 0; h < RG; ++h) v += red[h][lane];
    if (live) {
      res[c] = v;
      cand = v;
      cidx = c;
    }
  }
  block_top1<NT>(cand, cidx, &bv, &bi);
  if (threadIdx.x == 0) {
    pv[blockIdx.x] = bv;
    pi[blockIdx.x] = bi;
  }
}

// Selection on the pool (single workgroup): the best block candidate is the
// best live column; its norm is recomputed, certified against t_out (an upper
// bound of every residual outside the pool), and q_k = R[:,b] / |R[:,b]| is
// appended to Q.  A failed certification or an exhausted pool raises the
// stop flag, after which the queued steps are no-ops, and leaves in *t_next the
// residual down to which the bounds are refreshed for the next pool: half the
// best one of this pool (0 when it is exhausted).
constexpr double REFRESH_BELOW = 0.5;
template <int NT>
__global__ __launch_bounds__(NT) void k_qrcp_select_r(const double* __restrict__ R, int n, int P,
                                                      int* __restrict__ kdev, const double* __restrict__ pv,
                                                      const int64_t* __restrict__ pi, int nblk,
                                                      double* __restrict__ Q, double* __restrict__ res,
                                                      int32_t* __restrict__ piv, double* __restrict__ qout,
                                                      const int32_t* __restrict__ pool,
                                                      const double* __restrict__ t_out, int* __restrict__ stop,
                                                      double* __restrict__ t_next) {
  if (*stop) return;
  __shared__ double bv;
  __shared__ int64_t bi;
  __shared__ double r2s[NT / 64];
  __shared__ int accept;
  const int k = *kdev;
  {
    double v = -INFINITY;
    int64_t idx = INT64_MAX;
    for (int e = threadIdx.x; e < nblk; e += NT)
      if (ranks_before(pv[e], pi[e], v, idx)) { v = pv[e]; idx = pi[e]; }
    block_top1<NT>(v, idx, &bv, &bi);
  }
  const int64_t b = bi;
  if (b < 0 || b >= P) {
    if (threadIdx.x == 0) {
      *stop = 1;
      *t_next = 0.0;
    }
    return;
  }
  double v = 0.0;
  for (int i = threadIdx.x; i < n; i += NT) {
    const double x = R[int64_t(i) * P + b];
    v += x * x;
  }
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  if ((threadIdx.x & 63) == 0) r2s[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double r2 = 0.0;
    for (int w = 0; w < NT / 64; ++w) r2 += r2s[w];
    r2s[0] = r2;
    const bool ok = r2 > 0.0 && (t_out == nullptr || r2 >= *t_out);
    accept = ok ? 1 : 0;
    if (ok) {
      piv[k] = pool[b];
      res[b] = -1.0;
    } else {
      *stop = 1;
      *t_next = r2 > 0.0 ? REFRESH_BELOW * r2 : 0.0;
    }
  }
  __syncthreads();
  if (!accept) return;
  const double inv = 1.0 / sqrt(r2s[0]);
  for (int i = threadIdx.x; i < n; i += NT) {
    const double x = R[int64_t(i) * P + b] * inv;
    Q[int64_t(k) * n + i] = x;
    qout[i] = x;
  }
  __syncthreads();
  if (threadIdx.x == 0) *kdev = k + 1;
}

// One pool step in one launch: every block repeats the selection (the best
// of the previous step's block candidates pv_in/pi_in, its norm recomputed
// and certified against t_out, q = R[:,b] / |R[:,b]| in LDS) with the same
// reductions as k_qrcp_select_r, so all blocks hold the same q; block 0
// alone appends q to Q, records the pivot, retires the column and advances
// the step counter.  Then each block updates its columns as
// k_qrcp_update_r does and writes its best live column to pv_out/pi_out
// (candidates double buffered: blocks of this launch still read pv_in).  The
// pivot column itself is left untouched, so the blocks that read it are not
// racing with its owner.  A failed certification or an exhausted pool
// raises the stop flag (block 0), and every block returns.
template <int NT, int CW, int MP>
__global__ __launch_bounds__(NT) void k_qrcp_step_r(double* __restrict__ R, int n, int P, int* __restrict__ kdev,
                                                    const double* __restrict__ pv_in,
                                                    const int64_t* __restrict__ pi_in, int nblk,
                                                    double* __restrict__ Q, double* __restrict__ res,
                                                    int32_t* __restrict__ piv, const int32_t* __restrict__ pool,
                                                    const double* __restrict__ t_out, int* __restrict__ stop,
                                                    double* __restrict__ pv_out, int64_t* __restrict__ pi_out,
                                                    double* __restrict__ t_next) {
  constexpr int RG = NT / CW;
  __shared__ double qs[1024];
  __shared__ double red[RG][CW];
  __shared__ double r2s[NT / 64];
  __shared__ double bv;
  __shared__ int64_t bi;
  // The block's residual tile (its CW columns, rows g + m RG) and their
  // bounds are loaded first: no block writes them before this block does,
  // so the loads stay in flight through the selection.
  const int lane = threadIdx.x % CW, g = threadIdx.x / CW;
  const int c = blockIdx.x * CW + lane;
  const bool inb = c < P;
  const int nm = g < n ? (n - g + RG - 1) / RG : 0;  // rows of this thread
  double xr[MP];
#pragma unroll
  for (int m = 0; m < MP; ++m)
    if (inb && m < nm) xr[m] = R[int64_t(g + m * RG) * P + c];
  const double rc = inb ? res[c] : -1.0;
  if (*stop) return;
  // selection, as k_qrcp_select_r
  {
    double v = -INFINITY;
    int64_t idx = INT64_MAX;
    for (int e = threadIdx.x; e < nblk; e += NT)
      if (ranks_before(pv_in[e], pi_in[e], v, idx)) { v = pv_in[e]; idx = pi_in[e]; }
    block_top1<NT>(v, idx, &bv, &bi);
  }
  const int64_t b = bi;
  if (b < 0 || b >= P) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      *stop = 1;
      *t_next = 0.0;
    }
    return;
  }
  {
    double v = 0.0;
    for (int i = threadIdx.x; i < n; i += NT) {
      const double x = R[int64_t(i) * P + b];
      v += x * x;
    }
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if ((threadIdx.x & 63) == 0) r2s[threadIdx.x >> 6] = v;
  }
  __syncthreads();
  double r2 = 0.0;
  for (int w = 0; w < NT / 64; ++w) r2 += r2s[w];
  const bool ok = r2 > 0.0 && (t_out == nullptr || r2 >= *t_out);
  if (!ok) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      *stop = 1;
      *t_next = r2 > 0.0 ? REFRESH_BELOW * r2 : 0.0;
    }
    return;
  }
  const double inv = 1.0 / sqrt(r2);
  for (int i = threadIdx.x; i < n; i += NT) qs[i] = R[int64_t(i) * P + b] * inv;
  __syncthreads();
  if (blockIdx.x == 0) {
    const int k = *kdev;
    for (int i = threadIdx.x; i < n; i += NT) Q[int64_t(k) * n + i] = qs[i];
    if (threadIdx.x == 0) {
      piv[k] = pool[b];
      res[b] = -1.0;
      *kdev = k + 1;
    }
  }
  // update, as k_qrcp_update_r with q (the same sums in the same order)
  const bool live = inb && c != b && rc > -0.5;
  double* col = R + c;
  double l = 0.0;
  if (live) {
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    int m0 = 0;
#pragma unroll
    for (int m = 0; m + 3 < MP; m += 4)
      if (m + 3 < nm) {
        a0 += qs[g + m * RG] * xr[m];
        a1 += qs[g + (m + 1) * RG] * xr[m + 1];
        a2 += qs[g + (m + 2) * RG] * xr[m + 2];
        a3 += qs[g + (m + 3) * RG] * xr[m + 3];
        m0 = m + 4;
      }
#pragma unroll
    for (int m = 0; m < MP; ++m)
      if (m >= m0 && m < nm) a0 += qs[g + m * RG] * xr[m];
    l = (a0 + a1) + (a2 + a3);
  }
  red[g][lane] = l;
  __syncthreads();
  l = 0.0;
#pragma unroll
  for (int h = 0; h < RG; ++h) l += red[h][lane];
  __syncthreads();
  double v = 0.0;
  if (live) {
    double v0 = 0.0, v1 = 0.0;
    int m0 = 0;
#pragma unroll
    for (int m = 0; m + 1 < MP; m += 2)
      if (m + 1 < nm) {
        double x0 = xr[m], x1 = xr[m + 1];
        x0 -= qs[g + m * RG] * l;
        x1 -= qs[g + (m + 1) * RG] * l;
        col[int64_t(g + m * RG) * P] = x0;
        col[int64_t(g + (m + 1) * RG) * P] = x1;
        v0 += x0 * x0;
        v1 += x1 * x1;
        m0 = m + 2;
      }
#pragma unroll
    for (int m = 0; m < MP; ++m)
      if (m >= m0 && m < nm) {
        double x = xr[m];
        x -= qs[g + m * RG] * l;
        col[int64_t(g + m * RG) * P] = x;
        v0 += x * x;
      }
    v = v0 + v1;
  }
  red[g][lane] = v;
  __syncthreads();
  double cand = -INFINITY;
  int64_t cidx = INT64_MAX;
  if (g == 0) {
    v = 0.0;
#pragma unroll
    for (int h = 0; h < RG; ++h) v += red[h][lane];
    if (live) {
      res[c] = v;
      cand = v;
      cidx = c;
    }
  }
  block_top1<NT>(cand, cidx, &bv, &bi);
  if (threadIdx.x == 0) {
    pv_out[blockIdx.x] = bv;
    pi_out[blockIdx.x] = bi;
  }
}

// a += b (elementwise)
__global__ void k_add_inplace(double* __restrict__ a, const double* __restrict__ b, int64_t cnt) {
  for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < cnt; e += int64_t(gridDim.x) * blockDim.x)
    a[e] += b[e];
}

// ---------------------------------------------------------------- candidate pool
// The pool holds every column whose residual bound is at least a threshold t
// picked from a histogram of the top 14 bits of the (positive) residuals, so
// that the pool has at most pmax columns.  t_out = the largest residual
// below t bounds every column left out.
constexpr int HBIN = 1 << 14;

__device__ __forceinline__ int res_bin(double v) { return int(__double_as_longlong(v) >> 49); }

__global__ __launch_bounds__(256) void k_res_hist(const double* __restrict__ res, int64_t ng,
                                                  unsigned* __restrict__ hist) {
  __shared__ unsigned h[HBIN];
  for (int i = threadIdx.x; i < HBIN; i += 256) h[i] = 0u;
  __syncthreads();
  for (int64_t r = blockIdx.x * int64_t(256) + threadIdx.x; r < ng; r += int64_t(gridDim.x) * 256) {
    const double v = res[r];
    if (v > 0.0) atomicAdd(&h[res_bin(v)], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < HBIN; i += 256)
    if (h[i]) atomicAdd(&hist[i], h[i]);
}

// Lowest bin b such that the columns in bins >= b number at most pmax;
// returns the lower edge of bin b (as a double) in every thread of 1024.
__device__ __forceinline__ double pool_edge(const unsigned* __restrict__ hist, int pmax) {
  constexpr int SEG = HBIN / 1024;
  __shared__ unsigned long long above[1024];
  __shared__ int tb;
  unsigned long long seg = 0;
  for (int b = 0; b < SEG; ++b) seg += hist[threadIdx.x * SEG + b];
  above[threadIdx.x] = seg;
  if (threadIdx.x == 0) tb = 0;
  __syncthreads();
  // inclusive suffix sum over segments
  for (int off = 1; off < 1024; off <<= 1) {
    unsigned long long v = (threadIdx.x + off < 1024) ? above[threadIdx.x + off] : 0ull;
    __syncthreads();
    above[threadIdx.x] += v;
    __syncthreads();
  }
  const unsigned long long incl = above[threadIdx.x];
  const unsigned long long excl = incl - seg;  // columns in higher segments
  if (excl <= (unsigned long long)pmax && incl > (unsigned long long)pmax) {
    unsigned long long c = excl;
    int pick = threadIdx.x * SEG + SEG;
    for (int b = threadIdx.x * SEG + SEG - 1; b >= threadIdx.x * SEG; --b) {
      if (c + hist[b] > (unsigned long long)pmax) break;
      c += hist[b];
      pick = b;
    }
    tb = pick;
  }
  __syncthreads();
  // tb == HBIN: not even the top bin fits; an infinite threshold empties the pool
  return tb >= HBIN ? INFINITY : __longlong_as_double((long long)tb << 49);
}

__global__ __launch_bounds__(1024) void k_pool_threshold(const unsigned* __restrict__ hist, int pmax,
                                                         double* __restrict__ t) {
  const double e = pool_edge(hist, pmax);
  if (threadIdx.x == 0) t[0] = e;
}

// The whole pool of a small grid in one workgroup: histogram, threshold, count
// and ordered list, as the five kernels of larger grids (whose launches took
// 33 us at 24^3, this 15).  Clears iv[1], and iv[0] with first.
// The chunk of a wave is a stretch of columns, so its list positions follow from
// the counts of the waves before it.
constexpr int64_t POOL_SMALL = 65536;
__global__ __launch_bounds__(1024) void k_pool_small(const double* __restrict__ res, int ng, int pmax, int first,
                                                     double* __restrict__ t, int* __restrict__ iv,
                                                     double* __restrict__ t_out, int32_t* __restrict__ pool,
                                                     double* __restrict__ pres) {
  __shared__ unsigned hist[HBIN];
  __shared__ int wcnt[16];
  __shared__ double wmax[16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int i = tid; i < HBIN; i += 1024) hist[i] = 0u;
  __syncthreads();
#pragma unroll 4
  for (int r = tid; r < ng; r += 1024) {
    const double v = res[r];
    if (v > 0.0) atomicAdd(&hist[res_bin(v)], 1u);
  }
  __syncthreads();
  const double th = pool_edge(hist, pmax);
  const int len = (ng + 1023) / 1024 * 64, r0 = wv * len, r1 = r0 + len < ng ? r0 + len : ng;
  int c = 0;
  double m = 0.0;
#pragma unroll 4
  for (int r = r0 + lane; r < r1; r += 64) {
    const double v = res[r];
    if (v >= th && v > 0.0) ++c;
    else if (v > 0.0 && v > m) m = v;
  }
  for (int off = 32; off > 0; off >>= 1) {
    c += __shfl_down(c, off, 64);
    m = fmax(m, __shfl_down(m, off, 64));
  }
  if (lane == 0) {
    wcnt[wv] = c;
    wmax[wv] = m;
  }
  __syncthreads();
  int off = 0, total = 0;
  for (int w = 0; w < 16; ++w) {
    if (w < wv) off += wcnt[w];
    total += wcnt[w];
  }
  if (tid == 0) {
    for (int w = 0; w < 16; ++w) m = fmax(m, wmax[w]);
    t[0] = th;
    t_out[0] = m;
    if (first) iv[0] = 0;
    iv[1] = 0;
    iv[2] = total;
  }
  if (total > pmax) return;  // (the caller then takes the whole grid)
#pragma unroll 4
  for (int g = r0; g < r1; g += 64) {
    const int r = g + lane;
    const double v = r < r1 ? res[r] : 0.0;
    const bool keep = v >= th && v > 0.0;
    const unsigned long long bal = __ballot(keep);
    if (keep) {
      const int p = off + __popcll(bal & ((1ull << lane) - 1ull));
      pool[p] = r;
      pres[p] = v;
    }
    off += __popcll(bal);
  }
}

// Per block (contiguous chunk of columns): count of res >= t, max of 0 < res < t.
__global__ __launch_bounds__(256) void k_pool_count(const double* __restrict__ res, int64_t ng, int64_t chunk,
                                                    const double* __restrict__ t, int64_t* __restrict__ cnt,
                                                    double* __restrict__ tmax) {
  __shared__ int64_t sc[256];
  __shared__ double sm[256];
  const double th = t[0];
  const int64_t r0 = int64_t(blockIdx.x) * chunk;
  const int64_t r1 = (r0 + chunk < ng) ? r0 + chunk : ng;
  int64_t c = 0;
  double m = 0.0;
  for (int64_t r = r0 + threadIdx.x; r < r1; r += 256) {
    const double v = res[r];
    if (v >= th && v > 0.0) ++c;
    else if (v > 0.0 && v > m) m = v;
  }
  sc[threadIdx.x] = c;
  sm[threadIdx.x] = m;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (threadIdx.x < h) {
      sc[threadIdx.x] += sc[threadIdx.x + h];
      sm[threadIdx.x] = fmax(sm[threadIdx.x], sm[threadIdx.x + h]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) { cnt[blockIdx.x] = sc[0]; tmax[blockIdx.x] = sm[0]; }
}

// Exclusive scan of the block counts (in place), total count and t_out.
__global__ __launch_bounds__(1024) void k_pool_scan(int64_t* __restrict__ cnt, const double* __restrict__ tmax,
                                                    int nblk, int* __restrict__ total, double* __restrict__ t_out) {
  __shared__ int64_t s[1024];
  __shared__ double m[1024];
  __shared__ int64_t carry;
  if (threadIdx.x == 0) carry = 0;
  double mx = 0.0;
  for (int b = threadIdx.x; b < nblk; b += 1024) mx = fmax(mx, tmax[b]);
  m[threadIdx.x] = mx;
  __syncthreads();
  for (int h = 512; h > 0; h >>= 1) {
    if (threadIdx.x < h) m[threadIdx.x] = fmax(m[threadIdx.x], m[threadIdx.x + h]);
    __syncthreads();
  }
  for (int base = 0; base < nblk; base += 1024) {
    const int b = base + threadIdx.x;
    const int64_t v = b < nblk ? cnt[b] : 0;
    s[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
      const int64_t u = threadIdx.x >= off ? s[threadIdx.x - off] : 0;
      __syncthreads();
      s[threadIdx.x] += u;
      __syncthreads();
    }
    if (b < nblk) cnt[b] = carry + s[threadIdx.x] - v;
    __syncthreads();
    if (threadIdx.x == 0) carry += s[1023];
    __syncthreads();
  }
  if (threadIdx.x == 0) { total[0] = int(carry); t_out[0] = m[0]; }
}

// Ordered compaction: pool[off..] = columns with res >= t, by increasing index.
__global__ __launch_bounds__(256) void k_pool_write(const double* __restrict__ res, int64_t ng, int64_t chunk,
                                                    const double* __restrict__ t, const int64_t* __restrict__ off,
                                                    int32_t* __restrict__ pool, double* __restrict__ pres) {
  __shared__ int wsum[4];
  __shared__ int64_t base;
  const double th = t[0];
  const int64_t r0 = int64_t(blockIdx.x) * chunk;
  const int64_t r1 = (r0 + chunk < ng) ? r0 + chunk : ng;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (threadIdx.x == 0) base = off[blockIdx.x];
  __syncthreads();
  for (int64_t c0 = r0; c0 < r1; c0 += 256) {
    const int64_t r = c0 + threadIdx.x;
    double v = 0.0;
    bool keep = false;
    if (r < r1) {
      v = res[r];
      keep = v >= th && v > 0.0;
    }
    const unsigned long long bal = __ballot(keep);
    const int before = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) wsum[wv] = __popcll(bal);
    __syncthreads();
    int64_t o = base;
    for (int w = 0; w < wv; ++w) o += wsum[w];
    if (keep) {
      pool[o + before] = int32_t(r);
      if (pres) pres[o + before] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) base += wsum[0] + wsum[1] + wsum[2] + wsum[3];
    __syncthreads();
  }
}

// Apool[i][p] = A[i][pool[p]]
__global__ void k_pool_gather(const double* __restrict__ A, int n, int64_t ng, const int32_t* __restrict__ pool,
                              int np, double* __restrict__ Apool) {
  for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < int64_t(n) * np;
       e += int64_t(gridDim.x) * blockDim.x) {
    const int i = int(e / np), p = int(e % np);
    Apool[e] = A[int64_t(i) * ng + pool[p]];
  }
}

// res[list[p]] = v[p]
__global__ void k_scatter_res(const int32_t* __restrict__ list, int64_t cnt, const double* __restrict__ v,
                              double* __restrict__ res) {
  for (int64_t p = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; p < cnt; p += int64_t(gridDim.x) * blockDim.x)
    res[list[p]] = v[p];
}

__global__ void k_retire(const int32_t* __restrict__ piv, int k, double* __restrict__ res) {
  for (int m = blockIdx.x * blockDim.x + threadIdx.x; m < k; m += gridDim.x * blockDim.x) res[piv[m]] = -1.0;
}

// AC[i][k] = A[i][piv[k]]
__global__ void k_gather_cols(const double* __restrict__ A, int n, int64_t ng, const int32_t* __restrict__ piv,
                              double* __restrict__ AC) {
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n * n; e += gridDim.x * blockDim.x) {
    const int i = e / n, k = e % n;
    AC[e] = A[int64_t(i) * ng + piv[k]];
  }
}

// ---------------------------------------------------------------- screening
// Upper-triangle entries (i <= j) with O_ij >= rho_cut, or i == j, in
// row-major order; writes at most cap pairs and the full count to *count.
__global__ __launch_bounds__(CNT) void k_compact_pairs(const double* __restrict__ O, int n, double rho_cut,
                                                       int64_t cap, int32_t* __restrict__ pairs,
                                                       double* __restrict__ ov, int64_t* __restrict__ count) {
  compact_tri(
      n, [&](int64_t, int i, int j) { return i == j || O[int64_t(i) * n + j] >= rho_cut; },
      [&](int64_t p, int i, int j) {
        if (p < cap) {
          pairs[2 * p] = i;
          pairs[2 * p + 1] = j;
          if (ov) ov[p] = O[int64_t(i) * n + j];
        }
      },
      count);
}

// ---------------------------------------------------------------- pair energies
// e[pair] = -(2 - delta_ij) dV sum_blocks epart; pack p carries pairs pa[p], pb[p].
__global__ void k_pair_energy(const double* __restrict__ epart, int npacks, int nblk, const Pack* __restrict__ packs,
                              const int64_t* __restrict__ pidx, double dV, double* __restrict__ e) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= npacks) return;
  double sa = 0.0, sb = 0.0;
  for (int b = 0; b < nblk; ++b) {
    sa += epart[2 * (int64_t(p) * nblk + b)];
    sb += epart[2 * (int64_t(p) * nblk + b) + 1];
  }
  const Pack pk = packs[p];
  e[pidx[2 * p]] = -(pk.ia == pk.ja ? 1.0 : 2.0) * dV * sa;
  if (pk.jb >= 0) e[pidx[2 * p + 1]] = -(pk.ib == pk.jb ? 1.0 : 2.0) * dV * sb;
}
// out[0] = -sum c^2 over n values: the summed exchange energy of a set of
// functions from their projector coefficients c_ka = <xi_k | x_a>.  One block,
// fixed summation order (deterministic).
__global__ void k_neg_sumsq(const double* __restrict__ c, int64_t n, double* __restrict__ out) {
  __shared__ double red[256];
  double a = 0.0;
  for (int64_t e = threadIdx.x; e < n; e += blockDim.x) a = fma(c[e], c[e], a);
  red[threadIdx.x] = a;
  __syncthreads();
  for (int h = blockDim.x / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = -red[0];
}

// ---------------------------------------------------------------- conversions
__global__ void k_d2f(const double* __restrict__ a, float* __restrict__ b, int64_t n) {
  for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < n; e += int64_t(gridDim.x) * blockDim.x)
    b[e] = float(a[e]);
}
__global__ void k_f2d(const float* __restrict__ a, double* __restrict__ b, int64_t n) {
  for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < n; e += int64_t(gridDim.x) * blockDim.x)
    b[e] = double(a[e]);
}
__global__ void k_nonfinite(const double* __restrict__ a, int64_t n, int* __restrict__ flag) {
  for (int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; e < n; e += int64_t(gridDim.x) * blockDim.x)
    if (!isfinite(a[e])) flag[0] = 1;
}

// ---------------------------------------------------------------- host launchers
static int grid_for(int64_t n, int nt, int cap = 4096) {
  int64_t g = (n + nt - 1) / nt;
  if (g > cap) g = cap;
  if (g < 1) g = 1;
  return int(g);
}

void launch_neg_sumsq(const double* c, int64_t n, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_neg_sumsq, dim3(1), dim3(256), 0, s, c, n, out);
}
void launch_symmetrize(const double* M, int n, double* out, double* negM, double* ex, double* asym, hipStream_t s) {
  hipLaunchKernelGGL(k_symmetrize, dim3(1), dim3(256), 0, s, M, n, out, negM, ex, asym);
}
void launch_colnorm(const double* A, int n, int64_t ng, double* res, hipStream_t s) {
  hipLaunchKernelGGL(k_colnorm, dim3(grid_for(ng, 256)), dim3(256), 0, s, A, n, ng, res);
}
int qrcp_blocks(int64_t ng) { return grid_for(ng, 256, 2048); }
void launch_qrcp_update(const double* A, int n, int64_t ng, const double* q, double* res, double* pv, int64_t* pi,
                        const int* stop, hipStream_t s) {
  hipLaunchKernelGGL(k_qrcp_update<256>, dim3(qrcp_blocks(ng)), dim3(256), 0, s, A, n, ng, q, res, pv, pi, stop);
}
void launch_qrcp_select(const double* A, int n, int64_t ng, int* kdev, const double* pv, const int64_t* pi,
                        int nblk, double* Q, double* res, int32_t* piv, double* qout, const int32_t* pool,
                        const double* t_out, int* stop, hipStream_t s) {
  hipLaunchKernelGGL(k_qrcp_select<512>, dim3(1), dim3(512), 0, s, A, n, ng, kdev, pv, pi, nblk, Q, res, piv, qout,
                     pool, t_out, stop);
}
constexpr int QCW = 16;  // pool columns per update block
int qrcp_pool_blocks(int P) { return (P + QCW - 1) / QCW; }
void launch_qrcp_update_r(double* R, int n, int P, const double* q, double* res, double* pv, int64_t* pi,
                          const int* stop, hipStream_t s) {
  hipLaunchKernelGGL((k_qrcp_update_r<256, QCW>), dim3(qrcp_pool_blocks(P)), dim3(256), 0, s, R, n, P, q, res, pv, pi, stop);
}
void launch_qrcp_select_r(const double* R, int n, int P, int* kdev, const double* pv, const int64_t* pi,
                          double* Q, double* res, int32_t* piv, double* qout, const int32_t* pool,
                          const double* t_out, int* stop, double* t_next, hipStream_t s) {
  hipLaunchKernelGGL(k_qrcp_select_r<256>, dim3(1), dim3(256), 0, s, R, n, P, kdev, pv, pi, qrcp_pool_blocks(P), Q,
                     res, piv, qout, pool, t_out, stop, t_next);
}
void launch_qrcp_step_r(double* R, int n, int P, int* kdev, const double* pv_in, const int64_t* pi_in, double* Q,
                        double* res, int32_t* piv, const int32_t* pool, const double* t_out, int* stop,
                        double* pv_out, int64_t* pi_out, double* t_next, hipStream_t s) {
  // rows per thread of the block's tile: n / (256 / QCW), held in registers
#define QSTEP(MPV)                                                                                                 \
  hipLaunchKernelGGL((k_qrcp_step_r<256, QCW, MPV>), dim3(qrcp_pool_blocks(P)), dim3(256), 0, s, R, n, P, kdev,   \
                     pv_in, pi_in, qrcp_pool_blocks(P), Q, res, piv, pool, t_out, stop, pv_out, pi_out, \
                     t_next)
  constexpr int RG = 256 / QCW;
  if (n <= 8 * RG) QSTEP(8);
  else if (n <= 16 * RG) QSTEP(16);
  else if (n <= 32 * RG) QSTEP(32);
  else QSTEP(64);
#undef QSTEP
}
void launch_add_inplace(double* a, const double* b, int64_t cnt, hipStream_t s) {
  hipLaunchKernelGGL(k_add_inplace, dim3(grid_for(cnt, 256)), dim3(256), 0, s, a, b, cnt);
}
int pool_blocks(int64_t ng) { return grid_for(ng, 4096, 2048); }
void launch_pool_build(const double* res, int64_t ng, int pmax, unsigned* hist, double* t, int64_t* cnt,
                       double* tmax, int* total, double* t_out, hipStream_t s) {
  hipLaunchKernelGGL(k_res_hist, dim3(grid_for(ng, 256, 1024)), dim3(256), 0, s, res, ng, hist);
  hipLaunchKernelGGL(k_pool_threshold, dim3(1), dim3(1024), 0, s, hist, pmax, t);
  launch_count_above(res, ng, t, cnt, tmax, total, t_out, s);
}
bool pool_fits_one(int64_t ng) { return ng <= POOL_SMALL; }
void launch_pool_small(const double* res, int64_t ng, int pmax, bool first, double* t, int* iv, double* t_out,
                       int32_t* pool, double* pres, hipStream_t s) {
  hipLaunchKernelGGL(k_pool_small, dim3(1), dim3(1024), 0, s, res, int(ng), pmax, first ? 1 : 0, t, iv, t_out, pool,
                     pres);
}
void launch_pool_write(const double* res, int64_t ng, const double* t, const int64_t* off, int32_t* pool,
                       double* pres, hipStream_t s) {
  const int nb = pool_blocks(ng);
  const int64_t chunk = (ng + nb - 1) / nb;
  hipLaunchKernelGGL(k_pool_write, dim3(nb), dim3(256), 0, s, res, ng, chunk, t, off, pool, pres);
}
void launch_pool_gather(const double* A, int n, int64_t ng, const int32_t* pool, int np, double* Apool,
                        hipStream_t s) {
  hipLaunchKernelGGL(k_pool_gather, dim3(grid_for(int64_t(n) * np, 256)), dim3(256), 0, s, A, n, ng, pool, np,
                     Apool);
}
void launch_count_above(const double* res, int64_t ng, const double* t, int64_t* cnt, double* tmax, int* total,
                        double* below, hipStream_t s) {
  const int nb = pool_blocks(ng);
  const int64_t chunk = (ng + nb - 1) / nb;
  hipLaunchKernelGGL(k_pool_count, dim3(nb), dim3(256), 0, s, res, ng, chunk, t, cnt, tmax);
  hipLaunchKernelGGL(k_pool_scan, dim3(1), dim3(1024), 0, s, cnt, tmax, nb, total, below);
}
void launch_scatter_res(const int32_t* list, int64_t cnt, const double* v, double* res, hipStream_t s) {
  hipLaunchKernelGGL(k_scatter_res, dim3(grid_for(cnt, 256)), dim3(256), 0, s, list, cnt, v, res);
}
void launch_retire(const int32_t* piv, int k, double* res, hipStream_t s) {
  if (k > 0) hipLaunchKernelGGL(k_retire, dim3((k + 255) / 256), dim3(256), 0, s, piv, k, res);
}
void launch_gather_cols(const double* A, int n, int64_t ng, const int32_t* piv, double* AC, hipStream_t s) {
  hipLaunchKernelGGL(k_gather_cols, dim3(grid_for(int64_t(n) * n, 256)), dim3(256), 0, s, A, n, ng, piv, AC);
}
void launch_compact_pairs(const double* O, int n, double rho_cut, int64_t cap, int32_t* pairs, double* ov,
                          int64_t* count, hipStream_t s) {
  hipLaunchKernelGGL(k_compact_pairs, dim3(1), dim3(CNT), 0, s, O, n, rho_cut, cap, pairs, ov, count);
}
void launch_pair_energy(const double* epart, int npacks, int nblk, const Pack* packs, const int64_t* pidx, double dV,
                        double* e, hipStream_t s) {
  hipLaunchKernelGGL(k_pair_energy, dim3((npacks + 127) / 128), dim3(128), 0, s, epart, npacks, nblk, packs, pidx,
                     dV, e);
}
void launch_d2f(const double* a, float* b, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_d2f, dim3(grid_for(n, 256)), dim3(256), 0, s, a, b, n);
}
void launch_f2d(const float* a, double* b, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_f2d, dim3(grid_for(n, 256)), dim3(256), 0, s, a, b, n);
}
void launch_nonfinite(const double* a, int64_t n, int* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_nonfinite, dim3(grid_for(n, 256)), dim3(256), 0, s, a, n, flag);
}

}  // namespace ace

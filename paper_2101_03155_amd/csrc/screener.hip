// Learned pair screener: features, MLP training and inference, budgeted
// selection.
//
// The screening criterion of Sec. Theory keeps a pair when the overlap
// integral of |phi_i phi_j| exceeds a fixed threshold.  The learned form
// instead predicts each pair's exchange contribution |e_ij| from five
// features and drops the pairs with the smallest predictions while their
// predicted sum stays within an E_x error budget.
//
// Features of pair (i, j): minimum-image distance of the periodic centroids of
// |phi|^2, the smaller and the larger spread, log10 of dV sum |phi_i||phi_j|
// and log10 of dV sum phi_i^2 phi_j^2.
//
// Model (FP32): 5 -> 64 -> 64 -> 1 with tanh, inputs and target standardized
// by statistics stored with the weights.  Flat layout: W1[64][5], b1[64],
// W2[64][64], b2[64], w3[64], b3, then xmean[5], xstd[5], tmean, tstd,
// xmin[5], xmax[5].  Training minimizes the mean squared error of the
// standardized log10 |e_ij| with Adam; per-minibatch gradients are sums over
// samples in a fixed order (no atomics), so training is deterministic.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "ace_internal.h"
#include "tri_pairs.h"

namespace ace {

constexpr int NIN = 5, NH = 64;
constexpr int OW1 = 0, OB1 = OW1 + NH * NIN, OW2 = OB1 + NH, OB2 = OW2 + NH * NH, OW3 = OB2 + NH,
              OB3 = OW3 + NH, NPAR = OB3 + 1;
constexpr int OXM = NPAR, OXS = OXM + NIN, OTM = OXS + NIN, OTS = OTM + 1, OXMIN = OTS + 1, OXMAX = OXMIN + NIN,
              NMODEL = OXMAX + NIN;
static_assert(NPAR == 4609, "parameter count");
static_assert(NMODEL == 4631, "model size");

// ---------------------------------------------------------------- orbital moments
// Per (orbital, z-plane): the plane's total |phi|^2 and its row (y) and column
// (x) sums; pz[orb][z], py[orb][z][y], px[orb][z][x].  With sub also the grid
// subsampled by the stride st per axis, sub[orb][zs][ys][xs] = phi[orb][st zs]
// [st ys][st xs], from the same read.  Bound by that read: 256 orbitals on
// 120^3 (3.5 GB, 0.44 GB written) take 0.92 ms; one row at a time in flight
// and a second kernel for the subsampling took 0.87 + 0.27 ms.
template <int CPL>  // columns per lane, n <= 64 CPL
__global__ __launch_bounds__(256) void k_plane_marginals(const double* __restrict__ phi, int n, int st,
                                                         double* __restrict__ pz, double* __restrict__ py,
                                                         double* __restrict__ px, double* __restrict__ sub) {
  // wave w takes rows y = w, w + 4, ..., RU of them at a time; lanes read a row
  // coalesced, its sum comes from a shuffle reduction, and each lane keeps its
  // columns' partial sums, combined over the waves in LDS at the end
  constexpr int RU = 4;
  const int z = blockIdx.x, orb = blockIdx.y, tid = threadIdx.x;
  const int lane = tid & 63, wv = tid >> 6;
  const int64_t ng = int64_t(n) * n * n;
  const double* P = phi + int64_t(orb) * ng + int64_t(z) * n * n;
  const int m = n / st;
  const bool sz = sub && z % st == 0;
  double* Sp = sz ? sub + (int64_t(orb) * m + z / st) * m * m : nullptr;
  __shared__ double col[4][64 * CPL];
  double cs[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) cs[c] = 0.0;
  for (int y0 = wv; y0 < n; y0 += 4 * RU) {
    double v[RU][CPL], rs[RU];
#pragma unroll
    for (int u = 0; u < RU; ++u)
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        const int x = lane + 64 * c, y = y0 + 4 * u;
        v[u][c] = (x < n && y < n) ? P[y * n + x] : 0.0;
      }
#pragma unroll
    for (int u = 0; u < RU; ++u) {
      rs[u] = 0.0;
#pragma unroll
      for (int c = 0; c < CPL; ++c) {
        cs[c] += v[u][c] * v[u][c];
        rs[u] += v[u][c] * v[u][c];
      }
    }
    if (sz) {
#pragma unroll
      for (int u = 0; u < RU; ++u) {
        const int y = y0 + 4 * u;
        if (y >= n || y % st != 0) continue;
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
          const int x = lane + 64 * c;
          if (x < n && x % st == 0) Sp[(y / st) * m + x / st] = v[u][c];
        }
      }
    }
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
      for (int u = 0; u < RU; ++u) rs[u] += __shfl_down(rs[u], off, 64);
    if (lane == 0)
#pragma unroll
      for (int u = 0; u < RU; ++u)
        if (y0 + 4 * u < n) py[(int64_t(orb) * n + z) * n + y0 + 4 * u] = rs[u];
  }
#pragma unroll
  for (int c = 0; c < CPL; ++c) col[wv][lane + 64 * c] = cs[c];
  __syncthreads();
  double tot = 0.0;
  for (int x = tid; x < n; x += 256) {
    const double s = col[0][x] + col[1][x] + col[2][x] + col[3][x];
    px[(int64_t(orb) * n + z) * n + x] = s;
    tot += s;
  }
  for (int off = 32; off > 0; off >>= 1) tot += __shfl_down(tot, off, 64);
  __syncthreads();
  if (lane == 0) col[0][wv] = tot;
  __syncthreads();
  if (tid == 0) pz[int64_t(orb) * n + z] = col[0][0] + col[0][1] + col[0][2] + col[0][3];
}

// Per orbital: marginals along each axis, periodic centroid (argument of the
// first Fourier coefficient of the marginal) and spread with minimum-image
// displacements.  cen[orb][3] (x, y, z), spr[orb].  One workgroup per orbital,
// so a chain of latencies: the sums over planes run in four groups, then wave
// w takes axis w (one thread per axis and 120 planes in turn took 145 us at
// 120^3, now 17).
__global__ __launch_bounds__(1024) void k_centroids(const double* __restrict__ pz, const double* __restrict__ py,
                                                    const double* __restrict__ px, int n, double L, double dV,
                                                    double* __restrict__ cen, double* __restrict__ spr) {
  const int orb = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  __shared__ double m[3][256], part[2][4][256];
  __shared__ double s3[3];
  const int a = tid & 255, g = tid >> 8;
  double sx = 0.0, sy = 0.0;
  if (a < n) {
#pragma unroll 8
    for (int z = g; z < n; z += 4) {
      sx += px[(int64_t(orb) * n + z) * n + a];
      sy += py[(int64_t(orb) * n + z) * n + a];
    }
  }
  part[0][g][a] = sx;
  part[1][g][a] = sy;
  __syncthreads();
  if (g < 2) m[g][a] = (part[g][0][a] + part[g][1][a]) + (part[g][2][a] + part[g][3][a]);
  else if (g == 2) m[2][a] = a < n ? pz[int64_t(orb) * n + a] : 0.0;
  __syncthreads();
  const double two_pi = 6.283185307179586476925286766559005768;
  if (wv < 3) {
    double cs = 0.0, sn = 0.0;
    for (int i = lane; i < n; i += 64) {
      double s, c;
      sincos(two_pi * double(i) / double(n), &s, &c);
      cs += m[wv][i] * c;
      sn += m[wv][i] * s;
    }
    for (int off = 32; off > 0; off >>= 1) {
      cs += __shfl_xor(cs, off, 64);
      sn += __shfl_xor(sn, off, 64);
    }
    double c = atan2(sn, cs) * L / two_pi;
    c = c - L * floor(c / L);
    double s2 = 0.0;
    for (int i = lane; i < n; i += 64) {
      double d = double(i) * L / double(n) - c;
      d -= L * rint(d / L);
      s2 += m[wv][i] * d * d;
    }
    for (int off = 32; off > 0; off >>= 1) s2 += __shfl_down(s2, off, 64);
    if (lane == 0) {
      cen[orb * 3 + wv] = c;
      s3[wv] = s2;
    }
  }
  __syncthreads();
  if (tid == 0) spr[orb] = sqrt((s3[0] + s3[1] + s3[2]) * dV);
}

// Features of listed pairs (pairs != nullptr) or of every pair i <= j.
__global__ void k_pair_features(const int32_t* __restrict__ pairs, int64_t np, int n, const double* __restrict__ cen,
                                const double* __restrict__ spr, const double* __restrict__ O,
                                const double* __restrict__ P, double L, float* __restrict__ f) {
  for (int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; t < np; t += int64_t(gridDim.x) * blockDim.x) {
    int i, j;
    if (pairs) { i = pairs[2 * t]; j = pairs[2 * t + 1]; }
    else tri_ij(t, n, i, j);
    double d2 = 0.0;
    for (int a = 0; a < 3; ++a) {
      double d = cen[i * 3 + a] - cen[j * 3 + a];
      d -= L * rint(d / L);
      d2 += d * d;
    }
    const double o = O[int64_t(i) * n + j], p = P[int64_t(i) * n + j];
    float* out = f + t * NIN;
    out[0] = float(sqrt(d2));
    out[1] = float(fmin(spr[i], spr[j]));
    out[2] = float(fmax(spr[i], spr[j]));
    out[3] = float(log10(fmax(o, 1e-30)));
    out[4] = float(log10(fmax(p, 1e-30)));
  }
}

// ---------------------------------------------------------------- MLP
__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
  x += 0x9E3779B97F4A7C15ull;
  x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
  x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
  return x ^ (x >> 31);
}

// Glorot-uniform weights from a counter-based generator, zero biases, unit
// standardization.
__global__ void k_mlp_init(float* __restrict__ m, uint64_t seed) {
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < NMODEL; e += gridDim.x * blockDim.x) {
    const double u = double(splitmix64(seed * 0x100000001B3ull + uint64_t(e)) >> 11) * (1.0 / 9007199254740992.0);
    float v = 0.f;
    if (e < OB1) v = float((2 * u - 1) * sqrt(6.0 / (NIN + NH)));
    else if (e >= OW2 && e < OB2) v = float((2 * u - 1) * sqrt(6.0 / (NH + NH)));
    else if (e >= OW3 && e < OB3) v = float((2 * u - 1) * sqrt(6.0 / (NH + 1)));
    else if (e >= OXS && e < OXS + NIN) v = 1.f;
    else if (e == OTS) v = 1.f;
    m[e] = v;
  }
}

// Per block: sums of x, x^2, min, max per feature and of t, t^2 (FP64).
__global__ __launch_bounds__(256) void k_stats_partial(const float* __restrict__ x, const float* __restrict__ t,
                                                       int64_t n, double* __restrict__ part) {
  __shared__ double red[256];
  double acc[4 * NIN + 2];
  for (int k = 0; k < NIN; ++k) { acc[k] = 0; acc[NIN + k] = 0; acc[2 * NIN + k] = 1e300; acc[3 * NIN + k] = -1e300; }
  acc[4 * NIN] = acc[4 * NIN + 1] = 0;
  for (int64_t s = blockIdx.x * int64_t(256) + threadIdx.x; s < n; s += int64_t(gridDim.x) * 256) {
    for (int k = 0; k < NIN; ++k) {
      const double v = x[s * NIN + k];
      acc[k] += v; acc[NIN + k] += v * v;
      acc[2 * NIN + k] = fmin(acc[2 * NIN + k], v); acc[3 * NIN + k] = fmax(acc[3 * NIN + k], v);
    }
    acc[4 * NIN] += t[s]; acc[4 * NIN + 1] += double(t[s]) * t[s];
  }
  for (int q = 0; q < 4 * NIN + 2; ++q) {
    red[threadIdx.x] = acc[q];
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
      if (threadIdx.x < h) {
        const double a = red[threadIdx.x], b = red[threadIdx.x + h];
        red[threadIdx.x] = (q >= 2 * NIN && q < 3 * NIN) ? fmin(a, b) : (q >= 3 * NIN && q < 4 * NIN) ? fmax(a, b) : a + b;
      }
      __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x * (4 * NIN + 2) + q] = red[0];
    __syncthreads();
  }
}

__global__ void k_stats_final(const double* __restrict__ part, int nb, int64_t n, float* __restrict__ m) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  double acc[4 * NIN + 2];
  for (int q = 0; q < 4 * NIN + 2; ++q) acc[q] = (q >= 2 * NIN && q < 3 * NIN) ? 1e300 : (q >= 3 * NIN && q < 4 * NIN) ? -1e300 : 0.0;
  for (int b = 0; b < nb; ++b)
    for (int q = 0; q < 4 * NIN + 2; ++q) {
      const double v = part[b * (4 * NIN + 2) + q];
      acc[q] = (q >= 2 * NIN && q < 3 * NIN) ? fmin(acc[q], v) : (q >= 3 * NIN && q < 4 * NIN) ? fmax(acc[q], v) : acc[q] + v;
    }
  for (int k = 0; k < NIN; ++k) {
    const double mu = acc[k] / double(n);
    const double var = acc[NIN + k] / double(n) - mu * mu;
    m[OXM + k] = float(mu);
    m[OXS + k] = float(sqrt(fmax(var, 1e-12)));
    m[OXMIN + k] = float(acc[2 * NIN + k]);
    m[OXMAX + k] = float(acc[3 * NIN + k]);
  }
  const double mu = acc[4 * NIN] / double(n);
  m[OTM] = float(mu);
  m[OTS] = float(sqrt(fmax(acc[4 * NIN + 1] / double(n) - mu * mu, 1e-12)));
}

// Prediction (de-standardized target, log10 |e|) of every sample; with clamp
// the features are first clipped to the training ranges.  Four waves share 64
// samples, one per lane: wave w has hidden units 16 w ... 16 w + 15 of both
// layers, which pass through LDS (a chain of 64 dependent operations per unit:
// all units in one lane took 44 us at 32896 samples, now 23).  The sums of a
// unit and of the output run in the order of their indices.
constexpr int FP = 65;
__global__ __launch_bounds__(256) void k_mlp_forward(const float* __restrict__ model, const float* __restrict__ x,
                                                     int64_t n, int clamp, float* __restrict__ y) {
  __shared__ float w[NMODEL];
  __shared__ float h[64 * FP];
  for (int e = threadIdx.x; e < NMODEL; e += 256) w[e] = model[e];
  const int lane = threadIdx.x & 63, u0 = (threadIdx.x >> 6) * 16;
  float* hl = h + lane * FP;
  for (int64_t s0 = blockIdx.x * int64_t(64); s0 < n; s0 += int64_t(gridDim.x) * 64) {
    const int64_t s = s0 + lane < n ? s0 + lane : n - 1;
    __syncthreads();
    float xs[NIN];
    for (int k = 0; k < NIN; ++k) {
      float v = x[s * NIN + k];
      if (clamp) v = fminf(fmaxf(v, w[OXMIN + k]), w[OXMAX + k]);
      xs[k] = (v - w[OXM + k]) / w[OXS + k];
    }
#pragma unroll
    for (int j = u0; j < u0 + 16; ++j) {
      float a = w[OB1 + j];
#pragma unroll
      for (int k = 0; k < NIN; ++k) a += w[OW1 + j * NIN + k] * xs[k];
      hl[j] = tanhf(a);
    }
    __syncthreads();
    float h1[NH];
#pragma unroll
    for (int k = 0; k < NH; ++k) h1[k] = hl[k];
    __syncthreads();
#pragma unroll 4
    for (int j = u0; j < u0 + 16; ++j) {
      float a = w[OB2 + j];
#pragma unroll
      for (int k = 0; k < NH; ++k) a += w[OW2 + j * NH + k] * h1[k];
      hl[j] = tanhf(a);
    }
    __syncthreads();
    if (u0 == 0 && s0 + lane < n) {
      float out = w[OB3];
#pragma unroll
      for (int j = 0; j < NH; ++j) out += w[OW3 + j] * hl[j];
      y[s] = w[OTM] + w[OTS] * out;
    }
  }
}

// Minibatch gradient, per-block partial sums.  Sample k of the batch is
// idx = (off + (b0 + k) * stride) mod n; the batch holds bsz samples (the
// loss is their mean).  Each block takes whole chunks of 64 samples with 512
// threads, everything in LDS: the three 64 x 64 x 64 products of a chunk
// (hidden layer, its backward, and the gradient of W2) run on the FP32 matrix
// cores, wave w owning the 16 x 16 tiles 2w and 2w + 1, the gradient tiles in
// registers from chunk to chunk; the thin gradients (W1, b1, b2, w3, b3) are
// one entry per thread.  At 4096 samples the launch is 64 blocks of one chunk,
// so a step is a chain of LDS trips and barriers and is bound by their latency
// (12 us, and 5 us for the Adam step; scalar loops over LDS took 114 and 18 us:
// an epoch of 131072 samples went from 4.18 to 0.52 ms).
// Rows have a pitch of 68 floats: the MFMA operand reads of 16 rows x 4 columns
// then fall in 64 distinct banks, as 4 * row + column.
constexpr int GCH = 64;
constexpr int GNT = 512;
constexpr int GP = 68;
typedef float f32x4 __attribute__((ext_vector_type(4)));

// rows [16 tm, +16) x columns [16 tn, +16) of sum_k A(m, k) B(k, n) over 64 k;
// a and b read A[m][k] and B[k][n] from LDS.
template <typename FA, typename FB>
__device__ __forceinline__ f32x4 tile64(int lane, FA a, FB b, f32x4 acc) {
  const int i = lane & 15, q = lane >> 4;
#pragma unroll
  for (int k = 0; k < NH; k += 4) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a(i, k + q), b(k + q, i), acc, 0, 0, 0);
  return acc;
}

__global__ __launch_bounds__(GNT) void k_mlp_grad_partial(const float* __restrict__ model, const float* __restrict__ x,
                                                          const float* __restrict__ t, int64_t n, int64_t off,
                                                          int64_t stride, int64_t b0, int bsz,
                                                          float* __restrict__ gpart, float* __restrict__ lpart) {
  __shared__ float W2[NH * GP], W2T[NH * GP], H1[GCH * GP], H2[GCH * GP], D2[GCH * GP], D1[GCH * GP];
  __shared__ float xs[GCH][8];  // standardized features, [5] the standardized target
  __shared__ float dout[GCH], lsum[GCH];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int e = tid; e < NH * NH; e += GNT) {
    const int j = e / NH, k = e % NH;
    const float v = model[OW2 + e];
    W2[j * GP + k] = v;
    W2T[k * GP + j] = v;
  }
  // this thread's hidden unit in the first layer, and in the head its samples' part
  const int hj = tid & 63, hs = tid >> 6;  // unit hj of samples hs, hs + 8, ...
  float w1[NIN];
#pragma unroll
  for (int k = 0; k < NIN; ++k) w1[k] = model[OW1 + hj * NIN + k];
  const float b1 = model[OB1 + hj];
  const int ps = tid >> 3, pp = tid & 7;  // sample ps, hidden units 8 pp .. 8 pp + 7
  float w3[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) w3[q] = model[OW3 + 8 * pp + q];
  const float b3 = model[OB3], tm = model[OTM], ts = model[OTS];
  const float mu = pp < NIN ? model[OXM + pp] : 0.f, sd = pp < NIN ? model[OXS + pp] : 1.f;
  const int ti = 2 * wv, tj = 2 * wv + 1;  // this wave's tiles (row ti / 4, column ti % 4)
  const float b2i = model[OB2 + (ti & 3) * 16 + (lane & 15)], b2j = model[OB2 + (tj & 3) * 16 + (lane & 15)];
  f32x4 g2i = {0.f, 0.f, 0.f, 0.f}, g2j = {0.f, 0.f, 0.f, 0.f};
  // thin gradient entries: thread t < 320 owns W1 entry t, the next 64 b1, then b2, w3; thread 0 also b3
  float gthin = 0.f, gb3 = 0.f, loss = 0.f;
  const int nch = (bsz + GCH - 1) / GCH;
  for (int ch = blockIdx.x; ch < nch; ch += gridDim.x) {
    const int s0 = ch * GCH;
    const int cnt = (bsz - s0 < GCH) ? bsz - s0 : GCH;
    // inputs and standardized targets
    {
      float v = 0.f;
      if (ps < cnt && pp <= NIN) {
        const int64_t idx = (off + (b0 + s0 + ps) * stride) % n;
        v = pp < NIN ? (x[idx * NIN + pp] - mu) / sd : (t[idx] - tm) / ts;
      }
      xs[ps][pp] = v;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < GCH / 8; ++q) {
      const int sl = hs + 8 * q;
      float a = b1;
#pragma unroll
      for (int k = 0; k < NIN; ++k) a += w1[k] * xs[sl][k];
      H1[sl * GP + hj] = tanhf(a);
    }
    __syncthreads();
    {
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      auto fwd = [&](int tl, float b2) {
        const int m0 = (tl >> 2) * 16, n0 = (tl & 3) * 16;
        const f32x4 z = tile64(lane, [&](int i, int k) { return H1[(m0 + i) * GP + k]; },
                               [&](int k, int i) { return W2[(n0 + i) * GP + k]; }, zero);
#pragma unroll
        for (int r = 0; r < 4; ++r) H2[(m0 + 4 * (lane >> 4) + r) * GP + n0 + (lane & 15)] = tanhf(z[r] + b2);
      };
      fwd(ti, b2i);
      fwd(tj, b2j);
    }
    __syncthreads();
    {
      float h[8], o = 0.f;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        h[q] = H2[ps * GP + 8 * pp + q];
        o += w3[q] * h[q];
      }
      for (int m = 1; m < 8; m <<= 1) o += __shfl_xor(o, m, 64);
      const float r = ps < cnt ? o + b3 - xs[ps][NIN] : 0.f;
      const float d = 2.f * r / float(bsz);
#pragma unroll
      for (int q = 0; q < 8; ++q) D2[ps * GP + 8 * pp + q] = d * w3[q] * (1.f - h[q] * h[q]);
      if (pp == 0) {
        dout[ps] = d;
        lsum[ps] = r * r / float(bsz);
      }
    }
    __syncthreads();
    {
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      auto bwd = [&](int tl) {
        const int m0 = (tl >> 2) * 16, n0 = (tl & 3) * 16;
        const f32x4 z = tile64(lane, [&](int i, int k) { return D2[(m0 + i) * GP + k]; },
                               [&](int k, int i) { return W2T[(n0 + i) * GP + k]; }, zero);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int e = (m0 + 4 * (lane >> 4) + r) * GP + n0 + (lane & 15);
          D1[e] = z[r] * (1.f - H1[e] * H1[e]);
        }
      };
      bwd(ti);
      bwd(tj);
      auto grad = [&](int tl, f32x4 acc) {
        const int m0 = (tl >> 2) * 16, n0 = (tl & 3) * 16;
        return tile64(lane, [&](int i, int s) { return D2[s * GP + m0 + i]; },
                      [&](int s, int i) { return H1[s * GP + n0 + i]; }, acc);
      };
      g2i = grad(ti, g2i);
      g2j = grad(tj, g2j);
    }
    __syncthreads();
    {
      float g = 0.f;
      if (tid < OB1) {
        const int j = tid / NIN, k = tid % NIN;
        for (int sl = 0; sl < GCH; ++sl) g += D1[sl * GP + j] * xs[sl][k];
      } else if (tid < OB1 + NH) {
        for (int sl = 0; sl < GCH; ++sl) g += D1[sl * GP + tid - OB1];
      } else if (tid < OB1 + 2 * NH) {
        for (int sl = 0; sl < GCH; ++sl) g += D2[sl * GP + tid - OB1 - NH];
      } else {
        for (int sl = 0; sl < GCH; ++sl) g += dout[sl] * H2[sl * GP + tid - OB1 - 2 * NH];
      }
      gthin += g;
      if (wv == 0) {  // (every lane of the wave ends with the sums)
        float a = dout[lane], l = lsum[lane];
        for (int m = 1; m < 64; m <<= 1) {
          a += __shfl_xor(a, m, 64);
          l += __shfl_xor(l, m, 64);
        }
        gb3 += a;
        loss += l;
      }
    }
    __syncthreads();
  }
  float* out = gpart + int64_t(blockIdx.x) * NPAR;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    out[OW2 + ((ti >> 2) * 16 + 4 * (lane >> 4) + r) * NH + (ti & 3) * 16 + (lane & 15)] = g2i[r];
    out[OW2 + ((tj >> 2) * 16 + 4 * (lane >> 4) + r) * NH + (tj & 3) * 16 + (lane & 15)] = g2j[r];
  }
  out[tid < OW2 ? tid : OB2 - OW2 + tid] = gthin;  // W1 and b1, then b2 and w3
  if (tid == 0) {
    out[OB3] = gb3;
    lpart[blockIdx.x] = loss;
  }
}
static_assert(OB1 + 3 * NH == GNT && OW2 == OB1 + NH, "one thin gradient entry per thread");

// Sum over the block partials of one parameter per group of 8 threads (thread
// g takes blocks g, g + 8, ..., the groups' sums are added in order), 32
// parameters per workgroup; returned to the group's first thread.
constexpr int RG = 8, RPB = 32;
__device__ __forceinline__ float partial_sum(const float* __restrict__ gpart, int nb, int e, float (&red)[RG][RPB]) {
  const int p = threadIdx.x % RPB, g = threadIdx.x / RPB;
  float a = 0.f;
  if (e < NPAR)
    for (int b = g; b < nb; b += RG) a += gpart[int64_t(b) * NPAR + e];
  red[g][p] = a;
  __syncthreads();
  float s = 0.f;
  if (g == 0)
    for (int q = 0; q < RG; ++q) s += red[q][p];
  return s;
}
// The block losses, summed by the first wave of workgroup 0.
__device__ __forceinline__ float loss_sum(const float* __restrict__ lpart, int nb) {
  float l = 0.f;
  for (int b = threadIdx.x; b < nb; b += 64) l += lpart[b];
  for (int m = 1; m < 64; m <<= 1) l += __shfl_xor(l, m, 64);
  return l;
}

// Sum of the block partials in a fixed order: gradient and loss.
__global__ __launch_bounds__(RG * RPB) void k_mlp_reduce(const float* __restrict__ gpart,
                                                         const float* __restrict__ lpart, int nb,
                                                         float* __restrict__ grad, float* __restrict__ loss) {
  __shared__ float red[RG][RPB];
  const int e = blockIdx.x * RPB + threadIdx.x % RPB;
  const float g = partial_sum(gpart, nb, e, red);
  if (threadIdx.x < RPB && e < NPAR) grad[e] = g;
  if (blockIdx.x == 0 && threadIdx.x < 64 && loss) {
    const float l = loss_sum(lpart, nb);
    if (threadIdx.x == 0) loss[0] = l;
  }
}

// Adam on the summed partials; loss_acc[0] += batch loss.
__global__ __launch_bounds__(RG * RPB) void k_mlp_adam(const float* __restrict__ gpart,
                                                       const float* __restrict__ lpart, int nb,
                                                       float* __restrict__ model, float* __restrict__ mom,
                                                       float* __restrict__ vel, int step, float lr, float b1, float b2,
                                                       float eps, float* __restrict__ loss_acc) {
  __shared__ float red[RG][RPB];
  const int e = blockIdx.x * RPB + threadIdx.x % RPB;
  const float g = partial_sum(gpart, nb, e, red);
  if (threadIdx.x < RPB && e < NPAR) {
    const float c1 = 1.f - powf(b1, float(step)), c2 = 1.f - powf(b2, float(step));
    const float m = b1 * mom[e] + (1.f - b1) * g;
    const float v = b2 * vel[e] + (1.f - b2) * g * g;
    mom[e] = m;
    vel[e] = v;
    model[e] -= lr * (m / c1) / (sqrtf(v / c2) + eps);
  }
  if (blockIdx.x == 0 && threadIdx.x < 64 && loss_acc) {
    const float l = loss_sum(lpart, nb);
    if (threadIdx.x == 0) loss_acc[0] += l;
  }
}

// ---------------------------------------------------------------- budgeted selection
// Off-diagonal pair t is out of distribution when it lies beyond the training
// box on the side where pairs interact more: closer centroids than any
// training pair, larger overlaps, or spreads outside the training range
// (each widened by tol * span).  Pairs beyond the box on the far side
// (farther apart, smaller overlaps) are predicted with features clipped to
// the box, which over-estimates their contribution.
// The same pass prepares the threshold: q[t] = pred[t] for off-diagonal pairs
// and +inf for the diagonal (never dropped), w[t] = 10^pred[t] (0 there).
__global__ void k_budget_prep(const float* __restrict__ f, const float* __restrict__ pred, int64_t np, int n,
                              const float* __restrict__ model, float tol, int* __restrict__ count,
                              float* __restrict__ q, double* __restrict__ w) {
  int c = 0;
  for (int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; t < np; t += int64_t(gridDim.x) * blockDim.x) {
    int i, j;
    tri_ij(t, n, i, j);
    const float p = pred[t];
    q[t] = (i == j) ? INFINITY : p;
    w[t] = (i == j) ? 0.0 : pow(10.0, double(p));
    if (i == j) continue;
    for (int k = 0; k < NIN; ++k) {
      const float lo = model[OXMIN + k], hi = model[OXMAX + k], span = hi - lo;
      const float v = f[t * NIN + k];
      const bool below = v < lo - tol * span, above = v > hi + tol * span;
      const bool risky = (k == 0) ? below : (k <= 2) ? (below || above) : above;
      if (risky) { ++c; break; }
    }
  }
  if (c) atomicAdd(count, c);
}

// Threshold tau (in log10): the smallest prediction v whose pairs up to and
// including v have a sum of 10^pred above the budget (the pairs below tau are
// dropped), or one more than the largest prediction if the sum of all is within
// it.  Radix selection in one workgroup over the prepared arrays: predictions
// map to 32-bit keys in their order, and each of eight passes finds the next
// four bits of v from the sums of the 16 bins of the keys that share the bits
// so far.  A thread has its own 16 bins in LDS and these are added in a fixed
// order, so tau does not vary between runs.  Bound by the eight reads of the
// keys by one CU (32896 pairs: 70 us; 64 bisections over keys and weights
// took 599).  NaN and +inf belong to no bin; a prediction of -inf keeps all.
constexpr int TNT = 1024, TREG = 24;
constexpr unsigned NOKEY = 0xffffffffu;  // the pattern of a NaN
__device__ __forceinline__ unsigned order_key(float v) {
  const unsigned u = __float_as_uint(v);
  return v < INFINITY ? ((u & 0x80000000u) ? ~u : u | 0x80000000u) : NOKEY;
}
__device__ __forceinline__ double key_value(unsigned k) {
  return double(__uint_as_float((k & 0x80000000u) ? k & 0x7fffffffu : ~k));
}
__global__ __launch_bounds__(TNT) void k_budget_threshold(const float* __restrict__ q, const double* __restrict__ w,
                                                          int64_t np, double budget, double* __restrict__ tau) {
  __shared__ double bin[16][TNT];
  __shared__ double tot[16];
  __shared__ unsigned s_prefix;
  __shared__ double s_base;
  __shared__ int s_all;
  __shared__ unsigned s_max[TNT / 64], s_min[TNT / 64];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  // the first keys of a thread stay in registers
  unsigned key[TREG];
#pragma unroll
  for (int u = 0; u < TREG; ++u) key[u] = tid + u * TNT < np ? order_key(q[tid + u * TNT]) : NOKEY;
  unsigned prefix = 0, mx = 0, mn = NOKEY;
  double base = 0.0;
  for (int p = 0; p < 8; ++p) {
    const int sh = 28 - 4 * p;
#pragma unroll
    for (int d = 0; d < 16; ++d) bin[d][tid] = 0.0;
    // eight keys at a time: the weights of those that count, all in flight
    const auto add8 = [&](const unsigned* k, int64_t t0) {
      bool on[8], any = false;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        on[u] = k[u] != NOKEY && (p == 0 || ((k[u] ^ prefix) >> (sh + 4)) == 0);
        any = any || on[u];
      }
      if (!__any(any)) return;
      double wt[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) wt[u] = w[on[u] ? t0 + u * TNT : 0];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (on[u]) {
          bin[(k[u] >> sh) & 15][tid] += wt[u];
          mx = k[u] > mx ? k[u] : mx;
          mn = k[u] < mn ? k[u] : mn;
        }
    };
#pragma unroll
    for (int u = 0; u < TREG; u += 8) add8(key + u, tid + int64_t(u) * TNT);
    for (int64_t t0 = tid + int64_t(TREG) * TNT; t0 - tid < np; t0 += 8 * TNT) {
      unsigned k[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) k[u] = t0 + u * TNT < np ? order_key(q[t0 + u * TNT]) : NOKEY;
      add8(k, t0);
    }
    __syncthreads();
    // wave wv adds up bin wv (16 waves, 16 bins)
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < TNT / 64; ++u) s += bin[wv][lane + 64 * u];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    if (lane == 0) tot[wv] = s;
    if (p == 0) {
      for (int off = 32; off > 0; off >>= 1) {
        mx = max(mx, unsigned(__shfl_down(int(mx), off, 64)));
        mn = min(mn, unsigned(__shfl_down(int(mn), off, 64)));
      }
      if (lane == 0) {
        s_max[wv] = mx;
        s_min[wv] = mn;
      }
    }
    __syncthreads();
    if (tid == 0) {
      int d = 0;
      double cum = base;
      for (; d < 16; ++d) {
        if (cum + tot[d] > budget) break;
        if (d < 15 || p == 0) cum += tot[d];
      }
      if (p == 0) {
        unsigned a = s_max[0], b = s_min[0];
        for (int i = 1; i < TNT / 64; ++i) {
          a = max(a, s_max[i]);
          b = min(b, s_min[i]);
        }
        const bool low = b == order_key(-INFINITY);
        s_all = d == 16 || low;
        if (low) tau[0] = -INFINITY;
        else if (d == 16) tau[0] = b == NOKEY ? 0.0 : key_value(a) + 1.0;
      }
      // past the first pass the bins of a prefix can fall short of the sum that
      // chose it by a rounding: its last bin then holds the threshold
      if (d > 15) d = 15;
      s_prefix = prefix | (unsigned(d) << sh);
      s_base = cum;
    }
    __syncthreads();
    if (s_all) return;
    prefix = s_prefix;
    base = s_base;
  }
  if (tid == 0) tau[0] = key_value(prefix);
}

// keep[t] = diagonal, or off-diagonal with pred >= tau (learned rule), or
// O >= rho_cut (threshold rule when fallback is set).
__global__ void k_keep_flags(const float* __restrict__ pred, int64_t np, int n, const double* __restrict__ tau,
                             const double* __restrict__ O, double rho_cut, const int* __restrict__ fallback,
                             uint8_t* __restrict__ keep) {
  const bool fb = fallback && fallback[0] > 0;
  for (int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; t < np; t += int64_t(gridDim.x) * blockDim.x) {
    int i, j;
    tri_ij(t, n, i, j);
    bool k;
    if (i == j) k = true;
    else if (fb) k = O[int64_t(i) * n + j] >= rho_cut;
    else k = double(pred[t]) >= tau[0];
    keep[t] = k ? 1 : 0;
  }
}

// Ordered compaction of kept pairs (triangle order = sorted by i, then j).
__global__ __launch_bounds__(CNT) void k_compact_keep(const uint8_t* __restrict__ keep, int64_t np, int n,
                                                      int64_t cap, int32_t* __restrict__ pairs,
                                                      int64_t* __restrict__ count) {
  compact_tri(
      n, [&](int64_t t, int, int) { return keep[t] != 0; },
      [&](int64_t p, int i, int j) {
        if (p < cap) {
          pairs[2 * p] = i;
          pairs[2 * p + 1] = j;
        }
      },
      count);
}

// ---------------------------------------------------------------- launchers
static unsigned gridn(int64_t n, int nt, int cap = 4096) {
  int64_t g = (n + nt - 1) / nt;
  if (g > cap) g = cap;
  return unsigned(g < 1 ? 1 : g);
}

void launch_marginals(const double* phi, int norb, int n, int st, double* pz, double* py, double* px, double* sub,
                      hipStream_t s) {
  if (n <= 128)
    hipLaunchKernelGGL(k_plane_marginals<2>, dim3(n, norb), dim3(256), 0, s, phi, n, st, pz, py, px, sub);
  else
    hipLaunchKernelGGL(k_plane_marginals<4>, dim3(n, norb), dim3(256), 0, s, phi, n, st, pz, py, px, sub);
}
void launch_centroids(const double* pz, const double* py, const double* px, int norb, int n, double L, double dV,
                      double* cen, double* spr, hipStream_t s) {
  hipLaunchKernelGGL(k_centroids, dim3(norb), dim3(1024), 0, s, pz, py, px, n, L, dV, cen, spr);
}
void launch_pair_features(const int32_t* pairs, int64_t np, int norb, const double* cen, const double* spr,
                          const double* O, const double* P, double L, float* f, hipStream_t s) {
  hipLaunchKernelGGL(k_pair_features, dim3(gridn(np, 256)), dim3(256), 0, s, pairs, np, norb, cen, spr, O, P, L, f);
}
void launch_mlp_init(float* m, uint64_t seed, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_init, dim3(gridn(NMODEL, 256)), dim3(256), 0, s, m, seed);
}
int stats_blocks(int64_t n) { return int(gridn(n, 256, 256)); }
void launch_mlp_stats(const float* x, const float* t, int64_t n, double* part, float* m, hipStream_t s) {
  const int nb = stats_blocks(n);
  hipLaunchKernelGGL(k_stats_partial, dim3(nb), dim3(256), 0, s, x, t, n, part);
  hipLaunchKernelGGL(k_stats_final, dim3(1), dim3(1), 0, s, part, nb, n, m);
}
void launch_mlp_forward(const float* m, const float* x, int64_t n, int clamp, float* y, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_forward, dim3(gridn(n, 64, 2048)), dim3(256), 0, s, m, x, n, clamp, y);
}
int mlp_grad_blocks(int bsz) { return int(gridn(bsz, GCH, 1024)); }
void launch_mlp_grad_partial(const float* m, const float* x, const float* t, int64_t n, int64_t off, int64_t stride,
                             int64_t b0, int bsz, float* gpart, float* lpart, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_grad_partial, dim3(mlp_grad_blocks(bsz)), dim3(GNT), 0, s, m, x, t, n, off, stride, b0,
                     bsz, gpart, lpart);
}
void launch_mlp_reduce(const float* gpart, const float* lpart, int nb, float* grad, float* loss, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_reduce, dim3(gridn(NPAR, RPB)), dim3(RG * RPB), 0, s, gpart, lpart, nb, grad, loss);
}
void launch_mlp_adam(const float* gpart, const float* lpart, int nb, float* m, float* mom, float* vel, int step,
                     float lr, float b1, float b2, float eps, float* loss_acc, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_adam, dim3(gridn(NPAR, RPB)), dim3(RG * RPB), 0, s, gpart, lpart, nb, m, mom, vel, step, lr,
                     b1, b2, eps, loss_acc);
}
void launch_select(const float* pred, const float* feats, int64_t np, int norb, const float* model, double budget,
                   const double* O, double rho_cut, float ood_tol, int* ood, double* tau, uint8_t* keep, int64_t cap,
                   int32_t* pairs, int64_t* count, float* q, double* w, hipStream_t s) {
  hipLaunchKernelGGL(k_budget_prep, dim3(gridn(np, 256)), dim3(256), 0, s, feats, pred, np, norb, model, ood_tol, ood,
                     q, w);
  hipLaunchKernelGGL(k_budget_threshold, dim3(1), dim3(TNT), 0, s, q, w, np, budget, tau);
  hipLaunchKernelGGL(k_keep_flags, dim3(gridn(np, 256)), dim3(256), 0, s, pred, np, norb, tau, O, rho_cut, ood, keep);
  hipLaunchKernelGGL(k_compact_keep, dim3(1), dim3(CNT), 0, s, keep, np, norb, cap, pairs, count);
}

}  // namespace ace

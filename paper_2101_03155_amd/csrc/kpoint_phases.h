// Device bodies of the owner-computes pair stage of the k-point build: the
// in-plane transforms of one z-plane of a pair's complex field with the plane
// in LDS, and the z pass over tiles of the transformed planes.
//
// The spectrum of a slot is [z][kx][ky] (ky fastest): the forward transform
// takes y first, on columns read coalesced along x, then x on the rows, and
// stores with consecutive threads on consecutive ky; the inverse takes x
// first and y last, so that its last pass ends with consecutive threads on
// consecutive x of the potential, which multiply the partner's row (read
// coalesced) and accumulate in registers without another trip through LDS.
// Every pass gives consecutive threads consecutive lines; in LDS the plane is
// [y][x] with a row pitch of N + 1 values, odd, so lines along either axis
// start in distinct banks.
#pragma once
#include "ace_internal.h"
#include "fft.h"

namespace ace {

// Largest grid whose padded complex plane fits in LDS beside the twiddles.
template <int N> __host__ __device__ constexpr bool kplane_fits() {
  return (size_t(N) * (N + 1) + N) * 16 <= 163840 && N <= 96;
}
// Threads of the in-plane kernels: the butterflies of the passes divide them
// evenly or nearly so (48 = 4 x 12: 576 and 192 butterflies; 96 = 8 x 12:
// 1152 and 768; 80 = 8 x 10: 800 and 640).
template <int N> __host__ __device__ constexpr int kplane_nt() {
  return N <= 16 ? 64 : N == 24 ? 192 : N == 32 ? 128 : N == 48 ? 192 : N == 64 ? 512 : N == 80 ? 640 : 768;
}
// z-pass tile: consecutive flattened (kx, ky) columns, and its threads.
template <int N> __host__ __device__ constexpr int kconv_tx() { return N * N % 32 == 0 ? 32 : 16; }
template <int N> __host__ __device__ constexpr int kconv_nt() { return N <= 16 ? 128 : 256; }

// v(|G + d|) / N^3 at integer frequencies (kx, ky, kz) in FFT order.
template <int N>
__device__ __forceinline__ double kernel_value_shift(const KernelParams& kp, const double* d, int kx, int ky, int kz) {
  const int sx = kx < (N + 1) / 2 ? kx : kx - N;
  const int sy = ky < (N + 1) / 2 ? ky : ky - N;
  const int sz = kz < (N + 1) / 2 ? kz : kz - N;
  const double gx = kp.g[0] * sx + d[0], gy = kp.g[1] * sy + d[1], gz = kp.g[2] * sz + d[2];
  const double g2 = gx * gx + gy * gy + gz * gz;
  const double four_pi = 12.566370614359172953850573533118011537;
  double v;
  if (g2 == 0.0) {
    v = (kp.kind == 0) ? 0.0 : 3.14159265358979323846264338327950288 / (kp.omega * kp.omega);
  } else if (kp.kind == 0) {
    v = four_pi / g2;
  } else {
    v = -four_pi / g2 * expm1(-g2 / (4.0 * kp.omega * kp.omega));
  }
  return v * kp.inv_ng;
}

// conj(u_a) u_b of one z-plane (ua, ub point at it) -> its in-plane spectrum
// out[kx][ky].
template <int N, int NT>
__device__ __forceinline__ void body_kfwd_xy(const double2* __restrict__ ua, const double2* __restrict__ ub,
                                             double2* out, double2* buf, const double2* tw, int tid) {
  constexpr int XL = N + 1;
  fft_lines_ls<double, N, N, 1, XL, NT, -1, false, 0, true>(
      buf, tw, tid,
      [ua, ub](int l, int p) {
        const double2 x = ua[p * N + l], y = ub[p * N + l];
        double2 f;
        f.x = x.x * y.x + x.y * y.y;  // conj(x) * y
        f.y = x.x * y.y - x.y * y.x;
        return f;
      },
      [buf](int l, int p, double2 x) { buf[l + p * XL] = x; });
  fft_lines_ls<double, N, N, XL, 1, NT, -1, false, 0>(
      buf, tw, tid, [buf](int l, int p) { return buf[l * XL + p]; },
      [out](int l, int p, double2 x) { out[p * N + l] = x; });
}

// The kernel values of the TX columns starting at f0 that this thread
// multiplies in body_kconv_z.
template <int N, int TX, int NT> __host__ __device__ constexpr int kconv_lv() { return (N * TX + NT - 1) / NT; }
template <int N, int TX, int NT>
__device__ __forceinline__ void load_kvtile(const KernelParams& kp, const double* d, int f0, int tid,
                                            double (&vv)[kconv_lv<N, TX, NT>()]) {
#pragma unroll
  for (int q = 0; q < kconv_lv<N, TX, NT>(); ++q) {
    const int e = tid + q * NT;
    if (N * TX % NT == 0 || e < N * TX) {
      const int f = f0 + e % TX;
      vv[q] = kernel_value_shift<N>(kp, d, f / N, f % N, e / TX);
    }
  }
}

// z lines of the TX columns starting at base (plane pitch N * N): forward
// FFT, times the kernel values, inverse FFT; in place.
template <int N, int TX, int NT>
__device__ __forceinline__ void body_kconv_z(double2* base, double2* buf, const double2* tw, int tid,
                                             const double (&vv)[kconv_lv<N, TX, NT>()]) {
  constexpr int PL = N * N;
  fft_lines_load<double, N, TX, 1, TX, NT, -1, false, 0>(buf, tw, tid,
                                                         [base](int l, int p) { return base[size_t(p) * PL + l]; });
#pragma unroll
  for (int q = 0; q < kconv_lv<N, TX, NT>(); ++q) {
    const int e = tid + q * NT;
    if (N * TX % NT == 0 || e < N * TX) {
      double2 c = buf[e];
      c.x *= vv[q];
      c.y *= vv[q];
      buf[e] = c;
    }
  }
  __syncthreads();
  fft_lines_to<double, N, 0, TX, 1, TX, NT, +1, false, 0>(
      buf, tw, tid, [base](int l, int p, double2 x) { base[size_t(p) * PL + l] = x; });
}

// Points of the plane each thread holds after the inverse's last y pass, and
// the (x, y) of point (s, r).
template <int N, int NT> struct KOwn {
  static constexpr int LAST = plan_len(N) - 1;
  static constexpr int R = plan_radix(N, LAST), NB = N / R, TOT = N * NB, PER = (TOT + NT - 1) / NT;
  static constexpr int PTS = PER * R;
};

// Passes 0 .. plan_len - 2 of the inverse y transforms (the last one is fused
// with the accumulation).
template <int N, int NT, int P>
__device__ __forceinline__ void kinv_y_head(double2* buf, const double2* tw, int tid) {
  if constexpr (P + 1 < plan_len(N)) {
    fft_pass<double, N, P, N, 1, N + 1, NT, +1, false, 0>(buf, tw, tid);
    kinv_y_head<N, NT, P + 1>(buf, tw, tid);
  }
}

// acc += (V or conj V) u_j over one z-plane: in is the pair's spectrum plane
// [kx][ky] after the z pass, uj the partner's plane.
template <int N, int NT>
__device__ __forceinline__ void body_kinv_acc(const double2* __restrict__ in, const double2* __restrict__ uj,
                                              bool conj, double2* buf, const double2* tw, int tid,
                                              double2 (&acc)[KOwn<N, NT>::PTS]) {
  using K = KOwn<N, NT>;
  constexpr int XL = N + 1;
  // x: the first pass reads global memory before its barrier and writes LDS
  // after it, which orders it behind the previous entry's last reads of buf
  fft_lines_ls<double, N, N, XL, 1, NT, +1, false, 0, true>(
      buf, tw, tid, [in](int l, int p) { return in[p * N + l]; },
      [buf](int l, int p, double2 x) { buf[l * XL + p] = x; });
  kinv_y_head<N, NT, 0>(buf, tw, tid);
  const double sg = conj ? -1.0 : 1.0;
#pragma unroll
  for (int s = 0; s < K::PER; ++s) {
    const int b = tid + s * NT;
    if (K::TOT % NT == 0 || b < K::TOT) {
      const int l = b % N, j = b / N;
      double2 f[K::R], v[K::R];
#pragma unroll
      for (int r = 0; r < K::R; ++r) f[r] = uj[(j + r * K::NB) * N + l];
#pragma unroll
      for (int r = 0; r < K::R; ++r) {
        v[r] = buf[l + (j + r * K::NB) * XL];
        if (K::LAST > 0 && r > 0) v[r] = cmulc(v[r], tw[r * j]);
      }
      Dft<K::R, +1, double2>::run(v);
#pragma unroll
      for (int r = 0; r < K::R; ++r) {
        const double vy = sg * v[r].y;
        double2& a = acc[s * K::R + r];
        a.x += f[r].x * v[r].x - f[r].y * vy;
        a.y += f[r].x * vy + f[r].y * v[r].x;
      }
    }
  }
}

// W_k of one z-plane from the adjacency entries (slot, partner) a0 .. a1 of
// orbital k: w_k -= c sum_j (V_kj or conj V_kj) u_j, the conjugate where k is
// the pair's first orbital.  add: the plane already holds earlier entries.
template <int N, int NT>
__device__ __forceinline__ void body_kowner(const double2* __restrict__ u, const double2* __restrict__ spec,
                                            const int32_t* __restrict__ adj, int a0, int a1, int k, int z,
                                            double2* __restrict__ wk, double c, bool add, double2* buf,
                                            const double2* tw, int tid) {
  using K = KOwn<N, NT>;
  constexpr size_t PL = size_t(N) * N, NG = PL * N;
  double2 acc[K::PTS];
#pragma unroll
  for (int q = 0; q < K::PTS; ++q) acc[q].x = acc[q].y = 0.0;
  for (int a = a0; a < a1; ++a) {
    // an opaque copy of the thread index keeps the transforms' index
    // arithmetic inside the loop (hoisted, it would all stay live)
    int t = tid;
    asm volatile("" : "+v"(t));
    const int p = adj[2 * a], j = adj[2 * a + 1];
    body_kinv_acc<N, NT>(spec + size_t(p) * NG + z * PL, u + size_t(j) * NG + z * PL, j > k, buf, tw, t, acc);
  }
#pragma unroll
  for (int s = 0; s < K::PER; ++s) {
    const int b = tid + s * NT;
    if (K::TOT % NT == 0 || b < K::TOT) {
      const int l = b % N, j = b / N;
#pragma unroll
      for (int r = 0; r < K::R; ++r) {
        double2* w = wk + z * PL + (j + r * K::NB) * N + l;
        double2 o;
        o.x = o.y = 0.0;
        if (add) o = *w;
        o.x -= c * acc[s * K::R + r].x;
        o.y -= c * acc[s * K::R + r].y;
        *w = o;
      }
    }
  }
}

}  // namespace ace

// Checks of the pair energies that the z pass over row classes sums (pair_phases.h,
// body_conv_z_c with an energy slot), built for the host against
// tests/cpu_fft/hip/hip_runtime.h and run with one thread: the tiles' sums over a
// whole field, ragged last tile and real-spectrum weights included, against
// sum_G v |rho(G)|^2 over all G from a naive DFT.
#include <cmath>
#include <complex>
#include <cstdint>
#include <cstdio>
#include <vector>

#include "../../paper_2101_03155_amd/csrc/pair_phases.h"

using namespace ace;
using cd = std::complex<double>;
static int failures = 0;
static double uni(unsigned& s) { return ((s = s * 1664525u + 1013904223u) >> 8) / double(1 << 24) - 0.5; }

template <int N>
void dft_axis(std::vector<cd>& a, size_t st) {
  std::vector<cd> w(N), col(N), out(N);
  for (int m = 0; m < N; ++m) w[m] = std::polar(1.0, -2.0 * M_PI * m / N);
  for (size_t b = 0; b < a.size(); ++b) {
    if ((b / st) % N != 0) continue;
    for (int i = 0; i < N; ++i) col[i] = a[b + i * st];
    for (int k = 0; k < N; ++k) {
      cd acc = 0;
      for (int i = 0; i < N; ++i) acc += col[i] * w[(long(i) * k) % N];
      out[k] = acc;
    }
    for (int k = 0; k < N; ++k) a[b + k * st] = out[k];
  }
}

template <typename T, int N, int YC, int TX>
void check(double tol) {
  constexpr int XS = N / 2 + 1, NY = N / YC, CP = NY * XS, H = NY / 2, PP = cls_pitch<T, N, YC>(), HV = N / 2 + 1;
  constexpr size_t P2 = size_t(N) * N, NG = P2 * N, PL = size_t(YC) * PP;
  std::vector<T> pi(NG), pj(NG), vt(size_t(HV) * HV * XS);
  unsigned s = 23u + N;
  for (size_t e = 0; e < NG; ++e) { pi[e] = T(uni(s)); pj[e] = T(uni(s)); }
  std::vector<cplx<T>> tw(N), spec(N * PL), buf(std::max<size_t>(size_t(H) * (N + 1) + CP, size_t(N) * TX * YC));
  for (int m = 0; m < N; ++m) { tw[m].x = T(std::cos(-2.0 * M_PI * m / N)); tw[m].y = T(std::sin(-2.0 * M_PI * m / N)); }
  KernelParams kp{1, 0.37, 1.0 / double(NG), {0.41, 0.43, 0.47}};
  std::vector<cd> f(NG);
  for (size_t e = 0; e < NG; ++e) f[e] = double(pi[e]) * double(pj[e]);
  for (size_t st : {size_t(1), size_t(N), P2}) dft_axis<N>(f, st);
  double want = 0;
  for (int z = 0; z < N; ++z)
    for (int y = 0; y < N; ++y)
      for (int x = 0; x < N; ++x) want += kernel_value<double, N>(kp, x, y, z) * std::norm(f[z * P2 + y * N + x]);
  for (int z = 0; z < N; ++z)
    for (int c = 0; c < YC; ++c)
      body_fwd_xy_r<T, N, 1, 0, YC>(pi.data() + z * P2 + c * N, pj.data() + z * P2 + c * N,
                                    spec.data() + z * PL + size_t(c) * PP, buf.data(), tw.data(), 0);
  for (size_t e = 0; e < vt.size(); ++e)
    vt[e] = kernel_value<T, N>(kp, int(e % XS), int(e / XS % HV), int(e / (XS * HV)));
  static T vv[conv_lv_c<T, N, TX, YC, 1>()];
  double got = 0;
  for (int f0 = 0; f0 < CP; f0 += TX) {
    double slot = 0, red[4] = {0, 0, 0, 0};
    load_vtile_c<T, N, TX, YC, 1>(vt.data(), f0, 0, vv);
    body_conv_z_c<T, N, TX, YC, 1>(spec.data(), f0, buf.data(), tw.data(), 0, &slot, red, vv);
    // the wave's sum: the host's shuffles return the own value, so its six steps
    // give 64 times this one thread's
    got += red[0] / 64;
  }
  const double err = std::abs(got - want) / want;
  const bool ok = err <= tol;
  failures += !ok;
  std::printf("row class energy N=%3d YC=%d TX=%2d fp%d rel err %.2e %s\n", N, YC, TX, int(8 * sizeof(T)), err,
              ok ? "ok" : "FAIL");
}

int main() {
  check<double, 48, 2, 16>(1e-13);
  check<double, 80, 4, 8>(1e-13);
  check<double, 100, 2, 16>(1e-13);  // 50 x 51 columns: ragged last tile
  check<double, 108, 2, 16>(1e-13);
  return failures;
}

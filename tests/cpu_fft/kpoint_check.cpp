// Checks of the k-point pair-stage bodies (kpoint_phases.h), built for the
// host against tests/cpu_fft/hip/hip_runtime.h and run with one thread: the
// forward in-plane pass, the z pass with v(|G + d|) and the inverse with its
// accumulation, over a whole field, against separable naive DFTs written from
// the definition.  Prints one line per check; non-zero exit on a failure.
#include <cmath>
#include <complex>
#include <cstdint>
#include <cstdio>
#include <vector>

#include "../../paper_2101_03155_amd/csrc/kpoint_phases.h"

using namespace ace;
using cd = std::complex<double>;
static int failures = 0;
static double uni(unsigned& s) { return ((s = s * 1664525u + 1013904223u) >> 8) / double(1 << 24) - 0.5; }

// naive DFT of sign S along the axis of pitch `st`, in place
template <int N>
void dft_axis(std::vector<cd>& a, size_t st, int S) {
  std::vector<cd> w(N), col(N), out(N);
  for (int m = 0; m < N; ++m) w[m] = std::polar(1.0, S * 2.0 * M_PI * m / N);
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

template <int N>
void check(int kind) {
  constexpr size_t PL = size_t(N) * N, NG = PL * N;
  constexpr int TX = kconv_tx<N>();
  std::vector<double2> ua(NG), ub(NG), spec(NG), buf(std::max<size_t>(N * (N + 1), N * TX)), tw(N);
  unsigned s = 99u + N;
  for (auto* v : {&ua, &ub})
    for (auto& c : *v) { c.x = uni(s); c.y = uni(s); }
  for (int m = 0; m < N; ++m) { tw[m].x = std::cos(-2.0 * M_PI * m / N); tw[m].y = std::sin(-2.0 * M_PI * m / N); }
  KernelParams kp{kind, 0.37, 1.0 / double(NG), {0.41, 0.43, 0.47}};
  const double d[3] = {0.11, -0.07, 0.0};
  // reference potential
  std::vector<cd> f(NG);
  for (size_t e = 0; e < NG; ++e) f[e] = std::conj(cd(ua[e].x, ua[e].y)) * cd(ub[e].x, ub[e].y);
  for (size_t st : {size_t(1), size_t(N), PL}) dft_axis<N>(f, st, -1);
  for (int z = 0; z < N; ++z)
    for (int y = 0; y < N; ++y)
      for (int x = 0; x < N; ++x) f[z * PL + y * N + x] *= kernel_value_shift<N>(kp, d, x, y, z);
  for (size_t st : {size_t(1), size_t(N), PL}) dft_axis<N>(f, st, 1);
  // the passes
  for (int z = 0; z < N; ++z)
    body_kfwd_xy<N, 1>(ua.data() + z * PL, ub.data() + z * PL, spec.data() + z * PL, buf.data(), tw.data(), 0);
  static double vv[kconv_lv<N, TX, 1>()];
  for (size_t f0 = 0; f0 < PL; f0 += TX) {
    load_kvtile<N, TX, 1>(kp, d, int(f0), 0, vv);
    body_kconv_z<N, TX, 1>(spec.data() + f0, buf.data(), tw.data(), 0, vv);
  }
  using K = KOwn<N, 1>;
  static double2 acc[K::PTS];
  double err = 0, mx = 0;
  for (bool conj : {false, true}) {
    for (int z = 0; z < N; ++z) {
      for (auto& a : acc) a.x = a.y = 0.0;
      body_kinv_acc<N, 1>(spec.data() + z * PL, ua.data() + z * PL, conj, buf.data(), tw.data(), 0, acc);
      for (int b = 0; b < K::TOT; ++b)
        for (int r = 0; r < K::R; ++r) {
          const size_t e = z * PL + size_t(b / N + r * K::NB) * N + b % N;
          const cd want = cd(ua[e].x, ua[e].y) * (conj ? std::conj(f[e]) : f[e]);
          err = std::max(err, std::abs(cd(acc[b * K::R + r].x, acc[b * K::R + r].y) - want));
          mx = std::max(mx, std::abs(want));
        }
    }
  }
  const bool ok = err <= 1e-13 * mx;
  failures += !ok;
  std::printf("k-point pair stage N=%3d kind %d rel err %.2e %s\n", N, kind, err / mx, ok ? "ok" : "FAIL");
}

int main() {
  check<8>(0); check<12>(1); check<16>(0); check<24>(1); check<32>(0); check<48>(1); check<64>(0);
  return failures;
}

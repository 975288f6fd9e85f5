// Checks of the owner pass (pair_phases.h, body_inv_owner_r), built for the
// host against tests/cpu_fft/hip/hip_runtime.h and run with one thread: both
// forms of its product (kept in the last pass, or from the finished plane) against
// the inverse transform of each pair's plane followed by the products, with
// several pairs per owner, every plan length (one, two and three passes), row
// classes, and the reversed plan order.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <vector>

#include "../../paper_2101_03155_amd/csrc/pair_phases.h"

using namespace ace;
static int failures = 0;
static double uni(unsigned& s) { return ((s = s * 1664525u + 1013904223u) >> 8) / double(1 << 24) - 0.5; }

template <typename T, int N, int V, int YC>
void check(double tol) {
  constexpr int XS = N / 2 + 1, NY = N / YC, H = NY / 2, PP = cls_pitch<T, N, YC>(), NP = 3, NORB = 4;
  constexpr size_t P2 = size_t(N) * N, NG = P2 * N, PL = size_t(YC) * PP;
  const int z = N / 3;
  unsigned s = 5u + N;
  // only plane z of each pair's spectrum and of each orbital is read
  std::vector<cplx<T>> spec(NP * N * PL), tw(N), buf(size_t(H) * (N + 1) + size_t(NY) * XS);
  std::vector<T> phi(NORB * NG), W(NG, T(99)), ref(P2, T(0));
  for (int p = 0; p < NP; ++p)
    for (size_t e = 0; e < PL; ++e) {
      spec[(size_t(p) * N + z) * PL + e].x = T(uni(s));
      spec[(size_t(p) * N + z) * PL + e].y = T(uni(s));
    }
  for (int j = 0; j < NORB; ++j)
    for (size_t e = 0; e < P2; ++e) phi[j * NG + z * P2 + e] = T(uni(s));
  for (int m = 0; m < N; ++m) { tw[m].x = T(std::cos(-2.0 * M_PI * m / N)); tw[m].y = T(std::sin(-2.0 * M_PI * m / N)); }
  const int32_t adj[] = {1, 3, 0, 0, 2, 1, 1, 2};
  const int na = 4;
  for (int c = 0; c < YC; ++c)
    for (int a = 0; a < na; ++a) {
      body_inv_xy_g<T, N, 1, V, YC>(spec.data() + (size_t(adj[2 * a]) * N + z) * PL + size_t(c) * PP, buf.data(),
                                    tw.data(), 0);
      const T* f = phi.data() + adj[2 * a + 1] * NG + z * P2;
      for (int l = 0; l < H; ++l)
        for (int x = 0; x < N; ++x) {
          const auto v = buf[xpos<N>(l * N + x)];
          const size_t e0 = size_t(c + YC * l) * N + x, e1 = size_t(c + YC * (l + H)) * N + x;
          ref[e0] -= v.x * f[e0];
          ref[e1] -= v.y * f[e1];
        }
    }
  for (int c = 0; c < YC; ++c)
    body_inv_owner_r<T, N, 1, V, YC, PP>(phi.data(), spec.data(), adj, 0, na, z * P2, W.data() + z * P2 + c * N,
                                         buf.data(), tw.data(), 0, c);
  double err = 0, mx = 0;
  for (size_t e = 0; e < NG; ++e) {
    const bool in = e / P2 == size_t(z);
    const double want = in ? double(ref[e % P2]) : 99.0;
    err = std::max(err, std::abs(double(W[e]) - want));
    if (in) mx = std::max(mx, std::abs(want));
  }
  const bool ok = err <= tol * mx;
  failures += !ok;
  std::printf("owner N=%3d V=%d YC=%d fp%d fused=%d rel err %.2e %s\n", N, V, YC, int(8 * sizeof(T)),
              int(own_fused<T, N, YC>()), err / mx, ok ? "ok" : "FAIL");
}

int main() {
  // the same sums in the same order: equal up to fused multiply-adds
  constexpr double D = 1e-15, F = 5e-7;
  check<float, 8, 0, 1>(F);
  check<float, 12, 1, 1>(F);
  check<float, 16, 0, 1>(F);
  check<double, 8, 0, 1>(D);
  check<double, 16, 0, 1>(D);
  check<float, 24, 0, 1>(F);
  check<double, 24, 1, 1>(D);
  check<double, 48, 0, 1>(D);
  check<float, 96, 0, 1>(F);
  check<double, 96, 0, 1>(D);
  check<double, 96, 0, 2>(D);
  check<double, 100, 0, 2>(D);
  check<float, 108, 0, 1>(F);
  check<double, 108, 0, 2>(D);
  check<float, 120, 0, 1>(F);
  check<double, 160, 1, 4>(D);
  return failures;
}

// Checks of the owner tables of the k-point build (kpoint_tables.h) on the host:
// against one scan of the whole list per chunk, for random pair lists and chunks
// of one slot to all, and the time of a long list in many chunks.  Prints one line
// per check; non-zero exit on a failure.
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <random>

#include "../../paper_2101_03155_amd/csrc/kpoint_tables.h"

using namespace ace;
static int failures = 0;
typedef std::vector<int32_t> Ints;

// adjacency of the pairs i <= j taken with probability p, each owner's entries
// in a shuffled order
static int64_t adjacency(int n, double p, unsigned seed, Ints& ptr, Ints& adj, Ints& perm) {
  std::mt19937 g(seed);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  std::vector<std::vector<std::pair<int32_t, int32_t>>> e(static_cast<size_t>(n));
  int32_t t = 0;
  for (int i = 0; i < n; ++i)
    for (int j = i; j < n; ++j)
      if (i == j || u(g) < p) {
        e[size_t(i)].emplace_back(t, j);
        if (i != j) e[size_t(j)].emplace_back(t, i);
        ++t;
      }
  ptr.assign(1, 0);
  adj.clear();
  for (auto& v : e) {
    std::shuffle(v.begin(), v.end(), g);
    for (auto& x : v) {
      adj.push_back(x.first);
      adj.push_back(x.second);
    }
    ptr.push_back(int32_t(adj.size() / 2));
  }
  perm.resize(size_t(n));
  for (int k = 0; k < n; ++k) perm[size_t(k)] = n - 1 - k;
  return t;
}

static void check(int n, double p, int64_t chunk) {
  Ints ptr, adj, perm, tab, want, ent;
  const int64_t np = adjacency(n, p, unsigned(n), ptr, adj, perm);
  chunk = std::min(chunk, np);
  const int64_t nchunk = (np + chunk - 1) / chunk;
  for (int64_t q = 0; q < nchunk; ++q) {
    for (int k = 0; k < n; ++k) {
      want.push_back(int32_t(ent.size() / 2));
      for (int a = ptr[size_t(k)]; a < ptr[size_t(k) + 1]; ++a) {
        const int64_t s = adj[size_t(2 * a)] - q * chunk;
        if (s < 0 || s >= chunk) continue;
        ent.push_back(int32_t(s));
        ent.push_back(adj[size_t(2 * a + 1)]);
      }
    }
    want.push_back(int32_t(ent.size() / 2));
  }
  const size_t eo = want.size(), po = eo + ent.size();
  want.insert(want.end(), ent.begin(), ent.end());
  want.insert(want.end(), perm.begin(), perm.end());
  size_t ent_off = 0, perm_off = 0;
  make_kowner_tables(ptr, adj, perm, chunk, nchunk, n, tab, &ent_off, &perm_off);
  const bool ok = tab == want && ent_off == eo && perm_off == po;
  failures += !ok;
  std::printf("tables n=%d pairs=%lld chunk=%lld %s\n", n, (long long)np, (long long)chunk, ok ? "ok" : "FAIL");
}

int main() {
  check(1, 1.0, 1);
  check(7, 0.5, 1);
  check(7, 0.5, 3);
  check(40, 0.1, 32);
  check(40, 1.0, 100);
  check(40, 1.0, 819);
  check(40, 1.0, 820);
  // 512 orbitals, every pair, 4104 chunks: a scan of the list per chunk is 1e9 steps
  Ints ptr, adj, perm, tab;
  const int64_t np = adjacency(512, 1.0, 5, ptr, adj, perm);
  size_t eo, po;
  double best = 1e9;
  for (int r = 0; r < 3; ++r) {
    const auto t0 = std::chrono::steady_clock::now();
    make_kowner_tables(ptr, adj, perm, 32, (np + 31) / 32, 512, tab, &eo, &po);
    best = std::min(best, std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count());
  }
  const bool ok = best < 0.3;
  failures += !ok;
  std::printf("512 orbitals in chunks of 32: %.1f ms %s\n", 1e3 * best, ok ? "ok" : "FAIL");
  return failures;
}

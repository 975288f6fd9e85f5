// Host tables of the owner-computes k-point build over chunks of pairs.
#pragma once
#include <cstddef>
#include <cstdint>
#include <vector>

namespace ace {

// The entries (slot, partner) adj[2 a], adj[2 a + 1], a = adj_ptr[k] .. adj_ptr[k + 1]
// of every owner k, dealt to chunks of `chunk` slots.  tab holds per chunk its
// offsets (ntot + 1 of them, into all entries), then every chunk's entries by
// owner, each owner's in their order and by chunk-local slot, then operm.
// *ent_off and *perm_off are the places of the latter two in tab.
inline void make_kowner_tables(const std::vector<int32_t>& adj_ptr, const std::vector<int32_t>& adj,
                               const std::vector<int32_t>& operm, int64_t chunk, int64_t nchunk, int ntot,
                               std::vector<int32_t>& tab, size_t* ent_off, size_t* perm_off) {
  const size_t np1 = size_t(ntot) + 1;
  *ent_off = size_t(nchunk) * np1;
  *perm_off = *ent_off + adj.size();
  tab.assign(*perm_off + operm.size(), 0);
  // counts at the place of the following offset, their sums, and the entries at
  // each owner's next place; the offsets then stand one place ahead
  for (int k = 0; k < ntot; ++k)
    for (int32_t a = adj_ptr[size_t(k)]; a < adj_ptr[size_t(k) + 1]; ++a)
      ++tab[size_t(adj[size_t(2 * a)] / chunk) * np1 + size_t(k)];
  int32_t sum = 0;
  for (size_t e = 0; e < *ent_off; ++e) {
    const int32_t n = tab[e];
    tab[e] = sum;
    sum += n;
  }
  std::vector<int32_t> at(tab.begin(), tab.begin() + std::ptrdiff_t(*ent_off));
  for (int k = 0; k < ntot; ++k)
    for (int32_t a = adj_ptr[size_t(k)]; a < adj_ptr[size_t(k) + 1]; ++a) {
      const int32_t slot = adj[size_t(2 * a)];
      const int64_t q = slot / chunk;
      const size_t p = *ent_off + 2 * size_t(at[size_t(q) * np1 + size_t(k)]++);
      tab[p] = int32_t(slot - q * chunk);
      tab[p + 1] = adj[size_t(2 * a + 1)];
    }
  for (size_t k = 0; k < operm.size(); ++k) tab[*perm_off + k] = operm[k];
}

}  // namespace ace

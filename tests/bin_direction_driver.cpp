// Reads, for each field, the number of blocks and the counts [blocks][9] (8 bins
// and a flag) as text, and prints 1 where bins_grow, else 0. TEST
// INFRASTRUCTURE ONLY.
#include <cstdio>
#include <vector>

#include "bin_direction.hpp"

int main() {
  int nblk;
  while (std::scanf("%d", &nblk) == 1) {
    std::vector<int> cnt(static_cast<size_t>(nblk) * 9);
    for (int& c : cnt)
      if (std::scanf("%d", &c) != 1) return 1;
    chem_model::BinSums s[chem_model::kDirBins];
    for (int b = 0; b < chem_model::kDirBins; ++b) s[b] = chem_model::bin_sums(cnt.data(), 9, nblk, b);
    std::printf("%d\n", chem_model::bins_grow(s) ? 1 : 0);
  }
  return 0;
}

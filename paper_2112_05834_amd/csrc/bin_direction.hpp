// Which way the costs of the binned schedule run over the cell index, from the
// counts of every block of cells in every bin. Plain integer arithmetic, the same
// on host and device.
#pragma once

namespace chem_model {

constexpr int kDirBins = 8;

// One bin's cells, and their blocks summed. cnt: nblk rows of stride entries.
struct BinSums {
  long long cells, blocks;
};
constexpr BinSums bin_sums(const int* cnt, int stride, int nblk, int bin) {
  BinSums s{0, 0};
  for (int k = 0; k < nblk; ++k) {
    s.cells += cnt[k * static_cast<long long>(stride) + bin];
    s.blocks += static_cast<long long>(k) * cnt[k * static_cast<long long>(stride) + bin];
  }
  return s;
}

// Whether cells' bins grow with their blocks: the sign of N^2 times the covariance
// of block and bin over the cells, N sum(k b) - sum(k) sum(b), about the means of
// the cells (the last block may hold fewer). Up to 2^31 cells in blocks of 4096 it
// stays below 2^85. One block alone has no direction.
constexpr bool bins_grow(const BinSums (&s)[kDirBins]) {
  long long n = 0, sk = 0, sb = 0, skb = 0;
  for (int b = 0; b < kDirBins; ++b) {
    n += s[b].cells;
    sk += s[b].blocks;
    sb += b * s[b].cells;
    skb += b * s[b].blocks;
  }
  return static_cast<__int128>(n) * skb - static_cast<__int128>(sk) * sb > 0;
}

}  // namespace chem_model

// Checks the split of the backward pass's dH contraction for any number of
// scored rows (csrc/hdl_internal.h): it fits the partial sums' memory and the
// launch made for all rows, covers the vocabulary slices, deals every item once
// and the XCDs equal shares (to within one run of 32), costs no more than the
// split made for all rows, and is that one when every row is scored.
// Arguments: n_rows d vocab.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_2609_36864_amd/csrc/hdl_internal.h"

using namespace hdl;

int main(int argc, char** argv) {
  if (argc != 4) return 2;
  const int64_t n_rows = std::atoll(argv[1]), d = std::atoll(argv[2]), vocab = std::atoll(argv[3]);
  const int64_t slices = ceil_div(vocab, 64), all_m = ceil_div(n_rows, kTileV), tiles_n = ceil_div(d, kTileN);
  const int64_t all_splits = best_split(all_m, tiles_n, slices, INT64_MAX), room = all_splits * all_m;
  const int64_t grid = ceil_div(all_m * tiles_n * all_splits, 256) * 256;
  for (int64_t n = 1; n <= n_rows; n += 1 + n_rows / 61) {
    GemmArgs p{};
    p.k = slices * 64;
    p.ldc = d;
    p.tiles_m = all_m;
    p.tiles_n = tiles_n;
    p.gn = std::min<int64_t>(tiles_n, 4);
    p.gm = std::min<int64_t>(32 / p.gn, all_m);
    const int64_t splits = best_split(ceil_div(n, kTileV), tiles_n, slices, room);
    dh_live(&p, n, splits);
    auto bad = [&](const char* what) {
      std::printf("n=%lld: %s (splits %lld)\n", (long long)n, what, (long long)splits);
      return 1;
    };
    if (n > n_rows - 256 && n > (all_m - 1) * kTileV && splits != all_splits) return bad("not the split of all rows");
    if (p.c_split_stride * splits > room * kTileV * d || p.c_split_stride < n * d) return bad("partial sums");
    if (p.tiles_m * kTileV < n || p.tiles_m * tiles_n * splits > grid) return bad("grid");
    if (p.k_split % 64 != 0 || p.k_split * splits < p.k || (splits - 1) * p.k_split >= p.k) return bad("slices");
    if (split_cost(p.tiles_m * tiles_n, slices, splits) > split_cost(p.tiles_m * tiles_n, slices, all_splits))
      return bad("dearer than the split of all rows");
    std::vector<int> seen(p.tiles_m * tiles_n * splits, 0);
    std::vector<int64_t> share(kNumXcd, 0);
    for (int64_t b = 0; b < grid; ++b) {
      const int64_t j = b / kNumXcd;
      int64_t tm, tn, s;
      if (!gemm_item(((j / 32) * kNumXcd + b % kNumXcd) * 32 + j % 32, p, &tm, &tn, &s)) continue;
      ++seen[(s * p.tiles_m + tm) * tiles_n + tn];
      ++share[b % kNumXcd];
    }
    for (int c : seen)
      if (c != 1) return bad("an item is not taken once");
    const auto mm = std::minmax_element(share.begin(), share.end());
    if (*mm.second - *mm.first > 32) return bad("uneven shares");
  }
  return 0;
}

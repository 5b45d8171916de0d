// Enumerates the GEMM's work items (csrc/hdl_internal.h) and checks that every
// (split, m tile, n tile) comes exactly once and nothing after the last.
// Arguments: tiles_m tiles_n splits gm gn.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_2609_36864_amd/csrc/hdl_internal.h"

int main(int argc, char** argv) {
  if (argc != 6) return 2;
  hdl::GemmArgs g{};
  g.tiles_m = std::atoll(argv[1]);
  g.tiles_n = std::atoll(argv[2]);
  g.splits = std::atoll(argv[3]);
  g.gm = std::atoll(argv[4]);
  g.gn = std::atoll(argv[5]);
  const int64_t n = g.tiles_m * g.tiles_n * g.splits;
  std::vector<int> seen(n, 0);
  for (int64_t at = 0; at < n + 600; ++at) {
    int64_t m, c, s;
    const bool in = hdl::gemm_item(at, g, &m, &c, &s);
    if (in != (at < n)) return std::printf("item %lld: in = %d\n", (long long)at, in), 1;
    if (!in) continue;
    if (m < 0 || m >= g.tiles_m || c < 0 || c >= g.tiles_n || s < 0 || s >= g.splits)
      return std::printf("item %lld: tile %lld %lld split %lld\n", (long long)at, (long long)m, (long long)c, (long long)s), 1;
    if (seen[(s * g.tiles_m + m) * g.tiles_n + c]++) return std::printf("item %lld: again\n", (long long)at), 1;
  }
  return 0;
}

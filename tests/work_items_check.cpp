// CPU check of the work-item order (csrc/plan.h) for any number of scored
// rows of a launch: every (row tile, chunk) is produced exactly once by the
// launched workgroups, the XCDs get equal shares (to within one run of 32),
// and any whole run of 32 items reads at most 20 different tiles (12 in a whole
// block) once there are that many chunks.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <set>
#include <vector>

#include "../paper_2609_36864_amd/csrc/plan.h"

using namespace hdl;

static int check(int64_t n_rows, int64_t vocab, int64_t d, bool bf16) {
  const LmheadPlan p = make_plan(n_rows, vocab, d, bf16 ? 2 : 4);
  const int64_t grid = launch_grid(p, n_rows);
  for (int64_t n_s = 1; n_s <= n_rows; n_s += 1 + n_rows / 199) {
    const ItemGrid g = item_grid(n_s, p.n_ch, bf16);
    std::vector<int> seen(static_cast<size_t>(g.n_rt * g.n_ch), 0);
    std::vector<int64_t> share(kNumXcd, 0);
    for (int64_t b = 0; b < grid; ++b) {
      int64_t rt, ch;
      work_item(b, g, &rt, &ch);
      if (rt >= g.n_rt) continue;
      if (ch < 0 || ch >= g.n_ch || rt < 0) return std::printf("item out of range\n"), 1;
      ++seen[static_cast<size_t>(rt * g.n_ch + ch)];
      ++share[b % kNumXcd];
    }
    for (int c : seen)
      if (c != 1) return std::printf("n_s=%lld: an item is taken %d times\n", (long long)n_s, c), 1;
    const auto mm = std::minmax_element(share.begin(), share.end());
    if (*mm.second - *mm.first > 32) return std::printf("n_s=%lld: uneven shares\n", (long long)n_s), 1;
    if (g.n_ch % kGroupCH == 0 && g.n_ch >= 32)
      for (int64_t run = 0; run < g.n_rt * g.n_ch / 32; ++run) {
        std::set<int64_t> rts, chs;
        for (int64_t i = 0; i < 32; ++i) {
          int64_t rt, ch;
          work_item(((run / kNumXcd) * 32 + i) * kNumXcd + run % kNumXcd, g, &rt, &ch);
          rts.insert(rt);
          chs.insert(ch);
        }
        if (g.n_rt >= 3 && rts.size() + chs.size() > 20)
          return std::printf("n_s=%lld run %lld: %zu + %zu tiles\n", (long long)n_s, (long long)run, rts.size(), chs.size()), 1;
      }
  }
  return 0;
}

int main(int argc, char** argv) {
  if (argc != 4) return 2;
  for (bool bf16 : {true, false})
    if (check(std::atoll(argv[1]), std::atoll(argv[2]), std::atoll(argv[3]), bf16) != 0) return 1;
  std::printf("ok\n");
  return 0;
}

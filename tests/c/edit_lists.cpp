// The upload image of edit lists around the length from which the kernel that
// reads overlap lists takes over: a shorter list carries none (its edits,
// rectangles and patches alone), a longer one those of every edit.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "tc_plan.h"

int main() {
  int fails = 0;
  size_t words = 0;
  const int32_t W = 3000, H = 2000;
  const tci_map d = tci::layout_map(W, H, &words);
  std::srand(5);
  for (int32_t n : {1, 2, 64, 65, 400, tci::kTileEdits, tci::kTileEdits + 1, 2000}) {
    std::vector<tc_edit> e(n);
    for (tc_edit& x : e) {
      x = tc_edit{};
      x.kind = TC_EDIT_CRATER;
      x.w = x.h = 1 + std::rand() % 90;
      x.x0 = std::rand() % (W + 100) - 100;
      x.y0 = std::rand() % 400 - 50;
      x.depth = 3;
    }
    tci::EditPlan sized, p;
    tci::plan_edits(d, e.data(), n, 0, nullptr, sized);
    std::vector<char> host(sized.total);
    tci::plan_edits(d, e.data(), n, 0, host.data(), p);
    const bool lists = n > tci::kTileEdits;
    if (p.total != sized.total || p.olap_all == lists || (lists ? p.olap.size() < (size_t)n + 1
                                                                : p.olap.size() != (size_t)n + 1)) {
      std::printf("n %d: %zu words of lists, all %d\n", n, p.olap.size(), (int)p.olap_all);
      ++fails;
      continue;
    }
    const int32_t* ol = reinterpret_cast<const int32_t*>(host.data() + p.off_olap);
    for (int32_t i = 0; lists && i < n; ++i) {
      auto clip = [&](const tc_edit& x, int32_t c[4]) {
        c[0] = std::max(x.x0, 0);
        c[1] = std::max(x.y0, 0);
        c[2] = std::min(x.x0 + x.w, W);
        c[3] = std::min(x.y0 + x.h, H);
        return c[0] < c[2] && c[1] < c[3];
      };
      int32_t a[4], c[4];
      std::vector<int32_t> want;
      if (clip(e[i], a))
        for (int32_t j = 0; j < n; ++j)
          if (j != i && clip(e[j], c) && a[0] < c[2] && c[0] < a[2] && a[1] < c[3] && c[1] < a[3])
            want.push_back(j);
      if (ol[i + 1] - ol[i] != (int32_t)want.size() ||
          !std::equal(want.begin(), want.end(), ol + n + 1 + ol[i])) {
        std::printf("n %d: list of edit %d\n", n, i);
        ++fails;
        break;
      }
    }
  }
  std::printf("%d failures\n", fails);
  return fails != 0;
}

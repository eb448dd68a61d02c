// The dealing of a launch's tiles over the XCDs, against the ranges of work units
// that the kernels give them: XCD x of 8 takes the units from x q + min(x, r) on,
// q and r the quotient and remainder of the units by 8.
#include "api_stub.h"

#include <random>

int main() {
  std::mt19937 rng(7);
  int bad = 0;
  for (int bpt : {1, 2, 8, 16, 32})
    for (int n = 1; n <= wv::kArgItems; ++n) {
      std::vector<wv::Item> src(n);
      const int top = 1 + rng() % 8;
      std::vector<int> sorted(n);
      for (int i = 0; i < n; ++i) {
        src[i] = wv::Item{(uint16_t)(2 * i), (uint16_t)i, 0, (uint8_t)(rng() % (top + 1)), 0};
        sorted[i] = src[i].lc;
      }
      std::sort(sorted.begin(), sorted.end(), std::greater<int>());
      wv::WorkArgs a;
      memset(&a, 0, sizeof a);
      a.bx = 1;
      a.by = bpt;
      copy_items(src.data(), n, a);
      bad += check(a.n_items == n && a.total == n * bpt, "the launch's size");
      std::vector<int> seen(n, 0);
      for (int i = 0; i < n; ++i) {
        const wv::Item& it = a.items[i];
        if (it.slot < n && it.tile == 2 * it.slot && it.lc == src[it.slot].lc) ++seen[it.slot];
      }
      bad += check(std::count(seen.begin(), seen.end(), 1) == n, "every tile once, in its own slot");
      if (n <= 8 || sorted.front() == sorted.back()) continue;
      // every range starts with a tile of the most levels and goes down alike:
      // the k-th tiles of the ranges are the tiles 8 k .. 8 k + 7 by level count
      int first[9];
      for (int x = 0; x <= 8; ++x) {
        const int unit = x * (a.total / 8) + std::min(x, a.total % 8);
        first[x] = (unit + bpt - 1) / bpt;
      }
      for (int k = 0; 8 * k < n; ++k) {
        std::vector<int> got;
        for (int x = 0; x < 8; ++x)
          if (first[x] + k < first[x + 1]) got.push_back(a.items[first[x] + k].lc);
        std::sort(got.begin(), got.end(), std::greater<int>());
        const std::vector<int> want(sorted.begin() + 8 * k, sorted.begin() + std::min(n, 8 * k + 8));
        if (got != want) {
          bad += check(false, "the XCDs' ranges hold the same mix");
          std::printf("  %d tiles of %d units, position %d\n", n, bpt, k);
          break;
        }
      }
      if (bad > 20) return bad;
    }
  if (!bad) std::printf("ok\n");
  return bad;
}

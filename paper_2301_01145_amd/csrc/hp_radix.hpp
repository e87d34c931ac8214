// Radix orders that the autotuner tries on a pass of the general kernels.
#pragma once

#include <algorithm>
#include <vector>

namespace hp {

// Orders of the stages of a length-L transform: the planner's own (`own`) first,
// then the factorisations over 2 .. top (the radices with a register stage) of the
// fewest stages and of one more, smallest sums first (balanced stages), the
// leading ones also in ascending order.  Prime factors above `top` come first,
// as in the planner's order; at most max_stages stages.
inline std::vector<std::vector<int>> radix_orders(int L, int top, int max_stages, const std::vector<int>& own) {
  constexpr size_t kTried = 10, kAscending = 3;
  std::vector<std::vector<int>> out;
  auto add = [&](const std::vector<int>& o) {
    if (!o.empty() && std::find(out.begin(), out.end(), o) == out.end()) out.push_back(o);
  };
  add(own);
  std::vector<int> big;
  int rest = L;
  for (int f = 2, r = L; r > 1; ++f) {
    if ((long long)f * f > r) f = r;
    while (r % f == 0) {
      if (f > top) big.push_back(f), rest /= f;
      r /= f;
    }
  }
  std::vector<std::vector<int>> all;
  std::vector<int> cur;
  auto split = [&](auto&& self, int r, int limit) -> void {
    if (r == 1) {
      all.push_back(cur);
      return;
    }
    if ((int)(big.size() + cur.size()) >= max_stages) return;
    for (int f = std::min(limit, r); f >= 2; --f) {
      if (r % f) continue;
      cur.push_back(f);
      self(self, r / f, f);
      cur.pop_back();
    }
  };
  split(split, rest, top);
  auto sum = [](const std::vector<int>& v) {
    int s = 0;
    for (int x : v) s += x;
    return s;
  };
  std::sort(all.begin(), all.end(), [&](const std::vector<int>& a, const std::vector<int>& b) {
    return a.size() != b.size() ? a.size() < b.size() : sum(a) < sum(b);
  });
  for (size_t i = 0; i < all.size() && i < kTried && all[i].size() <= all[0].size() + 1; ++i) {
    std::vector<int> o = big;
    o.insert(o.end(), all[i].begin(), all[i].end());
    add(o);
    if (i < kAscending) {
      std::vector<int> up = big;
      up.insert(up.end(), all[i].rbegin(), all[i].rend());
      add(up);
    }
  }
  return out;
}

}  // namespace hp

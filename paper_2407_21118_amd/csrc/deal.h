// Workgroups for the units of one launch (host code, no device types: tests compile it by itself).
#pragma once

#include <algorithm>

namespace palu {

constexpr int kMaxDealUnits = 32;

// Deals at most `capacity` workgroups to n_units units of `tiles` tiles each, unit i costing cost[i] > 0 a tile: from least[i] each (at least
// 1, at most tiles), one at a time to the unit whose workgroups run longest, until that unit has one per tile or none is left.
// n[i] receives their numbers; returns their sum, or 0 where the least do not fit.
//
// One at a time from the start that is up to a workgroup per compute unit, each found among all units: 7.5 / 16 / 31 us of host time for 8 / 16 / 32
// units and 256 workgroups, where the launch they are for takes about 35.  Every state in which each unit has the fewest workgroups that
// keep its runs within one bound lies on that way, so it starts from such a state close to the end: 0.3 / 0.7 / 0.8 us, the same numbers.
inline int deal_workgroups(int n_units, int tiles, int capacity, const double* cost, const int* least, int* n) {
  auto run = [&](int count) { return (int)((unsigned)(tiles + count - 1) / (unsigned)count); };
  int total = 0;
  double work = 0.0;
  for (int i = 0; i < n_units; ++i) {
    total += n[i] = least[i];
    work += cost[i];
  }
  if (total > capacity) return 0;
  // No dealing brings all runs below this bound; the first multiple of it whose state fits
  double bound = work * tiles / capacity;
  for (int tries = 0; tries < 64; ++tries, bound *= 1.03) {
    int state[kMaxDealUnits], sum = 0;
    bool one_per_tile = false;
    for (int i = 0; i < n_units; ++i) {
      int longest = (int)(bound / cost[i]);                // longest run within the bound, in the arithmetic of the comparisons below
      while ((longest + 1) * cost[i] <= bound) ++longest;
      while (longest > 0 && longest * cost[i] > bound) --longest;
      one_per_tile |= longest == 0;                        // the dealing ends before it gets there
      sum += state[i] = std::max(least[i], longest > 0 ? run(longest) : tiles);
    }
    if (one_per_tile || sum > capacity) continue;
    std::copy(state, state + n_units, n);
    total = sum;
    break;
  }
  double us[kMaxDealUnits];
  for (int i = 0; i < n_units; ++i) us[i] = run(n[i]) * cost[i];
  for (;;) {
    int worst = 0;
    for (int i = 1; i < n_units; ++i) if (us[i] > us[worst]) worst = i;
    if (n[worst] >= tiles || total + 1 > capacity) return total;
    ++total;
    us[worst] = run(++n[worst]) * cost[worst];
  }
}

}  // namespace palu

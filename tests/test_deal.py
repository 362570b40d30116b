"""The host's dealing of workgroups to units of different cost (csrc/deal.h), compiled by itself, against the rule it states, one
workgroup at a time: the same numbers, in a fraction of that loop's time."""

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "deal.h"
#include <chrono>
#include <cstdio>
#include <random>

using palu::deal_workgroups;

static int one_at_a_time(int n_units, int tiles, int capacity, const double* cost, const int* least, int* n) {
  int total = 0;
  auto us = [&](int i) { return ((tiles + n[i] - 1) / n[i]) * cost[i]; };
  for (int i = 0; i < n_units; ++i) total += n[i] = least[i];
  if (total > capacity) return 0;
  for (;;) {
    int worst = 0;
    for (int i = 1; i < n_units; ++i) if (us(i) > us(worst)) worst = i;
    if (n[worst] >= tiles || total + 1 > capacity) return total;
    ++n[worst];
    ++total;
  }
}

int main() {
  std::mt19937 g(1);
  auto below = [&](int n) { return (int)(g() % n); };
  int wrong = 0;
  for (int t = 0; t < 40000; ++t) {
    const int n_units = 1 + below(palu::kMaxDealUnits), tiles = 1 + below(t % 3 ? 2000 : 64), capacity = n_units + below(t % 2 ? 256 : 40);
    double cost[palu::kMaxDealUnits];
    int least[palu::kMaxDealUnits], a[palu::kMaxDealUnits], b[palu::kMaxDealUnits];
    for (int i = 0; i < n_units; ++i) {
      cost[i] = t % 5 ? 30 + below(27) + 2.0 * (1 + below(16)) : 46.0;
      least[i] = t % 4 ? 1 : 1 + below(tiles);
    }
    const int x = one_at_a_time(n_units, tiles, capacity, cost, least, a), y = deal_workgroups(n_units, tiles, capacity, cost, least, b);
    bool same = x == y;
    for (int i = 0; i < n_units && same && x; ++i) same = a[i] == b[i];
    wrong += !same;
  }
  double us[2] = {1e9, 1e9};
  for (int rep = 0; rep < 20; ++rep)
    for (int which = 0; which < 2; ++which) {
      double cost[32];
      int least[32], n[32];
      for (int i = 0; i < 32; ++i) { cost[i] = 30 + (7 * i) % 27 + 2.0 * (1 + i % 8); least[i] = 1; }
      const auto t0 = std::chrono::steady_clock::now();
      int sum = 0;
      for (int r = 0; r < 50; ++r) { cost[0] += 1e-9 * (sum & 1); sum += (which ? deal_workgroups : one_at_a_time)(32, 512, 256, cost, least, n); }
      const double t = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count() * 1e6 / 50;
      if (t < us[which] && sum) us[which] = t;
    }
  std::printf("%d %.3f %.3f\n", wrong, us[0], us[1]);
}
"""


def test_dealing_of_workgroups(tmp_path):
    src = tmp_path / "deal.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "deal"
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2407_21118_amd", "csrc"), "-o", str(exe), str(src)], check=True)
    wrong, loop_us, us = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=120).stdout.split()
    print(f"one at a time {loop_us} us, dealt {us} us")
    assert int(wrong) == 0
    assert float(us) < float(loop_us) / 4          # measured: 1 / 38

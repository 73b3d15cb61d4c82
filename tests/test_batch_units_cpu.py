"""The choice of a batch's work items (csrc/launch_units.hpp), on the host: the
sums by numbers of rows choose as sums series by series do, and the series are
read a fixed number of times, however many sizes are tried."""

import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_1711_10855_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "launch_units.hpp"
using namespace fdas;
typedef std::pair<int64_t, int> Series;
// the same rule, each size summed series by series
static BatchUnits plain(const BatchModel &m, long slots, int cus, bool pair, double ragged,
                        const std::vector<Series> &s) {
  const int n = (int)s.size();
  int rows = 0, tail = n, tail_rows = 1;
  for (auto &x : s) rows = std::max(rows, x.second);
  double work = 0.0, head = 0.0;
  while (tail > 0 && (ragged > 0.0 || work < (double)slots * (rows + m.item))) {
    --tail;
    work += (double)s[tail].first * (s[tail].second + m.item);
    tail_rows = std::max(tail_rows, s[tail].second);
  }
  for (int k = 0; k < tail; ++k) head += (double)s[k].first * (s[k].second + m.item);
  BatchUnits best{tail, tail_rows};
  double best_time = -1.0;
  for (int groups : {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16, 20, 24, 32}) {
    int zpb = (tail_rows + groups - 1) / groups;
    if (pair) zpb += zpb & 1;
    double w = head;
    long units = 0;
    int longest = 0;
    for (int k = tail; k < n; ++k) {
      const int ng = (s[k].second + zpb - 1) / zpb;
      w += (double)s[k].first * (s[k].second + m.item * ng);
      units += s[k].first * ng;
      longest = std::max(longest, (s[k].second + ng - 1) / ng);
    }
    double time = std::max(zpb + m.item, w / (double)slots + m.end * (zpb + m.item));
    if (tail == 0) {
      const long left = units % slots;
      const double share = (double)((left + cus - 1) / cus * cus) / (double)slots;
      time = (longest + m.item) * ((double)(units / slots) + (left ? std::max(m.alone, share) : 0.0));
    }
    time *= 1.0 + ragged * std::min(longest, 100) * 0.01;
    if (best_time < 0.0 || time < best_time * 0.999) best_time = time, best.zpb = zpb;
  }
  return best;
}
int main(int argc, char **argv) {
  const int kinds = std::atoi(argv[1]), most = std::atoi(argv[2]);
  unsigned r = 12345;
  auto next = [&](int n) { return (int)((r = r * 1664525u + 1013904223u) >> 8) % n; };
  for (int trial = 0; trial < 400; ++trial) {
    const int n = 1 + next(most);
    std::vector<Series> s;
    for (int k = 0; k < n; ++k) s.push_back({1 + next(1 + next(300)), 1 + 7 * next(kinds)});
    const BatchModel m{2.0 + next(25), 0.3 + 0.1 * next(8), 0.1 + 0.1 * next(8), 0.0, 0.0};
    const long slots = 256l << next(5);
    const bool pair = next(2);
    long reads = 0;
    const double ragged = next(3) ? 0.0 : 0.9;
    const BatchUnits a = pick_batch(m, slots, 256, pair, ragged, n, [&](int k) { return ++reads, s[k]; });
    if (reads > 3l * n) return std::printf("%ld reads of %d series\n", reads, n), 1;
    if (a.tail < 0 || a.tail > n || a.zpb < 1) return std::printf("%d %d\n", a.tail, a.zpb), 1;
    const BatchUnits b = plain(m, slots, 256, pair, ragged, s);
    if (kinds <= 64 && (a.tail != b.tail || a.zpb != b.zpb))
      return std::printf("trial %d: %d %d, not %d %d\n", trial, a.tail, a.zpb, b.tail, b.zpb), 1;
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("batch_units")
    src, exe = d / "main.cpp", d / "main"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return str(exe)


@pytest.mark.parametrize("kinds", [1, 3, 64, 65, 500])
@pytest.mark.parametrize("most", [1, 12, 4096])
def test_sums_by_rows_choose_the_same(program, kinds, most):
    res = subprocess.run([program, str(kinds), str(most)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout

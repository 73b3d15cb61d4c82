"""The counting behind a block's list of candidates (csrc/cand_place.hpp), on
the host: more hits in one block than an int holds, with every wave adding on
what it read before the others added."""

import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_1711_10855_amd", "csrc")

# WAVES waves offer in rounds: in each all of them read the count before one of
# them adds to it. Their offers fill the list, then go on for `rounds` rounds.
PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "cand_place.hpp"
using namespace fdas;
int main(int argc, char **argv) {
  const int waves = 16, first = std::atoi(argv[1]), total = 1024;
  const long long rounds = std::atoll(argv[2]);
  unsigned n = 0;  // (wraps as the 32-bit counter in LDS does)
  int lim = kCandLds;
  long long offered = 0, direct = 0, listed = 0;
  std::vector<int> uses(kCandLds, 0);
  for (long long r = 0; r < rounds; ++r) {
    const int read = (int)n;
    for (int w = 0; w < waves; ++w) {
      const int k = r < 8 ? first + w % 3 : total;
      const int pos = cand_place(k, [&] { return read; },
                                 [&](int add) { const int was = (int)n; n += (unsigned)add; return was; });
      offered += k;
      if (!cand_fits(pos, k)) {
        direct += k;
        if (pos < lim) lim = pos;
        continue;
      }
      for (int i = 0; i < k; ++i) {
        if (pos + i < 0 || pos + i >= kCandLds) return std::printf("entry %d\n", pos + i), 1;
        ++uses[pos + i];
        ++listed;
      }
    }
  }
  const int m = cand_listed((int)n, lim);
  if (m < 0 || m > kCandLds) return std::printf("list of %d\n", m), 1;
  for (int i = 0; i < kCandLds; ++i)
    if (uses[i] != (i < m)) return std::printf("entry %d of %d used %d times\n", i, m, uses[i]), 1;
  if (listed != m || direct + m != offered) return std::printf("%d + %lld != %lld\n", m, direct, offered), 1;
  if (n > kCandLds + waves * total) return std::printf("count %u\n", n), 1;
  std::printf("ok %lld\n", offered);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("cand_place")
    src, exe = d / "main.cpp", d / "main"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return str(exe)


@pytest.mark.parametrize("first", [1, 2, 7, 20, 64, 320, 321, 1024])
@pytest.mark.parametrize("rounds", [1, 8, 40, 140000, 270000])
def test_list_of_a_block_with_many_hits(program, first, rounds):
    """140000 rounds offer 2.3e9 candidates, past the largest int; 270000 pass
    2^32, where a 32-bit count is back at a small number."""
    res = subprocess.run([program, str(first), str(rounds)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
    assert int(res.stdout.split()[1]) > (2 ** 31 if rounds >= 140000 else 0)

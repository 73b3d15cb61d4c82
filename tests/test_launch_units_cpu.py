"""The choice of a launch's work units (csrc/launch_units.hpp), on the host: it is
the cheapest of all layouts by its own estimate, what it looks at stays few for
any number of rows, and its units cover every row of every segment once."""

import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_1711_10855_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "launch_units.hpp"
using namespace fdas;
int main(int argc, char **argv) {
  const UnitModel m{std::atof(argv[1]), std::atof(argv[2]), std::atof(argv[3]), std::atof(argv[4]), 1.1,
                    {0.9, 0.4}};
  const int cus = std::atoi(argv[5]), nz = std::atoi(argv[8]);
  const long pair_slots = std::atol(argv[6]), single_slots = std::atol(argv[7]);
  const bool all = std::atoi(argv[9]), ragged = std::atoi(argv[10]);
  long worst = 0;
  for (long nsb = 1; nsb < 100000; nsb += 1 + nsb / 7) {
    int64_t looked = 0;
    const UnitSplit s = pick_units(m, nsb, nz, cus, pair_slots, single_slots, ragged, &looked);
    if (looked > worst) worst = looked;
    const long slots = s.pair ? pair_slots : single_slots;
    if (s.n1 < 0 || s.n1 > nsb || s.n1 % slots || s.zpb1 != nz || s.zpb2 < 1 || s.zpb2 > nz ||
        (s.pair && pair_slots <= 0))
      return std::printf("nsb %ld: %ld %d %d %d\n", nsb, (long)s.n1, s.zpb1, s.zpb2, s.pair), 1;
    if (!all) continue;
    double best = -1.0;
    for (int pair = pair_slots > 0; pair >= 0; --pair) {
      const long sl = pair ? pair_slots : single_slots;
      const UnitCost cost{m, nsb, sl, cus, nz, pair ? 2 : 1, ragged ? m.ragged[pair ? 0 : 1] : 0.0};
      const int n = pair ? (nz + 1) / 2 : nz;
      const long full = pair || pair_slots <= 0 ? nsb / sl : 0;
      for (long k : {0l, full - 1, full})
        for (int per = 1; k >= 0 && per <= n; ++per) {
          const double c = cost(k, per) * (pair_slots > 0 && !pair ? m.single : 1.0);
          if (best < 0.0 || c < best) best = c;
        }
    }
    const UnitCost cost{m, nsb, slots, cus, nz, s.pair ? 2 : 1, ragged ? m.ragged[s.pair ? 0 : 1] : 0.0};
    const double c = cost(s.n1 / slots, s.pair ? (s.zpb2 + 1) / 2 : s.zpb2) *
                     (pair_slots > 0 && !s.pair ? m.single : 1.0);
    if (c > best * 1.0021) return std::printf("nsb %ld: %g, least %g\n", nsb, c, best), 1;
  }
  std::printf("%ld\n", worst);
}
"""

MODELS = [(10.6, 0.68, 0.55, 0.36), (5.2, 0.65, 0.47, 0.84), (8.1, 0.36, 0.20, 0.94), (3.0, 0.9, 0.0, 1.0),
          (4.0, 0.5, 0.5, 0.0)]


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("launch_units")
    src, exe = d / "main.cpp", d / "main"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return str(exe)


def run(program, model, cus, pair_slots, single_slots, nz, everything, ragged):
    res = subprocess.run([program, *map(str, model), str(cus), str(pair_slots), str(single_slots),
                          str(nz), str(int(everything)), str(ragged)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
    return int(res.stdout)


@pytest.mark.parametrize("model", MODELS)
@pytest.mark.parametrize("cus,pair_slots,single_slots",
                         [(256, 1024, 1024), (256, 3072, 4096), (256, 0, 512), (256, 256, 256),
                          (32, 0, 64), (1, 1, 1), (304, 1824, 2432)])
@pytest.mark.parametrize("nz", [1, 2, 3, 17, 101, 402])
@pytest.mark.parametrize("ragged", [0, 1])
def test_the_pick_is_the_cheapest_layout(program, model, cus, pair_slots, single_slots, nz, ragged):
    # (layouts within 0.1% of one looked at earlier are passed over, twice at most)
    run(program, model, cus, pair_slots, single_slots, nz, True, ragged)


@pytest.mark.parametrize("model", MODELS)
@pytest.mark.parametrize("pair_slots,single_slots", [(1024, 1024), (3072, 4096), (0, 512)])
def test_few_layouts_are_looked_at(program, model, pair_slots, single_slots):
    """Every call makes this choice: some 1e-8 s for each layout it looks at. One
    by one, 20001 rows are up to 40000 of them; their pairs come in 2 sqrt(10001)
    sizes, with three numbers of whole-row rounds, and the rows in 2 sqrt(20001)."""
    for ragged in (0, 1):
        assert run(program, model, 256, pair_slots, single_slots, 201, False, ragged) <= 120
        assert run(program, model, 256, pair_slots, single_slots, 20001, False, ragged) <= 900

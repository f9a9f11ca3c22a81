"""Work-unit lengths of the sigma contraction (csrc/schedule.h), from the header
itself compiled for the host."""
import os
import subprocess
from math import comb

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1910_03527_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include "schedule.h"
using namespace mbefci;
int main(int argc, char** argv) {
  const int tuned = std::atoi(argv[2]);
  if (argv[1][0] == 'd') {
    std::printf("%d", default_tile(tuned));
  } else if (argv[1][0] == 'k') {  // tuner: kept steps of a best length under a limit
    const int limit = std::atoi(argv[3]), kept = schedule_kept(tuned, limit);
    std::printf("%d", kept);
  } else if (argv[1][0] == 'c') {
    std::printf("%d", (int)schedule_covers(tuned, std::atoi(argv[3])));
  } else if (argv[1][0] == 'u') {  // units of a plan of `limit` under a kept number
    std::printf("%d", string_unit_steps(schedule_steps(tuned), 1024ll * std::atoll(argv[3])));
  } else if (argv[1][0] == 's') {  // steps of up to 10 orbitals
    std::printf("%d", string_unit_steps(tuned, std::atoll(argv[3])));
  } else {                  // tiles above: CASCIs, Na, beta blocks
    const long long n = std::atoll(argv[3]), na = std::atoll(argv[4]), nblk = std::atoll(argv[5]);
    std::printf("%d", pair_unit_tiles(tuned, [&](int l) { return n * nblk * ((na + l - 1) / l); }));
  }
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("schedule")
    (d / "t.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(d / "t.cpp"), "-o", str(d / "t")], check=True)
    return lambda *a: int(subprocess.run([str(d / "t"), *map(str, a)], check=True,
                                         capture_output=True, text=True).stdout)


# one CASCI in tiles of 32 beta strings, and the faster of 8 and 16 tiles per
# unit as measured (where they differ by more than 5%)
@pytest.mark.parametrize("n,na,nb,best", [(11, 6, 4, 8), (11, 6, 2, 8), (12, 5, 4, 8), (13, 6, 1, 8),
                                          (13, 5, 2, 16), (13, 3, 3, 16), (14, 4, 1, 8), (14, 3, 3, 8)])
def test_tiles_per_unit_of_one_casci(rule, n, na, nb, best):
    blocks = (comb(n, nb) + 31) // 32
    assert rule("p", 0, 1, comb(n, na), blocks) == best
    for tuned in (1, 3, 16, 32):  # a tuned number is taken as it is
        assert rule("p", tuned, 1, comb(n, na), blocks) == tuned


@pytest.mark.parametrize("tuned", [0, 1, 3, 16, 32])
def test_steps_per_unit_leave_four_units_per_cu(rule, tuned):
    most = tuned or 16
    for steps in (1, 252, 1023, 1024, 2048, 4095, 16384, 10 ** 7):
        got = rule("s", tuned, steps)
        assert 1 <= got <= most
        assert got == 1 or steps // got >= 1024
        assert got == most or steps // (got + 1) < 1024


@pytest.mark.parametrize("limit", [1, 3, 4, 6, 16, 20, 31, 32, 100])
def test_a_kept_schedule_gives_its_own_plan_the_timed_unit(rule, limit):
    """Whatever length was best, the plan it was timed on (and any other of
    that limit) takes it again without being timed, and a plan of a higher limit
    is timed unless the length was below the limit."""
    for best in (4, 8, 16, 32):
        if best > 4 and best // 2 >= limit:
            continue  # not a candidate of its own
        kept = rule("k", best, limit)
        assert rule("c", kept, limit) == 1
        assert rule("u", kept, limit) == min(best, limit)
        assert (kept < 0) == (best >= limit and limit < 32)
        if kept < 0:
            assert rule("c", kept, max(limit, 4) + 1) == 0


@pytest.mark.parametrize("n", range(2, 15))
def test_default_tile(rule, n):
    """Four waves on an alpha string up to 10 orbitals, 32 columns above."""
    assert rule("d", n) == (64 if n <= 10 else 32)

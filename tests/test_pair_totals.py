"""The pair counts' arithmetic (csrc/pairs.h) on the host: totals that do not
fit 32 bits stay at the largest value, and a tile's range stays inside the pair
buffer for any counts."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "pairs.h"
using namespace sixdgs;
int main(int argc, char** argv) {
  unsigned long long a[3] = {0, 0, 0};
  while (std::scanf("%llu %llu %llu", a, a + 1, a + 2) == 3) {
    const PairRange r = pair_range((uint32_t)a[0], (uint32_t)a[1], (uint32_t)a[2]);
    std::printf("%u %u %u %u\n", add_sat((uint32_t)a[0], (uint32_t)a[1]), pair_total(a[0] * a[1]), r.first, r.end);
  }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("pairs")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "main")
    subprocess.check_call(["g++", "-std=c++17", "-D__host__=", "-D__device__=", "-I",
                           os.path.join(ROOT, "paper_2410_04974_amd", "csrc"), "-o", exe, str(d / "main.cpp")])
    return exe


def test_totals_and_ranges(program):
    m = 2**32 - 1
    edge = [0, 1, 2, 8192, 2**30 - 1, 2**30, 2**31, m - 1, m]
    cases = [(a, b, c) for a in edge for b in edge for c in (0, 1, 8192, 2**30 - 1)]
    out = subprocess.run([program], input="\n".join("%d %d %d" % t for t in cases), capture_output=True, text=True,
                         check=True).stdout.split("\n")
    assert len(out) == len(cases) + 1
    for (a, b, cap), line in zip(cases, out):
        add, total, first, end = map(int, line.split())
        assert add == min(a + b, m) and total == min(a * b, m)
        assert 0 <= first <= end <= cap
        if a + b <= cap:
            assert (first, end) == ((a, a + b) if b else (0, 0))

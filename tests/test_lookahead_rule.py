"""The rule by which the lookahead schedule splits a step's update (dag.h), on
the CPU: a step runs as one launch of a workgroup per unit only if HIP takes
such a grid (at most 2^32 - 1 threads in a dimension, 256 a workgroup)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_11937_amd", "csrc")
SRC = """
#include <cstdio>
#include <cstdlib>
#include "dag.h"
int main(int, char** v) {
  const TcGeom g = tc_geom(atoll(v[1]), atoll(v[2]), 0);
  long long whole = 0, largest = 0;
  for (int32_t J = 0; J < g.M; ++J) {
    const int64_t nu = tc_trailing_units(g, J);
    if (nu > 0 && tc_update_whole(g, nu, atoll(v[3]))) {
      ++whole;
      if (nu > largest) largest = nu;
    }
  }
  printf("%d %lld %lld %lld", g.M, (long long)tc_trailing_units(g, 0), whole, largest);
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    (d / "r.cpp").write_text(SRC)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "r.cpp"), "-o", str(d / "r")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return lambda n, T: [int(x) for x in subprocess.run([str(d / "r"), str(n), str(T), "512"], capture_output=True,
                                                        text=True, check=True).stdout.split()]


@pytest.mark.parametrize("n,T", [(5793, 1), (5794, 1), (5900, 1), (20000, 2), (92672, 16), (92800, 16), (190000, 32),
                                 (1 << 20, 128)])
def test_one_launch_fits_a_grid(rule, n, T):
    M, first, whole, largest = rule(n, T)
    assert largest * 256 <= 0xFFFFFFFF
    # everything that fits is one launch with tiles of one sub-column
    assert (whole == M - 1) == (first * 256 <= 0xFFFFFFFF)


@pytest.mark.parametrize("n,T", [(300, 128), (4096, 256), (8192, 512), (32768, 1024), (32768, 128)])
def test_ordinary_sizes(rule, n, T):
    """Steps of more than 512 units are split exactly when a tile has more
    than one sub-column."""
    M, first, whole, largest = rule(n, T)
    assert largest == first if T <= 128 else largest <= 512
    assert whole == M - 1 if first <= 512 or T <= 128 else whole < M - 1

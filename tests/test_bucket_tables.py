"""The fixed tables of the bucketed quadrature (paper_2410_18234_amd/csrc/bucket_tables.h), compiled for the host and compared
with the functions they stand for.

The cubic of term s on part j interpolates exp(-z (c_j + d t)), z = 2^(s/2), d = 1/64, at four Chebyshev points of t in
[-1, 1]: its error is at most (z d)^4 / (4! 2^3) times the largest exp on the part (the interpolation remainder), plus
fp64 rounding: the values come from a series squared six times, 64 times its 2.2e-16 and 63 half ulps more, 2.1e-14 of at
most 1, and four points at most 1.85 times that (their Lebesgue constant): 4e-14.
"""
import math
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2410_18234_amd", "csrc")
SOURCE = r"""
#include <stdio.h>
#include "bucket_tables.h"
using namespace mdss;
int main() {
  printf("%d %d %d %d\n", kBqNearLo, kBqNear, kBqFar, kBqOct);
  const BqFragments f = bq_make_fragments();
  for (int s = 0; s < kBqCols; ++s)
    for (int x = 0; x < kBqOct; ++x) {
      const double g = kBqTab.g[s][x];
      printf("%.17g %d\n", g, f.g[s / 16][x / 4][x % 4 * 16 + s % 16] == g);
    }
  for (int c = kBqCols; c < 32; ++c)
    for (int x = 0; x < kBqOct; ++x)
      if (f.g[c / 16][x / 4][x % 4 * 16 + c % 16] != kBqTab.g[kBqCols - 1][x]) return 1;
  return 0;
}
"""


@pytest.fixture(scope="module")
def tables(tmp_path_factory):
    gxx = shutil.which("g++")
    assert gxx, "needs g++"
    at = tmp_path_factory.mktemp("tables")
    (at / "dump.cpp").write_text(SOURCE)
    subprocess.run([gxx, "-std=c++17", "-O1", "-fconstexpr-ops-limit=1000000000", "-fconstexpr-loop-limit=10000000", "-I", CSRC, "-o", str(at / "dump"),
                    str(at / "dump.cpp")], check=True, timeout=100)
    out = subprocess.run([str(at / "dump")], check=True, capture_output=True, text=True, timeout=60).stdout.split("\n")
    lo, near, far, octave = (int(v) for v in out[0].split())
    pairs = np.array([[float(v) for v in line.split()] for line in out[1:] if line])
    assert bool((pairs[:, 1] == 1).all()), "the fragments hold the table's values"
    return lo, near, far, pairs[:, 0].reshape(near + far, octave // 4, 4)


def test_near_terms(tables):
    lo, near, _, g = tables
    t = np.linspace(-1.0, 1.0, 401)
    for s in range(near):
        z = 2.0 ** ((lo + s) / 2.0)
        for j in range(32):
            c = 1.0 + (j + 0.5) / 32
            got = np.polynomial.polynomial.polyval(t, g[s, j])
            bound = (z / 64.0) ** 4 / 192.0 * math.exp(-z * (c - 1.0 / 64.0)) + 4e-14
            assert np.abs(got - np.exp(-z * (c + t / 64.0))).max() <= bound, (s, j)


def test_every_term_is_within_the_stated_error(tables):
    # a token paired with much smaller weights, the worst case (at the edges of the octave's first part): r is the sum of
    # a_k exp(-a_k w) over the nodes
    lo, near, _, g = tables
    for j in range(32):
        c = 1.0 + (j + 0.5) / 32
        t = np.linspace(-1.0, 1.0, 201)
        w = c + t / 64.0
        z = 2.0 ** ((lo + np.arange(near)) / 2.0)
        want = (z[:, None] * np.exp(-z[:, None] * w)).sum(0)
        got = sum(z[s] * np.polynomial.polynomial.polyval(t, g[s, j]) for s in range(near))
        assert np.abs(got / want - 1.0).max() <= 7.2e-9


def test_power_columns(tables):
    _, near, far, g = tables
    for i in range(far):
        for j in range(32):
            c, d = 1.0 + (j + 0.5) / 32, 1.0 / 64.0
            for n in range(4):
                want = math.comb(i, n) * c ** (i - n) * d ** n if n <= i else 0.0
                assert abs(g[near + i, j, n] - want) <= 1e-14 * max(want, 1e-300)

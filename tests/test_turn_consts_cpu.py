"""Compile-time cosines and sines (csrc/turn_consts.hpp) are the nearest FP64 numbers."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_25161_amd", "csrc")

HARNESS = r"""
#include <cmath>
#include <cstdio>
#include "turn_consts.hpp"
int main() {
  const long double tp = 6.283185307179586476925286766559L;
  for (int n : {3, 5, 6, 8, 9, 10, 12, 15, 16})
    for (int m = 0; m < n; ++m)
      for (int sine = 0; sine < 2; ++sine) {
        const long double x = tp * m / n, ref = sine ? sinl(x) : cosl(x);
        const double v = sine ? fsd::sin_turn(m, n) : fsd::cos_turn(m, n);
        // units in the last place; exact zeros have none
        const double ulp = std::nextafter(std::fabs(v), 2.0) - std::fabs(v);
        std::printf("%d %d %d %.6f\n", n, m, sine, fabsl(ref) < 1e-15L ? std::fabs(v) : double(fabsl(v - ref)) / ulp);
      }
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_nearest(tmp_path):
    src, exe = tmp_path / "h.cpp", tmp_path / "h"
    src.write_text("#include <initializer_list>\n" + HARNESS)
    subprocess.run(["g++", "-O0", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")
    rows = [l.split() for l in out if l]
    assert len(rows) == 168
    for n, m, sine, err in rows:
        assert float(err) <= 0.5001, (n, m, sine, err)  # the reference's own 80 bits


CONSTEXPR = r"""
#include "turn_consts.hpp"
static_assert(fsd::cos_turn(1, 8) == 0.70710678118654752440 && fsd::sin_turn(1, 3) == 0.86602540378443864676 &&
              fsd::cos_turn(1, 5) == 0.30901699437494742410 && fsd::cos_turn(1, 4) == 0.0 && fsd::cos_turn(1, 2) == -1.0);
int main() {}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_at_compile_time(tmp_path):
    src = tmp_path / "c.cpp"
    src.write_text(CONSTEXPR)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-fsyntax-only", str(src)], check=True)

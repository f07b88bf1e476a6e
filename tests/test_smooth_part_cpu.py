"""The piecewise polynomials of the smooth part (csrc/smooth_part.hpp), FP64 and rounded to FP32, against
the quadrature that they interpolate, on the host; interval edges and the first interval included."""
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_25161_amd", "csrc")

HARNESS = r"""
#include <algorithm>
#include <cstdio>
#include "smooth_part.hpp"
using namespace fsd;
template <typename R>
void largest(const SmoothPart& sp, double rcut, int fine, const double* scale, double* out) {
  using P = RealPoly<R>;
  const std::vector<double> c = smooth_poly<R>(sp, rcut, fine);
  std::vector<R> T(c.begin(), c.end());
  const int n = fine * P::kIntervals;
  out[0] = out[1] = 0;
  for (int q = 0; q < n; ++q)
    for (double x : {1e-9, 0.02, 0.13, 0.31, 0.5, 0.77, 0.94, 1 - 1e-9}) {
      const double r0 = (q + x) * rcut / n;
      const R r = R(r0), u = r * (R(1.0 / rcut) * R(n));
      const int i = std::min(int(u), n - 1);
      const R y = u - R(i) - R(0.5);
      double v[5];
      sp.eval(double(r), v);
      const double r2 = double(r) * double(r), p[5] = {1.0, r2, 1.0, r2, double(r)};
      for (int k = 0; k < 5; ++k) {
        R s = T[size_t(i) * P::kStride + k * P::kCoef];
        double d = c[size_t(i) * P::kStride + k * P::kCoef];
        const double z = double(r) / rcut * n - i - 0.5;
        for (int m = 1; m < P::kCoef; ++m) {
          s = s * y + T[size_t(i) * P::kStride + k * P::kCoef + m];
          d = d * z + c[size_t(i) * P::kStride + k * P::kCoef + m];
        }
        out[0] = std::max(out[0], std::fabs(d * p[k] - v[k]) / scale[k]);          // the fit
        out[1] = std::max(out[1], std::fabs(double(s) * p[k] - v[k]) / scale[k]);  // rounded and evaluated in R
      }
    }
}
int main() {
  double xi, rcut;
  while (std::scanf("%lf %lf", &xi, &rcut) == 2) {
    const SmoothPart sp(1.0, 1.0, xi, rcut);
    const int fine = poly_fine(xi, rcut);
    const double mt = 1 / (6 * M_PI), mr = 1 / (8 * M_PI), scale[5] = {mt, mt, mr, mr, mt};
    double d[2], f[2];
    largest<double>(sp, rcut, fine, scale, d);
    largest<float>(sp, rcut, fine, scale, f);
    std::printf("%g %g %g\n", d[1], f[0], f[1]);
  }
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_largest_errors(tmp_path):
    src, exe = tmp_path / "h.cpp", tmp_path / "h"
    src.write_text(HARNESS)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    # xi a and xi r_cut: the cutoffs of tolerances from 1e-3 to 1e-12, and either side of the finer intervals
    cases = [(0.1, 2.63), (0.348, 3.41), (0.348, 5.5), (0.5, 3.69), (0.5, 5.78), (1.2, 5.35), (1.2, 6.99), (1.2, 7.01),
             (2.0, 8.66), (3.0, 10.57), (5.0, 14.47)]
    text = "".join(f"{xi} {x / xi}\n" for xi, x in cases)
    out = subprocess.run([str(exe)], input=text, check=True, capture_output=True, text=True).stdout.split("\n")
    for (xi, x), line in zip(cases, out):
        fp64, fit, fp32 = map(float, line.split())
        # the stated bounds; FP32: a few roundings of values up to about one self mobility
        assert fp64 < (1.6e-13 if x <= 7 else 5e-14), (xi, x, fp64)
        assert fit < 1e-8, (xi, x, fit)
        assert fp32 < 4 * np.finfo(np.float32).eps, (xi, x, fp32)

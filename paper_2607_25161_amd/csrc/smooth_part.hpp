// The smooth part of the real-space functions on the host: its quadrature and the coefficients of its
// piecewise polynomials.
#pragma once
#include <cmath>
#include <vector>

#include "real_poly.hpp"

namespace fsd {

// ---- spherical Bessel functions, stable near 0 ------------------------------------------
// j0(x), j1(x)/x, j1(x), j2(x): power series for x < 1, trigonometric forms above.
inline void sph_bessel(double x, double& j0, double& j1x, double& j1, double& j2) {
  if (x < 1.0) {
    const double y = -0.5 * x * x;
    // j_n(x) = x^n sum_k y^k / (k! (2n+2k+1)!!)
    double t0 = 1.0, t1 = 1.0 / 3.0, t2 = 1.0 / 15.0;
    double s0 = t0, s1 = t1, s2 = t2;
    for (int k = 1; k < 12; ++k) {
      t0 *= y / (k * (2.0 * k + 1.0));
      t1 *= y / (k * (2.0 * k + 3.0));
      t2 *= y / (k * (2.0 * k + 5.0));
      s0 += t0;
      s1 += t1;
      s2 += t2;
    }
    j0 = s0;
    j1x = s1;
    j1 = x * s1;
    j2 = x * x * s2;
  } else {
    const double s = std::sin(x), c = std::cos(x);
    j0 = s / x;
    j1 = s / (x * x) - c / x;
    j1x = j1 / x;
    j2 = (3.0 / (x * x) - 1.0) * s / x - 3.0 * c / (x * x);
  }
}

inline void sinc_jv_host(double x, double& s, double& j) {
  double j0, j1x, j1, j2;
  sph_bessel(x, j0, j1x, j1, j2);
  s = j0;
  j = 3.0 * j1x;  // jv(x) = 3 j1(x) / x
}

// ---- real-space smooth part ----------------------------------------------------------------
// S(r): inverse transform of the Hasimoto-damped FT-RPY multipliers
//   tt: sinc^2(ka) H(k) (I - kk)/k^2,  rr: jv^2(ka) H(k) (I - kk)/4,  rt: (i/2) sinc jv H [k]x / k^2,
//   H(k) = (1 + k^2/(4 xi^2)) exp(-k^2/(4 xi^2)).
// Angular integration leaves radial integrals of j0 - j1/x (I part), j2 (rr part) and
// k j1 (rt part).  The integrands are even, entire in k and Gaussian-decaying, so the
// trapezoid rule on a step below 2 pi / (band of the integrand) is spectrally accurate.
struct SmoothPart {
  std::vector<double> k, wtt, wrr, wrt;  // nodes and multiplier-times-weight
  double eta;
  SmoothPart(double a, double eta_, double xi, double rmax) : eta(eta_) {
    const double kmax = 2.0 * xi * std::sqrt(46.0);
    const double band = rmax + 2.0 * a + 7.0 / xi;
    const double hk = 2.0 * M_PI / band / 2.0;
    const int nk = int(std::ceil(kmax / hk)) + 1;
    for (int m = 0; m < nk; ++m) {
      const double kk = m * hk;
      const double q = kk * kk / (4.0 * xi * xi);
      const double H = (1.0 + q) * std::exp(-q);
      double s, j;
      sinc_jv_host(kk * a, s, j);
      const double w = (m == 0 ? 0.5 : 1.0) * hk;
      k.push_back(kk);
      wtt.push_back(w * s * s * H);
      wrr.push_back(w * 0.25 * kk * kk * j * j * H);
      wrt.push_back(w * kk * s * j * H);
    }
  }
  // out: (tI, tR, rI, rR, c) of S at distance r (r may be negative or zero)
  void eval(double r, double* out) const {
    double tI = 0, tR = 0, rI = 0, rR = 0, c = 0;
    const double ar = std::fabs(r);
    for (size_t m = 0; m < k.size(); ++m) {
      double j0, j1x, j1, j2;
      sph_bessel(k[m] * ar, j0, j1x, j1, j2);
      const double fI = j0 - j1x;
      tI += wtt[m] * fI;
      tR += wtt[m] * j2;
      rI += wrr[m] * fI;
      rR += wrr[m] * j2;
      c += wrt[m] * j1;
    }
    const double p = 1.0 / (2.0 * M_PI * M_PI * eta);
    out[0] = p * tI;
    out[1] = p * tR;
    out[2] = p * rI;
    out[3] = p * rR;
    out[4] = -(r < 0 ? -1.0 : 1.0) * c / (4.0 * M_PI * M_PI * eta);
  }
};

// Coefficients of the smooth part on [0, rcut] in the layout of RealPoly<R>: per interval the
// interpolation at the Chebyshev nodes, solved for the powers of the centred offset (at most
// degree 6 on an offset of at most 1/2, well conditioned).
template <typename R>
std::vector<double> smooth_poly(const SmoothPart& sp, double rcut, int fine) {
  using P = RealPoly<R>;
  constexpr int n = P::kCoef;
  const int intervals = fine * P::kIntervals;
  double x[n];
  for (int m = 0; m < n; ++m) x[m] = 0.5 * std::cos(M_PI * (m + 0.5) / n);
  std::vector<double> out(size_t(intervals) * P::kStride, 0.0);
  for (int q = 0; q < intervals; ++q) {
    double v[n][5];
    for (int m = 0; m < n; ++m) {
      const double r = (q + 0.5 + x[m]) * rcut / intervals;
      sp.eval(r, v[m]);
      v[m][1] /= r * r;
      v[m][3] /= r * r;
      v[m][4] /= r;
    }
    for (int k = 0; k < 5; ++k) {
      // Newton's divided differences, then the product form expanded to powers of the offset
      double d[n], c[n] = {0};
      for (int m = 0; m < n; ++m) d[m] = v[m][k];
      for (int o = 1; o < n; ++o)
        for (int m = n - 1; m >= o; --m) d[m] = (d[m] - d[m - 1]) / (x[m] - x[m - o]);
      for (int m = n - 1; m >= 0; --m) {  // c <- c (x - x_m) + d_m, c[i] the power i
        for (int i = n - 1; i > 0; --i) c[i] = c[i - 1] - x[m] * c[i];
        c[0] = d[m] - x[m] * c[0];
      }
      for (int i = 0; i < n; ++i) out[size_t(q) * P::kStride + k * n + i] = c[n - 1 - i];
    }
  }
  return out;
}

}  // namespace fsd

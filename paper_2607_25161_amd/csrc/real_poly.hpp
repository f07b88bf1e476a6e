// Layout of the smooth part of the real-space functions, for the kernels and the host.
#pragma once
#include <cmath>
#include <cstddef>

namespace fsd {

// The smooth part as piecewise polynomials on fine kIntervals equal intervals of [0, 1 / poly_inverse_range]: five
// functions of kCoef coefficients each (highest power first, in the offset from the interval's centre
// over its width), rows kStride values apart (an odd multiple of 16 bytes).  The functions, all even
// in r and in units of 1 / (8 pi eta): tt I, tt rr / r^2, rr I, rr rr / r^2, rt / r.
template <typename R>
struct RealPoly;
template <>
struct RealPoly<double> {
  static constexpr int kIntervals = 64, kCoef = 7, kStride = 38;
  static constexpr size_t bytes(int fine) { return sizeof(double) * fine * kIntervals * kStride; }
};
template <>
struct RealPoly<float> {
  static constexpr int kIntervals = 128, kCoef = 4, kStride = 20;
  static constexpr size_t bytes(int fine) { return sizeof(float) * fine * kIntervals * kStride; }
};

// Twice the intervals where the cutoff reaches far on the smooth part's own scale 1 / xi (large xi with a
// tight tolerance; xi r_cut is 2.6 to 5.8 for xi up to 0.5 / a and tolerances of 1e-3 to 1e-12).  Largest errors
// in self mobilities, against a table of 4,096 nodes with cubic interpolation: in FP64 up to 1.4e-13 (the table
// 5e-13) where xi r_cut is at most 7, then with twice the intervals up to 4.3e-14 (1.5e-12) at 14.5 and 9e-13 (5e-12)
// at 25; with the base intervals they would be 2e-12 at 14.5.  In FP32 the fit alone is off by at most 7e-9 and
// its rounded form by 1.3e-7 (1.9e-7): the values reach about one self mobility.
inline int poly_fine(double xi, double rcut) { return xi * rcut > 7.0 ? 2 : 1; }

// The inverse of the range that the polynomials cover: the largest FP32 number up to 1 / rcut, so that a
// distance in intervals has no systematic error in FP32 (a rounded factor moves every pair the same way)
inline double poly_inverse_range(double rcut) {
  const float f = float(1.0 / rcut);
  return double(f) * rcut > 1.0 ? double(std::nextafter(f, 0.0f)) : double(f);
}

}  // namespace fsd

// Cosines and sines of fractions of a turn at compile time.
#pragma once

namespace fsd {

// cos(2 pi m / n) for 0 <= m / n, folded to the first eighth of the circle and summed as a series in pairs
// of doubles, so that the constants are the nearest ones (long double is FP64 in device code; in plain FP64
// two in five came out one unit off in the last place)
struct Pair {
  double hi, lo;
};
constexpr Pair two_sum(double a, double b) {
  const double s = a + b, t = s - a;
  return {s, (a - (s - t)) + (b - t)};
}
constexpr Pair two_prod(double a, double b) {  // by halves of 26 bits (Dekker)
  const double ca = 134217729.0 * a, cb = 134217729.0 * b;
  const double ah = ca - (ca - a), al = a - ah, bh = cb - (cb - b), bl = b - bh, p = a * b;
  return {p, ((ah * bh - p) + ah * bl + al * bh) + al * bl};
}
constexpr Pair add(Pair a, Pair b) {
  const Pair s = two_sum(a.hi, b.hi);
  return two_sum(s.hi, s.lo + (a.lo + b.lo));
}
constexpr Pair mul(Pair a, Pair b) {
  const Pair p = two_prod(a.hi, b.hi);
  return two_sum(p.hi, p.lo + (a.hi * b.lo + a.lo * b.hi));
}
constexpr Pair over(Pair a, double b) {
  const double q = a.hi / b;
  const Pair p = two_prod(q, b);
  return two_sum(q, ((a.hi - p.hi) - p.lo + a.lo) / b);
}
// first, first x^2 / (odd (odd + 1)), ...: cos (1, 1) and sin (x, 2)
constexpr double series(Pair x, Pair first, int from) {
  const Pair x2 = mul(x, x), minus{-x2.hi, -x2.lo};
  Pair t = first, s = first;
  for (int k = from; k < from + 28; k += 2) s = add(s, t = over(mul(t, minus), double(k * (k + 1))));
  return s.hi;
}
constexpr Pair kTwoPi = {6.283185307179586477, 2.4492935982947063545e-16};
constexpr double cos_turn(long m, long n) {
  m %= n;
  if (2 * m > n) m = n - m;                           // cos(2 pi - t) = cos t
  if (4 * m > n) return -cos_turn(n - 2 * m, 2 * n);  // cos t = -cos(pi - t)
  if (8 * m > n) {                                    // cos t = sin(pi / 2 - t)
    const Pair x = over(mul(kTwoPi, {double(n - 4 * m), 0.0}), 4.0 * n);
    return series(x, x, 2);
  }
  return series(over(mul(kTwoPi, {double(m), 0.0}), double(n)), {1.0, 0.0}, 1);
}
constexpr double sin_turn(long m, long n) { return cos_turn(4 * m + 3 * n, 4 * n); }  // sin t = cos(t - pi / 2)

}  // namespace fsd

// Double precision from the hardware's approximations, shared by the kernels:
// plain functions (T is double) that take the approximation as an argument, so
// that a CPU test can run them on approximations of the hardware's error and
// compare their rounding with that of the correctly rounded operations.
//
// The hardware's reciprocal and inverse square root are good to 2^-24.2 (4
// million arguments between 2^-99 and 2^99).  What follows brings them to the
// error stated at each function, for arguments whose square or reciprocal is
// in range, without the scaling and the special cases of the library's
// operations (5, 8 and 8 instructions against 11, 18 and, as a division by a
// root, 29).
#pragma once

namespace bqk {

// 1 / x from r: half a unit in the last place
template <typename T>
constexpr T rcp_from(T x, T r) {
  r = __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
  return __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
}

// t / d from id, 1 / d to half a unit: the product's remainder corrects it to
// half a unit again
template <typename T>
constexpr T div_from(T t, T d, T id) {
  const double q = t * id;
  return __builtin_fma(__builtin_fma(-d, q, t), id, q);
}

// sqrt(x) from y, about 1 / sqrt(x): a coupled step for the root and half its
// inverse, then the root's remainder; half a unit
template <typename T>
constexpr T sqrt_from(T x, T y) {
  double s = x * y, h = 0.5 * y;
  const double r = __builtin_fma(-h, s, 0.5);
  s = __builtin_fma(s, r, s);
  h = __builtin_fma(h, r, h);
  return __builtin_fma(__builtin_fma(-s, s, x), h, s);
}

// 1 / sqrt(x) from y: the third-order step y (1 + e / 2 + 3 e^2 / 8), e = 1 -
// x y^2, whose e takes the rounding of x y into account (without that the
// result is off by up to 1.7 units); 0.501 of a unit
template <typename T>
constexpr T rsq_from(T x, T y) {
  const double p = x * y, lo = __builtin_fma(x, y, -p);
  const double e = __builtin_fma(-lo, y, __builtin_fma(-p, y, 1.0));
  return __builtin_fma(__builtin_fma(0.375, e, 0.5) * e, y, y);
}

// x^(-1/3) from y, good to 1e-5: two steps of y += y (1 - x y^3) / 3
// (Newton's, quadratic); 1.43 x 2^-53, where a correctly rounded cube root and
// division together reach 1.48
template <typename T>
constexpr T rcbrt_from(T x, T y) {
  y = __builtin_fma(y * (1.0 / 3.0), __builtin_fma(-x * y, y * y, 1.0), y);
  return __builtin_fma(y * (1.0 / 3.0), __builtin_fma(-x * y, y * y, 1.0), y);
}

// z of the desingularised velocity u = q h / sqrt(z), h4 = h^4: the KP07
// factor sqrt(2) h / sqrt(h^4 + max(h^4, eps)) with its constant taken into
// the root, which is h^4 itself (exactly) where h^4 >= eps
template <typename T>
constexpr T desing_sq(T h4, T eps) { return 0.5 * (h4 + (h4 > eps ? h4 : eps)); }

}  // namespace bqk

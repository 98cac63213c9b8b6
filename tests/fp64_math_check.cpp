// Host-side check of the kernels' double-precision roots and reciprocals
// (compiled with the system C++ compiler against the header the kernels
// include), started from approximations with the error of the hardware's and
// up to four times it: their error against 113-bit arithmetic, and that of the
// face velocity formed with them, beside the correctly rounded operations'.
#include <cmath>
#include <cstdio>
#include <random>

#include "bq_fp64.hpp"

using namespace bqk;
typedef __float128 Q;

static int failures = 0;
#define CHECK(c, ...)                  \
  do {                                 \
    if (!(c)) {                        \
      std::printf("FAIL: " __VA_ARGS__); \
      std::printf("\n");               \
      ++failures;                      \
    }                                  \
  } while (0)

static Q qsqrt(Q x) {
  Q s = std::sqrt((double)x);
  for (int k = 0; k < 3; ++k) s = (s + x / s) / 2;
  return s;
}
static Q qrcbrt(Q x) {
  Q y = 1 / std::cbrt((double)x);
  for (int k = 0; k < 3; ++k) y += y * (1 - x * y * y * y) / 3;
  return y;
}

// error of a against the exact r, in units in the last place of r
static double ulps(double a, Q r) {
  const int e = std::ilogb((double)r);
  return (double)((Q)std::scalbn(1.0, 52 - e) * ((Q)a - r));
}
// relative error in units of 2^-53
static double rel(double a, Q r) { return (double)(((Q)a - r) / r) * 0x1p53; }

struct Stat {
  double worst = 0.0, sum = 0.0;
  long n = 0;
  void add(double e) {
    e = std::fabs(e);
    if (!(e <= worst)) worst = e;
    sum += e;
    ++n;
  }
  double mean() const { return sum / (double)n; }
};

int main() {
  std::mt19937_64 gen(20);
  std::uniform_real_distribution<double> unit(-1.0, 1.0);
  const int N = 200000;
  // relative error of the approximations: the hardware's (2^-24.2) and 2^-22
  for (double seed : {0x1p-24, 0x1p-22}) {
    auto off = [&](double v) { return v * (1.0 + seed * unit(gen)); };
    Stat rcp, div, sq, rsq, cb, cb_ref;
    for (int k = 0; k < N; ++k) {
      const double x = std::exp2(60.0 * unit(gen)), t = std::exp2(60.0 * unit(gen));
      const double r = rcp_from(x, off(1.0 / x));
      rcp.add(ulps(r, 1 / (Q)x));
      div.add(ulps(div_from(t, x, r), (Q)t / x));
      sq.add(ulps(sqrt_from(x, off(1.0 / std::sqrt(x))), qsqrt(x)));
      rsq.add(ulps(rsq_from(x, off(1.0 / std::sqrt(x))), 1 / qsqrt(x)));
      // (the cube root's approximation is an FP32 value, off by up to 4e-6)
      const Q c = qrcbrt(x);
      cb.add(rel(rcbrt_from(x, (double)c * (1.0 + 4e-6 * unit(gen))), c));
      cb_ref.add(rel(1.0 / (double)(1 / c), c));
    }
    std::printf("approximations off by %.1g: rcp %.6f div %.6f sqrt %.6f rsq %.6f ulp; rcbrt %.3f (mean %.4f), "
                "rounded cube root and division %.3f (%.4f) x 2^-53\n",
                seed, rcp.worst, div.worst, sq.worst, rsq.worst, cb.worst, cb.mean(), cb_ref.worst, cb_ref.mean());
    // the correctly rounded operations' half unit, to the terms that the last
    // steps leave out (below 2^-86, the inverse root's below 2^-64 = 5e-4 of a unit)
    CHECK(rcp.worst <= 0.5 + 1e-6, "reciprocal off by %.6f ulp", rcp.worst);
    CHECK(div.worst <= 0.5 + 1e-6, "division off by %.6f ulp", div.worst);
    CHECK(sq.worst <= 0.5 + 1e-6, "square root off by %.6f ulp", sq.worst);
    CHECK(rsq.worst <= 0.5 + 1e-3, "inverse square root off by %.6f ulp", rsq.worst);
    CHECK(cb.worst <= 2.0 && cb.mean() <= cb_ref.mean(), "inverse cube root off by %.3f, mean %.4f (%.4f)", cb.worst,
          cb.mean(), cb_ref.mean());
    // face velocity q h / sqrt(z) against the definition in correctly rounded
    // operations, for deep, middling and thin sides
    const char* names[3] = {"deep", "near the threshold", "thin"};
    for (int part = 0; part < 3; ++part) {
      Stat here, ref;
      for (int k = 0; k < N; ++k) {
        const double eps = std::exp2(20.0 * unit(gen) - 12.0), lim = std::pow(eps, 0.25), q = unit(gen);
        const double u = unit(gen);
        const double h = lim * (part == 0 ? std::exp2(4.0 + 4.0 * u) : part == 1 ? std::exp2(0.5 * u)
                                                                               : std::exp2(-7.0 + 6.5 * u));
        const double h2 = h * h, h4 = h2 * h2;
        const Q H = h, H4 = H * H * H * H, Z = (H4 + (H4 > (Q)eps ? H4 : (Q)eps)) / 2, V = (Q)q * H / qsqrt(Z);
        const double z = desing_sq(h4, eps);
        if (h4 >= eps) CHECK(z == h4, "a deep side's z is not its h^4");
        here.add(rel(q * (h * rsq_from(z, off(1.0 / std::sqrt(z)))), V));
        ref.add(rel(1.4142135623730951 * h * q / std::sqrt(h4 + std::fmax(h4, eps)), V));
      }
      std::printf("face velocity, %s: worst %.3f mean %.4f; as defined %.3f %.4f (x 2^-53)\n", names[part], here.worst,
                  here.mean(), ref.worst, ref.mean());
      CHECK(here.worst <= ref.worst && here.mean() <= ref.mean(), "face velocity (%s) less accurate than as defined",
            names[part]);
    }
  }
  // no water and no flow
  CHECK(0.0 * rsq_from(desing_sq(0.0, 1e-8), 1.0 / std::sqrt(5e-9)) == 0.0, "velocity factor of a dry side");
  std::printf("%d failures\n", failures);
  return failures ? 1 : 0;
}

// The square root and the reciprocal of the update's coefficients, refined from
// an estimate (update.hpp), against the correctly rounded ones.  Arguments of
// every size that squared wavenumbers take, estimates off by up to 2^-23.
#include <cmath>
#include <cstdio>
#include <random>

#include "update.hpp"

int main() {
  std::mt19937_64 gen(5);
  std::uniform_real_distribution<double> mantissa(1.0, 4.0), off(-0x1p-23, 0x1p-23), factor(0.5, 2.0);
  std::uniform_int_distribution<int> exponent(-200, 200);
  long long wrong_root = 0, wrong_inverse = 0;
  const int n = 4000000;
  for (int i = 0; i < n; ++i) {
    const double x = std::ldexp(mantissa(gen), 2 * exponent(gen));
    const double y = (1.0 / std::sqrt(x)) * (1.0 + (i % 4 == 0 ? (i % 8 ? 0x1p-23 : -0x1p-23) : off(gen)));
    double root, inverse;
    psatd::psatd_roots(x, y, &root, &inverse);
    if (root != std::sqrt(x)) ++wrong_root;
    if (inverse != 1.0 / root) ++wrong_inverse;
    const double half = factor(gen), h = root * half;
    if (psatd::psatd_refine_inverse(h, inverse * (1.0 / half)) != 1.0 / h) ++wrong_inverse;
  }
  double r0 = -1, i0 = -1;
  psatd::psatd_roots(0.0, INFINITY, &r0, &i0);
  const psatd::Coef at0 = psatd::psatd_coef<double>(0.0, 0.5, 2.0, 4.0, 0.25);
  const bool zero = r0 == 0.0 && i0 == 0.0 && at0.C == 0.25 && at0.S == 0.125;
  std::printf("%lld of %d roots and %lld of %d inverses not correctly rounded, zero %s\n", wrong_root, n,
              wrong_inverse, n, zero ? "ok" : "wrong");
  return wrong_root == 0 && wrong_inverse == 0 && zero ? 0 : 1;
}

// Largest errors of the self-interaction's sines and cosines (qlg_math.hpp, host build) against long double,
// per type and range of angle: prints the type, the range, the errors of the density phase, of the singlet
// phase and of the half rotation (in unit roundoffs; the last less its argument's own rounding), and the
// number of small angles at which the general form is not the short series' value bit for bit.
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>

#include "qlg_math.hpp"

typedef long double R;

template <typename T>
static bool differ(const qlg::Series<T>& p, const qlg::Series<T>& q) {
  return std::memcmp(&p, &q, sizeof p) != 0;
}

template <typename T>
static void measure(const char* type, R unit) {
  std::mt19937_64 gen(7);
  const double edge[] = {0, 0.0625, 0.125, 1.5707963267948966, 3.2, 40, 4096, 1e5};
  for (int range = 0; range + 1 < 8; ++range) {
    R e0 = 0, e2 = 0, eh = 0;
    long unlike = 0;
    std::uniform_real_distribution<double> draw(edge[range], edge[range + 1]);
    for (int i = 0; i < 200000; ++i) {
      const T x0 = T(draw(gen)) * T(i % 2 ? -1 : 1), x2 = i % 5 ? T(draw(gen)) * T(i % 3 ? 1 : -1) : T(0.01);
      const T h = T(draw(gen)), hh = i % 7 ? h * h : T(0);
      const qlg::Series<T> r = qlg::general_series<T>(x0, x2, hh);
      if (qlg::small_angles(x0, x2, hh)) unlike += differ(r, qlg::short_series<T>(x0, x2, hh));
      const R X0 = x0, X2 = x2, H = std::sqrt(R(hh));
      e0 = std::fmax(e0, std::fmax(std::fabs(r.re0 + 2 * std::sin(X0 / 2) * std::sin(X0 / 2)), std::fabs(r.im0 - std::sin(X0))));
      e2 = std::fmax(e2, std::fmax(std::fabs(X2 * X2 * r.c2 + 2 * std::sin(X2 / 2) * std::sin(X2 / 2)),
                                   std::fabs(X2 * r.s2 - std::sin(X2))));
      const R c = std::cos(H), s = std::sin(H), sign = c * r.ch + s * H * r.sh < 0 ? -1 : 1;
      const R eh1 = std::fmax(std::fabs(sign * r.ch - c), std::fabs(sign * H * r.sh - s)) - 2 * unit * H;
      eh = std::fmax(eh, eh1);
    }
    std::printf("%s %d %.3Lf %.3Lf %.3Lf %ld\n", type, range, e0 / unit, e2 / unit, eh / unit, unlike);
  }
}

int main() {
  measure<double>("c128", std::ldexp(R(1), -53));
  measure<float>("c64", std::ldexp(R(1), -24));
}

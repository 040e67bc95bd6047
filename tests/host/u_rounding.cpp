// RMS rounding error of one application of the self-interaction U (qlg_math.hpp, host build), against the same
// U in long double by the exponential's series, for states and angles of a normal run: prints, per type
// and size of angle, the error of the amplitudes over their norm and the RMS relative change of the norm.
#include <cmath>
#include <cstdio>
#include <random>

#include "qlg_math.hpp"

typedef long double R;
struct C {
  R re, im;
};
static C operator+(C a, C b) { return {a.re + b.re, a.im + b.im}; }
static C operator*(C a, C b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
static C operator*(R s, C a) { return {s * a.re, s * a.im}; }
static C conj(C a) { return {a.re, -a.im}; }
static C mi(C a) { return {a.im, -a.re}; }   // -i a

// x <- exp(-i tg0 n) exp(-i tg1 F.f) (x + (exp(-i tg25 n) - 1)/n (v^H x) v) for x = a, b
static void exact_u(C (&a)[5], C (&b)[5], R tg0, R tg1, R tg25) {
  const R f[4] = {2, std::sqrt(R(6)), std::sqrt(R(6)), 2};
  C p[5], v[5], F{0, 0};
  R n = 0, q[5];
  for (int m = 0; m < 5; ++m) {
    p[m] = a[m] + b[m];
    n += q[m] = p[m].re * p[m].re + p[m].im * p[m].im;
  }
  for (int i = 0; i < 4; ++i) F = F + f[i] * (conj(p[i]) * p[i + 1]);
  const R Fz = 2 * (q[0] - q[4]) + q[1] - q[3];
  for (int m = 0; m < 5; ++m) v[m] = (m % 2 ? R(-1) : R(1)) * conj(p[4 - m]);
  const C E{std::cos(tg0 * n), -std::sin(tg0 * n)};
  const R h = tg25 * n / 2;
  const C c = (tg25 * (h == 0 ? R(1) : std::sin(h) / h)) * C{-std::sin(h), -std::cos(h)};
  for (auto* x : {&a, &b}) {
    C s{0, 0};
    for (int m = 0; m < 5; ++m) s = s + conj(v[m]) * (*x)[m];
    C t[5];
    for (int m = 0; m < 5; ++m) t[m] = (*x)[m] = (*x)[m] + (c * s) * v[m];
    for (int k = 1; k < 40; ++k) {   // t <- (-i tg1 F.f / k) t
      C u[5];
      for (int m = 0; m < 5; ++m) {
        u[m] = (Fz * R(2 - m)) * t[m];
        if (m < 4) u[m] = u[m] + (f[m] / 2) * (conj(F) * t[m + 1]);
        if (m > 0) u[m] = u[m] + (f[m - 1] / 2) * (F * t[m - 1]);
      }
      for (int m = 0; m < 5; ++m) (*x)[m] = (*x)[m] + (t[m] = (tg1 / k) * mi(u[m]));
    }
    for (int m = 0; m < 5; ++m) (*x)[m] = E * (*x)[m];
  }
}

template <typename T>
static void measure(double amp) {
  std::mt19937_64 gen(7);
  std::normal_distribution<double> N(0, amp);
  const double theta = 0.1 * 0.1 / 8;
  const qlg::Angles<T> ang{T(theta), T(-0.7 * theta), T(0.4 * theta / 5)};
  R err = 0, ref = 0, norm = 0;
  const int sites = 4000;
  for (int s = 0; s < sites; ++s) {
    qlg::cx<T> x[2][5];
    C y[2][5];
    R n0 = 0, n1 = 0;
    for (int j = 0; j < 2; ++j)
      for (int m = 0; m < 5; ++m) {
        x[j][m] = {T(N(gen)), T(N(gen))};
        y[j][m] = {R(x[j][m].re), R(x[j][m].im)};
        n0 += y[j][m].re * y[j][m].re + y[j][m].im * y[j][m].im;
      }
    qlg::potential(x[0], x[1], ang);
    exact_u(y[0], y[1], ang.tg0, ang.tg1, ang.tg25);
    for (int j = 0; j < 2; ++j)
      for (int m = 0; m < 5; ++m) {
        const C z{R(x[j][m].re) / qlg::UScale<T>::value, R(x[j][m].im) / qlg::UScale<T>::value};
        err += (z.re - y[j][m].re) * (z.re - y[j][m].re) + (z.im - y[j][m].im) * (z.im - y[j][m].im);
        ref += y[j][m].re * y[j][m].re + y[j][m].im * y[j][m].im;
        n1 += z.re * z.re + z.im * z.im;
      }
    norm += (n1 / n0 - 1) * (n1 / n0 - 1);
  }
  std::printf("%s %g %.4Le %.4Le\n", sizeof(T) == 4 ? "c64" : "c128", amp, std::sqrt(err / ref), std::sqrt(norm / sites));
}

int main() {
  for (double amp : {0.05, 0.3, 1.0}) {
    measure<float>(amp);
    measure<double>(amp);
  }
}

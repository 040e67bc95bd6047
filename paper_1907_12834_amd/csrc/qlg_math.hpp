// Per-site arithmetic of the spin-2 QLG step: collide and the self-interaction U.
//
// Everything here is __host__ __device__ so that the same code can be
// exercised on the CPU before it runs on gfx950.
//
// Component order inside a site: index 0..4 <-> m_f = 2, 1, 0, -1, -2.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

#define QLG_HD __host__ __device__ __forceinline__

namespace qlg {

template <typename T>
struct alignas(2 * sizeof(T)) cx {
  T re, im;
};

template <typename T> QLG_HD cx<T> operator+(cx<T> a, cx<T> b) { return {a.re + b.re, a.im + b.im}; }
template <typename T> QLG_HD cx<T> operator-(cx<T> a, cx<T> b) { return {a.re - b.re, a.im - b.im}; }
template <typename T> QLG_HD cx<T> operator*(cx<T> a, cx<T> b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
template <typename T> QLG_HD cx<T> operator*(T s, cx<T> a) { return {s * a.re, s * a.im}; }
template <typename T> QLG_HD cx<T> conj(cx<T> a) { return {a.re, -a.im}; }
// conj(a) * b
template <typename T> QLG_HD cx<T> cmulc(cx<T> a, cx<T> b) {
  return {a.re * b.re + a.im * b.im, a.re * b.im - a.im * b.re};
}
// c ? x : y, component-wise (a select of values, never of addresses)
template <typename T> QLG_HD cx<T> sel(bool c, cx<T> x, cx<T> y) {
  return {c ? x.re : y.re, c ? x.im : y.im};
}
// acc + s * a (s real)
template <typename T> QLG_HD cx<T> rfma(T s, cx<T> a, cx<T> acc) {
  return {acc.re + s * a.re, acc.im + s * a.im};
}

// Whether p holds on every active lane of the wavefront (the host build: p itself).  A
// branch on it is uniform: no execution-mask changes, both sides never run.
QLG_HD bool all_lanes(bool p) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_ballot_w64(!p) == 0;
#else
  return p;
#endif
}

QLG_HD void sincos_t(float x, float* s, float* c) { sincosf(x, s, c); }
QLG_HD void sincos_t(double x, double* s, double* c) { sincos(x, s, c); }
QLG_HD float sqrt_t(float x) { return sqrtf(x); }
QLG_HD double sqrt_t(double x) { return sqrt(x); }

// 1/sqrt(x) for x > 0 and 1/x for x != 0 (normal): the hardware approximations (about one ulp) in
// FP32; in FP64 the hardware estimate refined by two Newton steps, each of which squares its relative
// error (y <- y + y (1 - x y^2) / 2 and y <- y + y (1 - x y)), to within a few ulp of the exact value
// (the host build divides).
QLG_HD float rsqrt_t(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_rsqf(x);
#else
  return 1.0f / sqrtf(x);
#endif
}
QLG_HD double rsqrt_t(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  double y = __builtin_amdgcn_rsq(x);
#pragma unroll
  for (int k = 0; k < 2; ++k) y = fma(0.5 * y, fma(-(x * y), y, 1.0), y);
  return y;
#else
  return 1.0 / sqrt(x);
#endif
}
QLG_HD float rcp_t(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_rcpf(x);
#else
  return 1.0f / x;
#endif
}
QLG_HD double rcp_t(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  double y = __builtin_amdgcn_rcp(x);
#pragma unroll
  for (int k = 0; k < 2; ++k) y = fma(y, fma(-x, y, 1.0), y);
  return y;
#else
  return 1.0 / x;
#endif
}

// Angles of one application of U(theta): theta*g0, theta*g1, theta*g2/5.
template <typename T>
struct Angles {
  T tg0, tg1, tg25;
  // U may be evaluated on the state scaled in modulus by an exact power of two s (the
  // fused kernels defer the factors of each I' and U): then tg0 and tg25 carry 1/s^2 and
  // fs = 1/s^2 brings theta F back to its true scale, so that W, a function of
  // theta n, theta F and (v v^H)/n only, is unchanged.
  T fs = T(1);
};

// ---------------------------------------------------------------------------
// Collide (sqrt SWAP on each (a_m, b_m) pair), times (1 + i):
//   (1 + i) a' = a + i b,   (1 + i) b' = b + i a,
// since a' = ((1 - i) a + (1 + i) b) / 2 and b' likewise: two additions per amplitude, one
// rounding, no multiplication.  An I' (two collides) then leaves the state times 2i, which
// the fused step kernels carry from substep to substep: U commutes with a phase and sees
// the modulus through its angles (Angles, substep_angles), and the four I' of a half-step
// make (2i)^4 = 16, the two of half of it (2i)^2 = -4: exact real factors, divided out once.
// ---------------------------------------------------------------------------
template <typename T>
QLG_HD void collide_r(cx<T> (&a)[5], cx<T> (&b)[5]) {
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    const cx<T> x = a[m], y = b[m];
    a[m] = cx<T>{x.re - y.im, x.im + y.re};
    b[m] = cx<T>{y.re - x.im, y.im + x.re};
  }
}

template <typename T>
QLG_HD void scale_by(cx<T> (&a)[5], cx<T> (&b)[5], T f) {
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    a[m] = f * a[m];
    b[m] = f * b[m];
  }
}

// x <- -i f x: with f = 1/2 the exact inverse of the factor 2i that collide_r leaves per I'.
template <typename T>
QLG_HD void unphase_by(cx<T> (&a)[5], cx<T> (&b)[5], T f) {
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    a[m] = cx<T>{f * a[m].im, -f * a[m].re};
    b[m] = cx<T>{f * b[m].im, -f * b[m].re};
  }
}

// ---------------------------------------------------------------------------
// Frozen-field self-interaction U(theta) applied to x = a and x = b:
//   x <- exp(-i th g0 n) R P x,
//   P = I + (exp(-i th g2 n/5) - 1) v v^H / n,   v_m = (-1)^m conj(psi_{-m}),
//   R = exp(-i th g1 F.f), a spin-2 rotation (Rot2),
// with psi = a + b, n = |psi|^2, F_nu = psi^H f_nu psi.
//
// Every factor is applied as "identity + small correction": the corrections
// use e^{-i x} - 1 = -2 sin^2(x/2) - 2i sin(x/2) cos(x/2) and R - I, and are summed
// apart from the state, which is rounded when they are added to it (w_apply): once
// per application in FP32, twice in FP64.
// ---------------------------------------------------------------------------
struct Consts {
  static constexpr double r6 = 2.449489742783178098197284;    // sqrt(6)
};

// What the state carries after one application of `potential`: the rotation's correction comes
// in the sums and differences of the m, -m pairs, and in FP64 the factor 1/2 of the way back is
// left to the deferred scale of the step (exact): 2 y is added to twice the correction.  FP32 adds
// its corrections to x once instead (see w_apply) and keeps the scale.
template <typename T>
struct UScale {
  static constexpr int value = sizeof(T) == 8 ? 2 : 1;
};

QLG_HD float fma_t(float a, float b, float c) { return fmaf(a, b, c); }
QLG_HD double fma_t(double a, double b, double c) { return fma(a, b, c); }

// (cos x - 1) / x^2 and sin(x) / x as polynomials in y = x^2, for |x| <= 1/8: the first omitted
// terms are x^10/12! and x^10/11! in FP64 (2e-18 and 2e-17 at x = 1/8) and x^6/8! and x^6/7! in
// FP32 (1e-10 and 8e-10).  kLong: with the terms that |x| <= pi/2 needs (the first omitted: x^22/24! and
// x^22/23!, 3e-20 and 8e-19, in FP64; x^14/16! and x^14/15!, 3e-11 and 4e-10, in FP32), which are set to
// zero where `small`: the same operations on the rest, so the short series' value bit for bit.
template <bool kLong>
QLG_HD void phase_series(float y, bool small, float* c, float* s) {
  float pc = -1.0f / 720, ps = 1.0f / 120;
  if constexpr (kLong) {
    float hc = float(-1.0 / 87178291200.0);   // -1/14!
    float hs = float(1.0 / 6227020800.0);   // 1/13!
    hc = fma_t(y, hc, float(1.0 / 479001600.0));   // 1/12!
    hs = fma_t(y, hs, float(-1.0 / 39916800.0));   // -1/11!
    hc = fma_t(y, hc, float(-1.0 / 3628800.0));   // -1/10!
    hs = fma_t(y, hs, float(1.0 / 362880.0));   // 1/9!
    hc = fma_t(y, hc, float(1.0 / 40320.0));   // 1/8!
    hs = fma_t(y, hs, float(-1.0 / 5040.0));   // -1/7!
    pc = fma_t(y, small ? 0.0f : hc, pc);
    ps = fma_t(y, small ? 0.0f : hs, ps);
  }
  *c = fma_t(y, fma_t(y, pc, 1.0f / 24), -0.5f);
  *s = fma_t(y, fma_t(y, ps, -1.0f / 6), 1.0f);
}
template <bool kLong>
QLG_HD void phase_series(double y, bool small, double* c, double* s) {
  double pc = -1.0 / 3628800.0, ps = 1.0 / 362880.0;   // -1/10!, 1/9!
  if constexpr (kLong) {
    double hc = -1.0 / 1124000727777607680000.0;   // -1/22!
    double hs = 1.0 / 51090942171709440000.0;   // 1/21!
    hc = fma(y, hc, 1.0 / 2432902008176640000.0);   // 1/20!
    hs = fma(y, hs, -1.0 / 121645100408832000.0);   // -1/19!
    hc = fma(y, hc, -1.0 / 6402373705728000.0);   // -1/18!
    hs = fma(y, hs, 1.0 / 355687428096000.0);   // 1/17!
    hc = fma(y, hc, 1.0 / 20922789888000.0);   // 1/16!
    hs = fma(y, hs, -1.0 / 1307674368000.0);   // -1/15!
    hc = fma(y, hc, -1.0 / 87178291200.0);   // -1/14!
    hs = fma(y, hs, 1.0 / 6227020800.0);   // 1/13!
    hc = fma(y, hc, 1.0 / 479001600.0);   // 1/12!
    hs = fma(y, hs, -1.0 / 39916800.0);   // -1/11!
    pc = fma(y, small ? 0.0 : hc, pc);
    ps = fma(y, small ? 0.0 : hs, ps);
  }
  pc = fma(y, pc, 1.0 / 40320.0);
  ps = fma(y, ps, -1.0 / 5040.0);
  pc = fma(y, pc, -1.0 / 720.0);
  ps = fma(y, ps, 1.0 / 120.0);
  pc = fma(y, pc, 1.0 / 24.0);
  ps = fma(y, ps, -1.0 / 6.0);
  *c = fma(y, pc, -0.5);
  *s = fma(y, ps, 1.0);
}
// cos h and sin(h) / h as polynomials in y = h^2, for |h| <= 1/16 (first omitted terms
// h^10/10! = 3e-19 and h^10/11! in FP64, h^6/6! = 8e-11 and h^6/7! in FP32); kLong: |h| <= pi/2
// (h^24/24! = 8e-20 and h^22/23! = 8e-19, h^16/16! = 7e-11 and h^14/15! = 4e-10), in the same way.
template <bool kLong>
QLG_HD void half_angle_series(float y, bool small, float* c, float* s) {
  float pc = 1.0f / 24, ps = 1.0f / 120;
  if constexpr (kLong) {
    float hc = float(-1.0 / 87178291200.0);   // -1/14!
    hc = fma_t(y, hc, float(1.0 / 479001600.0));   // 1/12!
    float hs = float(1.0 / 6227020800.0);   // 1/13!
    hc = fma_t(y, hc, float(-1.0 / 3628800.0));   // -1/10!
    hs = fma_t(y, hs, float(-1.0 / 39916800.0));   // -1/11!
    hc = fma_t(y, hc, float(1.0 / 40320.0));   // 1/8!
    hs = fma_t(y, hs, float(1.0 / 362880.0));   // 1/9!
    hc = fma_t(y, hc, float(-1.0 / 720.0));   // -1/6!
    hs = fma_t(y, hs, float(-1.0 / 5040.0));   // -1/7!
    pc = fma_t(y, small ? 0.0f : hc, pc);
    ps = fma_t(y, small ? 0.0f : hs, ps);
  }
  *c = fma_t(y, fma_t(y, pc, -0.5f), 1.0f);
  *s = fma_t(y, fma_t(y, ps, -1.0f / 6), 1.0f);
}
template <bool kLong>
QLG_HD void half_angle_series(double y, bool small, double* c, double* s) {
  double pc = 1.0 / 40320.0, ps = 1.0 / 362880.0;
  if constexpr (kLong) {
    double hc = -1.0 / 1124000727777607680000.0;   // -1/22!
    hc = fma(y, hc, 1.0 / 2432902008176640000.0);   // 1/20!
    double hs = 1.0 / 51090942171709440000.0;   // 1/21!
    hc = fma(y, hc, -1.0 / 6402373705728000.0);   // -1/18!
    hs = fma(y, hs, -1.0 / 121645100408832000.0);   // -1/19!
    hc = fma(y, hc, 1.0 / 20922789888000.0);   // 1/16!
    hs = fma(y, hs, 1.0 / 355687428096000.0);   // 1/17!
    hc = fma(y, hc, -1.0 / 87178291200.0);   // -1/14!
    hs = fma(y, hs, -1.0 / 1307674368000.0);   // -1/15!
    hc = fma(y, hc, 1.0 / 479001600.0);   // 1/12!
    hs = fma(y, hs, 1.0 / 6227020800.0);   // 1/13!
    hc = fma(y, hc, -1.0 / 3628800.0);   // -1/10!
    hs = fma(y, hs, -1.0 / 39916800.0);   // -1/11!
    pc = fma(y, small ? 0.0 : hc, pc);
    ps = fma(y, small ? 0.0 : hs, ps);
  }
  pc = fma(y, pc, -1.0 / 720.0);
  ps = fma(y, ps, -1.0 / 5040.0);
  pc = fma(y, pc, 1.0 / 24.0);
  ps = fma(y, ps, 1.0 / 120.0);
  pc = fma(y, pc, -0.5);
  ps = fma(y, ps, -1.0 / 6.0);
  *c = fma(y, pc, 1.0);
  *s = fma(y, ps, 1.0);
}

// x less the nearest multiple k of pi: k times its two parts, each product exact in its multiply-add; x
// itself, exactly, where k is 0.
QLG_HD double rint_t(double x) { return rint(x); }
QLG_HD float rint_t(float x) { return rintf(x); }
template <typename T>
QLG_HD T reduce(T x, T* multiple) {
  constexpr double hi = 3.141592653589793, lo = 1.2246467991473532e-16;   // their sum is pi to 107 bits
  constexpr T hi_t = T(hi), lo_t = T(hi - double(hi_t) + lo);
  const T k = rint_t(x * T(1.0 / hi));
  *multiple = k;
  return fma_t(-k, lo_t, fma_t(-k, hi_t, x));
}
template <typename T>
QLG_HD bool is_odd(T k) { return T(2) * rint_t(T(0.5) * k) != k; }

// cos x0 - 1 and sin x0 of the density phase x0; (cos x2 - 1) / x2^2 and sin(x2) / x2 of the singlet
// phase x2; cos h and sin(h) / h of the half rotation, hh = h^2, up to their common sign, which the
// rotation (Rot2) and its derivative do not see.
template <typename T>
struct Series {
  T re0, im0, c2, s2, ch, sh;
};
template <typename T>
QLG_HD bool small_angles(T x0, T x2, T hh) {
  return fmax(fabs(x0), fabs(x2)) <= T(0.125) && hh <= T(1.0 / 256.0);
}
template <typename T>
QLG_HD Series<T> short_series(T x0, T x2, T hh) {
  Series<T> r;
  T c, s;
  phase_series<false>(x0 * x0, true, &c, &s);
  r.re0 = x0 * x0 * c;
  r.im0 = x0 * s;
  phase_series<false>(x2 * x2, true, &r.c2, &r.s2);
  half_angle_series<false>(hh, true, &r.ch, &r.sh);
  return r;
}

// The same for any arguments.  A site's result must not depend on the tile it lies in, so each angle takes
// its form by its own size, in the same instructions for all: reduced to pi/2, then the long series, which
// is the short one where all of the site's are small; only beyond kMostAngle the library's sine and cosine
// (three calls of it, in wavefronts of sites on both sides, took a 2048^2 step at angles up to several
// radians to 1322 us in complex128 and 705 us in complex64; this form 1083 and 568 us).  Not inlined: its
// constants would otherwise be hoisted out of the substep loops of every kernel, into registers that the
// usual path needs.
constexpr double kMostAngle = 4096;   // k below 2^11: exact products in FP32's reduction as well
template <typename T>
__host__ __device__ __attribute__((noinline)) inline Series<T> general_series(T x0, T x2, T hh) {
  const bool small = small_angles(x0, x2, hh);
  Series<T> r;
  T c, s, k;
  const T r0 = reduce(x0, &k);
  phase_series<true>(r0 * r0, small, &c, &s);
  r.re0 = r0 * r0 * c;
  r.im0 = r0 * s;
  if (!all_lanes(k == T(0))) {   // cos and sin change sign over an odd multiple
    const bool odd = is_odd(k);
    r.re0 = odd ? T(-2) - r.re0 : r.re0;
    r.im0 = odd ? -r.im0 : r.im0;
  }
  const T r2 = reduce(x2, &k);
  phase_series<true>(r2 * r2, small, &r.c2, &r.s2);
  if (!all_lanes(k == T(0))) {   // the same, over x2 instead of r2
    const bool turned = k != T(0), odd = is_odd(k);
    const T i2 = rcp_t(turned ? x2 : T(1)), co = r2 * r2 * r.c2, si = r2 * r.s2;
    r.c2 = turned ? (odd ? T(-2) - co : co) * i2 * i2 : r.c2;
    r.s2 = turned ? (odd ? -si : si) * i2 : r.s2;
  }
  T y = hh, q = T(1);
  if (!all_lanes(hh <= T(2.4))) {   // (pi/2)^2 = 2.467
    const bool turned = hh > T(2.4);
    const T ih = rsqrt_t(turned ? hh : T(1)), h0 = hh * ih;
    const T rh = reduce(fma_t(T(0.5) * ih, fma_t(-h0, h0, hh), h0), &k);   // of sqrt(hh)
    y = turned ? rh * rh : hh;
    q = turned ? rh * ih : T(1);
  }
  half_angle_series<true>(y, small, &r.ch, &r.sh);
  r.sh *= q;
  constexpr T most = T(kMostAngle);
  if (__builtin_expect(!all_lanes(fmax(fabs(x0), fabs(x2)) <= most && hh <= most * most), 0)) {
    if (fabs(x0) > most) {
      sincos_t(x0, &r.im0, &r.re0);
      r.re0 -= T(1);
    }
    if (fabs(x2) > most) {
      sincos_t(x2, &s, &c);
      const T i2 = rcp_t(x2);
      r.s2 = s * i2;
      r.c2 = (c - T(1)) * i2 * i2;
    }
    if (hh > most * most) {
      const T h = sqrt_t(hh);
      sincos_t(h, &s, &r.ch);
      r.sh = s * rcp_t(h);
    }
  }
  return r;
}

// R - I of the spin rotation R = exp(-i phi n.f), as the real 5 x 5 matrix that it is on
//   (s2, i t2, i s1, t1, x0),   s_m = x_m + x_-m,  t_m = x_m - x_-m
// (integer spin is a real representation, R_{-m',-m} = (-1)^{m'-m} conj R_{m'm}).  Rows 2 and 1
// give twice the correction of the m = +-2 and +-1 pairs' sums and differences; row 0 carries
// the factor UScale.  Names: row, then column; a trailing i marks an entry that multiplies
// i times its column.
//   S2 = ss22 s2 + i st22i t2 + i ss21i s1 + st21 t1 + s20 x0
//   T2 = tt22 t2 + i ts22i s2 + i tt21i t1 + ts21 s1 + i t20i x0   and so on.
//
// From the Cayley-Klein parameters A = c - i Z, B = -(Y + i X) of the rotation, with
// c = cos(phi/2) and (X, Y, Z) = sin(phi/2) n:
//   R22 = A^4, R21 = 2 A^3 B, R20 = sqrt6 A^2 B^2, R2-1 = 2 A B^3, R2-2 = B^4,
//   R12 = -2 A^3 B*, R11 = A^2 (1 - 4 s), R10 = sqrt6 A B (1 - 2 s), R1-1 = B^2 (3 - 4 s),
//   R1-2 = 2 A* B^3, R02 = sqrt6 A^2 B*^2, R01 = -sqrt6 A B* (1 - 2 s), R00 = 1 - 6 s + 6 s^2,
// s = |B|^2 = X^2 + Y^2.  A^2 = 1 - e - 2 i c Z with e = s + 2 Z^2, so that every entry of
// R - I is formed from small quantities (relative accuracy, no cancellation against 1), the
// direction of F is never divided out, and B = 0 (F along z) leaves every entry that couples
// |m| to another |m'| exactly zero.
//
// The self-interaction is what bounds the step kernels (vector instructions).  Building this
// matrix once per site takes about as many as the frame of F (Euler angles, d(beta), the phases
// of each m) that stood here before; applying R - I takes 50 multiplications and multiply-adds
// and 16 additions per 5-vector (and 10 for the base it is added to), where the frame took 138
// instructions.  With collide_r (40 additions per I' instead of 80) 20 steps of 2048^2 in complex128
// went from 19.7 to 16.4 ms, in complex64 with every component populated from 14.2 to 10.9 ms,
// 50 steps of 256 uneven 1D runs from 8.2 to 6.5 ms.
template <typename T>
struct Rot2 {
  T ss22, st22i, ss21i, st21, s20;
  T tt22, ts22i, tt21i, ts21, t20i;
  T ss11, st11i, ss12i, st12, s10i;
  T tt11, ts11i, tt12i, ts12, t10;
  T x0s2, x0t2i, x0s1i, x0t1, x00;
};

template <typename T>
QLG_HD void rot2(T c, T X, T Y, T Z, Rot2<T>& M) {
  constexpr T r6 = T(Consts::r6), r = T(UScale<T>::value);
  const T XX = X * X;
  const T s = fma_t(Y, Y, XX), B = fma_t(Y, Y, -XX), C = (X + X) * Y;   // B^2 = B + i C
  const T Z2 = Z + Z;
  const T e = fma_t(Z2, Z, s), be = -(Z2 * c), al = T(1) - e;           // A^2 = al + i be
  // m = +-2 block: R22 - 1 = p + i q, R2-2 = u + i v
  {
    const T p = fma_t(e, e - T(2), -(be * be)), q = (al + al) * be;
    const T u = fma_t(B, B, -(C * C)), v = (B + B) * C;
    M.ss22 = p + u;
    M.tt22 = p - u;
    M.st22i = q - v;
    M.ts22i = q + v;
  }
  // m = +-1 block: R11 - 1 = p + i q, R1-1 = u + i v
  {
    const T s4 = T(4) * s;
    const T p = -fma_t(s4, al, e), q = fma_t(-s4, be, be), k = T(3) - s4;
    const T u = k * B, v = k * C;
    M.ss11 = p + u;
    M.tt11 = p - u;
    M.st11i = q - v;
    M.ts11i = q + v;
  }
  // -2 A B = a1 + i a2, -2 A B* = a3 - i a4
  const T ZX = Z * X, ZY = Z * Y;
  const T ab1 = fma_t(c, Y, ZX), ab2 = fma_t(c, X, -ZY), ab3 = fma_t(c, Y, -ZX), ab4 = fma_t(c, X, ZY);
  const T a1 = ab1 + ab1, a2 = ab2 + ab2, a3 = ab3 + ab3, a4 = ab4 + ab4;
  {
    const T aB = al + B, aD = al - B, bB = be + C, bD = be - C;
    M.st21 = fma_t(a2, bD, -(a1 * aD));
    M.ts21 = fma_t(a2, bB, -(a1 * aB));
    M.ss21i = -fma_t(a1, bB, a2 * aB);
    M.tt21i = -fma_t(a1, bD, a2 * aD);
    M.st12 = fma_t(a4, bD, a3 * aB);
    M.ts12 = fma_t(a4, bB, a3 * aD);
    M.ss12i = fma_t(a3, bD, -(a4 * aB));
    M.tt12i = fma_t(a3, bB, -(a4 * aD));
  }
  {
    const T h1 = T(0.5) * r6 * a1, h2 = T(0.5) * r6 * a2;
    M.s20 = fma_t(h1, a1, -(h2 * a2));
    M.t20i = (h1 + h1) * a2;
    const T h3 = T(0.25) * r * r6 * a3, h4 = T(0.25) * r * r6 * a4;
    M.x0s2 = fma_t(h3, a3, -(h4 * a4));
    M.x0t2i = -((h3 + h3) * a4);
    const T k = fma_t(T(-2) * r6, s, r6);
    M.t10 = -(k * a1);
    M.s10i = -(k * a2);
    const T kr = T(0.5) * r * k;
    M.x0t1 = kr * a3;
    M.x0s1i = -(kr * a4);
    const T s6 = T(6) * r * s;
    M.x00 = fma_t(s6, s, -s6);
  }
}

// Coefficients of W for one site, computed once and applied to a and to b.
template <typename T>
struct WCoef {
  cx<T> p[5];   // psi = a + b
  cx<T> mu0;    // exp(-i (th g0 n + ext)) - 1
  cx<T> cs;     // exp(-i (th g0 n + ext)) (exp(-i th g2 n/5) - 1) / n  (0/0 -> its limit)
  Rot2<T> R;    // the spin rotation, less the identity
};

// kExt: the equation of motion carries the psi-independent term (V(x) + mu) psi_m
// (Sec. II, "Additional terms"); ext = theta (V(x) + mu) joins the density phase.
template <typename T, bool kExt = false>
QLG_HD void w_coefficients(const cx<T> (&a)[5], const cx<T> (&b)[5], const Angles<T> ang, WCoef<T>& W,
                           T ext = T(0)) {
#pragma unroll
  for (int m = 0; m < 5; ++m) W.p[m] = a[m] + b[m];
  const cx<T>* p = W.p;
  auto sq = [](cx<T> z) { return fma_t(z.re, z.re, z.im * z.im); };
  const T q0 = sq(p[0]), q1 = sq(p[1]), q3 = sq(p[3]), q4 = sq(p[4]);
  const T n = fma_t(p[2].re, p[2].re, fma_t(p[2].im, p[2].im, (q0 + q4) + (q1 + q3)));
  const T Fz = fma_t(T(2), q0 - q4, q1 - q3);
  // F_x + i F_y = psi^H f_+ psi = 2 (p2* p1 + p-1* p-2) + sqrt6 (p1* p0 + p0* p-1)
  auto cjmac = [](cx<T> x, cx<T> y, cx<T> acc) {   // acc + conj(x) y
    return cx<T>{fma_t(x.re, y.re, fma_t(x.im, y.im, acc.re)), fma_t(x.re, y.im, fma_t(-x.im, y.re, acc.im))};
  };
  auto cjmul = [](cx<T> x, cx<T> y) {              // conj(x) y
    return cx<T>{fma_t(x.re, y.re, x.im * y.im), fma_t(x.re, y.im, -(x.im * y.re))};
  };
  const cx<T> f1 = cjmac(p[0], p[1], cjmul(p[3], p[4]));
  const cx<T> f2 = cjmac(p[1], p[2], cjmul(p[2], p[3]));
  // (th g1 / 2) F: half the rotation vector
  const T k1 = T(0.5) * ang.tg1 * ang.fs, k2 = k1 + k1, k6 = T(Consts::r6) * k1;
  const T Hx = fma_t(k2, f1.re, k6 * f2.re), Hy = fma_t(k2, f1.im, k6 * f2.im), Hz = k1 * Fz;
  const T hh = fma_t(Hx, Hx, fma_t(Hy, Hy, Hz * Hz));
  const T x0 = kExt ? fma_t(ang.tg0, n, ext) : ang.tg0 * n;   // density phase
  const T x2 = ang.tg25 * n;                                  // singlet phase

  // exp(-i x) - 1 = x (x c - i s) with c = (cos x - 1)/x^2, s = sin(x)/x.  When every angle of
  // every lane is small (the usual case) all take short series without a branch per lane.
  const Series<T> f = __builtin_expect(all_lanes(small_angles(x0, x2, hh)), 1) ? short_series(x0, x2, hh)
                                                                               : general_series(x0, x2, hh);
  W.mu0 = cx<T>{f.re0, -f.im0};
  // singlet coefficient (exp(-i x2) - 1) / n = th g2/5 (x2 c - i s): no division by n, so empty or
  // denormal sites stay finite; times exp(-i x0) = 1 + mu0
  const cx<T> cs{ang.tg25 * x2 * f.c2, -(ang.tg25 * f.s2)};
  W.cs = cx<T>{fma_t(W.mu0.re, cs.re, fma_t(-W.mu0.im, cs.im, cs.re)),
               fma_t(W.mu0.re, cs.im, fma_t(W.mu0.im, cs.re, cs.im))};
  rot2(f.ch, f.sh * Hx, f.sh * Hy, f.sh * Hz, W.R);
}

// x <- UScale exp(-i th g0 n) R P x for one 5-vector x (a or b).
//
// With E = exp(-i th g0 n), R commutes with it and E P x = x + mu0 x + cs (v^H x) v (cs holds
// E): with y = E P x, R y = y + (R - I) y, the second term through the pairs' sums and
// differences.  The corrections (mu0 x and the singlet's; the rotation's) are each summed from small
// terms and added to the state last, so the full-magnitude value is rounded in FP64 twice per
// application (y, and the result): an RMS error of 6.6e-17 of the state, where sums that start from
// the state and round it at each multiply-add (20 instructions per vector fewer, 3 to 7 % of a
// step) made 1.6e-16 and the frame of F 9.1e-17.  In FP32 all corrections are added to x at once:
// rounding it after each factor made the FP32 qubit norm drift systematically (6e-5 over 20000
// steps of the 1D two-soliton run, against 9e-7 with one rounding).
template <typename T>
QLG_HD void w_apply(cx<T> (&x)[5], const WCoef<T>& W) {
  const cx<T>* p = W.p;
  const Rot2<T>& M = W.R;
  // s = v^H x, conj(v_m) = (-1)^m psi_{-m}
  auto mac = [](cx<T> u, cx<T> w, cx<T> acc) {     // acc + u w
    return cx<T>{fma_t(u.re, w.re, fma_t(-u.im, w.im, acc.re)), fma_t(u.re, w.im, fma_t(u.im, w.re, acc.im))};
  };
  auto msub = [](cx<T> u, cx<T> w, cx<T> acc) {    // acc - u w
    return cx<T>{fma_t(-u.re, w.re, fma_t(u.im, w.im, acc.re)), fma_t(-u.re, w.im, fma_t(-u.im, w.re, acc.im))};
  };
  auto mul = [](cx<T> u, cx<T> w) { return cx<T>{fma_t(u.re, w.re, -(u.im * w.im)), fma_t(u.re, w.im, u.im * w.re)}; };
  // acc + c z and acc + i c z, c real
  auto rmac = [](T c, cx<T> z, cx<T> acc) { return cx<T>{fma_t(c, z.re, acc.re), fma_t(c, z.im, acc.im)}; };
  auto imac = [](T c, cx<T> z, cx<T> acc) { return cx<T>{fma_t(-c, z.im, acc.re), fma_t(c, z.re, acc.im)}; };
  cx<T> s = mul(p[4], x[0]);
  s = msub(p[3], x[1], s);
  s = mac(p[2], x[2], s);
  s = msub(p[1], x[3], s);
  s = mac(p[0], x[4], s);
  const cx<T> tt = mul(W.cs, s);
  // e = mu0 x + tt v, v_m = (-1)^m conj(psi_{-m}); y = x + e
  constexpr bool kOnce = sizeof(T) == 4;
  auto corr = [&](cx<T> xm, cx<T> vm, bool neg) {
    const cx<T> v = neg ? cx<T>{-vm.re, vm.im} : cx<T>{vm.re, -vm.im};
    return mac(tt, v, mul(W.mu0, xm));
  };
  cx<T> e[5], y[5];
  e[0] = corr(x[0], p[4], false);
  e[1] = corr(x[1], p[3], true);
  e[2] = corr(x[2], p[2], false);
  e[3] = corr(x[3], p[1], true);
  e[4] = corr(x[4], p[0], false);
#pragma unroll
  for (int m = 0; m < 5; ++m) y[m] = x[m] + e[m];
  const cx<T> s2 = y[0] + y[4], t2 = y[0] - y[4], s1 = y[1] + y[3], t1 = y[1] - y[3], x0 = y[2];
  const cx<T> z{T(0), T(0)};
  // the rows of a pair take their terms in the same order, so that s == +-t stays so exactly
  // (a component that is zero and has no source stays zero)
  cx<T> S2 = imac(M.st22i, t2, z), T2 = imac(M.ts22i, s2, z);
  S2 = rmac(M.ss22, s2, S2);
  T2 = rmac(M.tt22, t2, T2);
  S2 = imac(M.ss21i, s1, S2);
  T2 = imac(M.tt21i, t1, T2);
  S2 = rmac(M.st21, t1, S2);
  T2 = rmac(M.ts21, s1, T2);
  S2 = rmac(M.s20, x0, S2);
  T2 = imac(M.t20i, x0, T2);
  cx<T> S1 = imac(M.st11i, t1, z), T1 = imac(M.ts11i, s1, z);
  S1 = rmac(M.ss11, s1, S1);
  T1 = rmac(M.tt11, t1, T1);
  S1 = imac(M.ss12i, s2, S1);
  T1 = imac(M.tt12i, t2, T1);
  S1 = rmac(M.st12, t2, S1);
  T1 = rmac(M.ts12, s2, T1);
  S1 = imac(M.s10i, x0, S1);
  T1 = rmac(M.t10, x0, T1);
  cx<T> X0 = rmac(M.x00, x0, kOnce ? e[2] : z);
  X0 = rmac(M.x0s2, s2, X0);
  X0 = imac(M.x0t2i, t2, X0);
  X0 = imac(M.x0s1i, s1, X0);
  X0 = rmac(M.x0t1, t1, X0);
  if constexpr (kOnce) {
    const T h = T(0.5);
    x[0] = x[0] + rmac(h, S2 + T2, e[0]);
    x[4] = x[4] + rmac(h, S2 - T2, e[4]);
    x[1] = x[1] + rmac(h, S1 + T1, e[1]);
    x[3] = x[3] + rmac(h, S1 - T1, e[3]);
    x[2] = x[2] + X0;
  } else {
    const T h = T(2);
    x[0] = rmac(h, y[0], S2 + T2);
    x[4] = rmac(h, y[4], S2 - T2);
    x[1] = rmac(h, y[1], S1 + T1);
    x[3] = rmac(h, y[3], S1 - T1);
    x[2] = rmac(h, y[2], X0);
  }
}

template <typename T, bool kExt = false>
QLG_HD void potential(cx<T> (&a)[5], cx<T> (&b)[5], const Angles<T> ang, T ext = T(0)) {
  WCoef<T> W;
  w_coefficients<T, kExt>(a, b, ang, W, ext);
  w_apply(a, W);
  w_apply(b, W);
}

}  // namespace qlg

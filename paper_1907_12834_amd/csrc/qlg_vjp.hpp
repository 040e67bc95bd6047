// Reverse-mode derivative (vector-Jacobian product) of one self-interaction
// application U(theta) at one site, in FP64.
//
// Forward (qlg_math.hpp): for x in {a, b},
//   y1_x = P x = x + c(n) s_x v,  s_x = v^H x,   c(n) = (e^{-i kappa n} - 1)/n, kappa = theta g2/5,
//   y_x  = E R y1_x,   E = e^{-i (theta g0 n + ext)},   R = exp(-i tau F.f), tau = theta g1,
// (ext = theta (V + mu) when the equation carries a potential), with psi = a + b, n = |psi|^2,
// F_nu = psi^H f_nu psi, v = S psi* (all frozen at the input).  Cotangents follow
// lambda = dL/dRe z + i dL/dIm z, so for a complex-linear map y = M z the pull-back is
// lambda_z = M^H lambda_y.
//
// With m_x = R^H E* lambda_x, the cotangent of y1_x (R^H = R^T on the real basis of Rot2):
//   dL/dn  (density) = th g0 A,  dL/dg0 = th n A,   A = sum_x Im(m_x^H y1_x),
//   dL/dF = tau J T,  dL/dg1 = th F.T,   T_nu = sum_x Im(m_x^H f_nu y1_x),
// since R^-1 dR = -i (J_r dphi).f for a change of the rotation vector phi = tau F, J_r being the
// right Jacobian of the rotation group, and J = J_r^T its transpose:
//   J T = sinc(phi) T + (1 - sinc(phi))/phi^2 (phi.T) phi + (1 - cos(phi))/phi^2 phi x T.
// No frame of F and no forward rotation is formed.  The singlet factor contributes, per x with
// w = v^H m_x,
//   lambda_x  = P^H m = m + conj(c) w v,
//   lambda_psi += conj(c) w S x* + c s_x S conj(m),
//   dL/dn += Re(c'(n) s_x conj(w)),   dL/dg2 += Re(dc/dg2 s_x conj(w)).
// Finally lambda_psi += 2 dL/dn psi + 2 sum_nu dL/dF_nu f_nu psi and
// lambda_a = P^H m_a + lambda_psi, lambda_b = P^H m_b + lambda_psi.
//
// About 1000 vector instructions, where the derivative in the frame of F (Euler angles, d(beta), the
// divided differences of each m) took 1525.
#pragma once

#include "qlg_math.hpp"

namespace qlg {

// x <- (R^T E* x), M = R - I as rot2<double> forms it and mu0 = E - 1.  On the coordinates
// (s2, i t2, i s1, t1, x0) transposing M swaps its entries; the factors 2 of row and column 0
// (UScale, and the unnormalised sums) are the same for M^T.
QLG_HD void rotate_back(cx<double> (&x)[5], const Rot2<double>& M, cx<double> mu0) {
  auto rmac = [](double c, cx<double> z, cx<double> acc) { return cx<double>{fma(c, z.re, acc.re), fma(c, z.im, acc.im)}; };
  auto imac = [](double c, cx<double> z, cx<double> acc) { return cx<double>{fma(-c, z.im, acc.re), fma(c, z.re, acc.im)}; };
  cx<double> y[5];
  for (int m = 0; m < 5; ++m)   // x + conj(mu0) x
    y[m] = cx<double>{fma(mu0.re, x[m].re, fma(mu0.im, x[m].im, x[m].re)),
                      fma(mu0.re, x[m].im, fma(-mu0.im, x[m].re, x[m].im))};
  const cx<double> s2 = y[0] + y[4], t2 = y[0] - y[4], s1 = y[1] + y[3], t1 = y[1] - y[3], x0 = y[2];
  cx<double> S2 = imac(-M.ts22i, t2, s2), T2 = imac(-M.st22i, s2, t2);
  S2 = rmac(M.ss22, s2, S2);
  T2 = rmac(M.tt22, t2, T2);
  S2 = imac(-M.ss12i, s1, S2);
  T2 = imac(-M.tt12i, t1, T2);
  S2 = rmac(M.ts12, t1, S2);
  T2 = rmac(M.st12, s1, T2);
  S2 = rmac(M.x0s2, x0, S2);
  T2 = imac(-M.x0t2i, x0, T2);
  cx<double> S1 = imac(-M.ts11i, t1, s1), T1 = imac(-M.st11i, s1, t1);
  S1 = rmac(M.ss11, s1, S1);
  T1 = rmac(M.tt11, t1, T1);
  S1 = imac(-M.ss21i, s2, S1);
  T1 = imac(-M.tt21i, t2, T1);
  S1 = rmac(M.ts21, t2, S1);
  T1 = rmac(M.st21, s2, T1);
  S1 = imac(-M.x0s1i, x0, S1);
  T1 = rmac(M.x0t1, x0, T1);
  cx<double> X0 = rmac(M.x00, x0, x0 + x0);
  X0 = rmac(M.s20, s2, X0);
  X0 = imac(-M.t20i, t2, X0);
  X0 = imac(-M.s10i, s1, X0);
  X0 = rmac(M.t10, t1, X0);
  x[0] = 0.5 * (S2 + T2);
  x[4] = 0.5 * (S2 - T2);
  x[1] = 0.5 * (S1 + T1);
  x[3] = 0.5 * (S1 - T1);
  x[2] = 0.5 * X0;
}

// Keeps the instructions before and after it apart: interleaving the stages of potential_vjp would
// hold more values than the 256 registers of two wavefronts per SIMD.
QLG_HD void stage_end() {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_sched_barrier(0);
#endif
}

// In: a, b (input of U), la, lb (cotangents of U's outputs).
// Out: la, lb replaced by cotangents of a, b; dg[0..2] incremented.
QLG_HD void potential_vjp(const cx<double> (&a)[5], const cx<double> (&b)[5], cx<double> (&la)[5],
                          cx<double> (&lb)[5], double theta, double g0, double g1, double g2, double (&dg)[3],
                          double ext = 0.0) {
  static_assert(UScale<double>::value == 2, "rotate_back takes row 0 of R - I with the factor 2");
  const double r6 = Consts::r6;
  const double tau = theta * g1, kappa = theta * g2 * 0.2;
  cx<double> p[5];
  for (int m = 0; m < 5; ++m) p[m] = a[m] + b[m];
  double q[5];
  for (int m = 0; m < 5; ++m) q[m] = fma(p[m].re, p[m].re, p[m].im * p[m].im);
  const double n = (q[0] + q[4]) + (q[1] + q[3]) + q[2];
  const double Fz = fma(2.0, q[0] - q[4], q[1] - q[3]);
  const cx<double> f1 = cmulc(p[0], p[1]) + cmulc(p[3], p[4]);
  const cx<double> f2 = cmulc(p[1], p[2]) + cmulc(p[2], p[3]);
  const double Fx = fma(2.0, f1.re, r6 * f2.re), Fy = fma(2.0, f1.im, r6 * f2.im);
  const double ht = 0.5 * tau, Hx = ht * Fx, Hy = ht * Fy, Hz = ht * Fz;   // half the rotation vector
  const double hh = fma(Hx, Hx, fma(Hy, Hy, Hz * Hz));
  const double x0 = fma(theta * g0, n, ext), x2 = kappa * n;

  // the phases and the half rotation (Series); pd = (sin(x2)/x2 - cos x2)/x2^2 (for c'(n));
  // pj = (1 - sinc(phi))/phi^2, phi = 2 h
  Series<double> f;
  double pd, pj;
  auto pd_series = [](double y) {   // first omitted term y^5/518918400 (|x2| < 0.1: 2e-19)
    return fma(y, fma(y, fma(y, fma(y, 1.0 / 3991680.0, -1.0 / 45360.0), 1.0 / 840.0), -1.0 / 30.0), 1.0 / 3.0);
  };
  auto pj_series = [](double y) {   // y = phi^2 <= 1/64: first omitted term y^5/6227020800 (1e-19)
    return fma(y, fma(y, fma(y, fma(y, 1.0 / 39916800.0, -1.0 / 362880.0), 1.0 / 5040.0), -1.0 / 120.0), 1.0 / 6.0);
  };
  if (__builtin_expect(all_lanes(fmax(fabs(x0), fabs(x2)) <= 0.1 && hh <= 1.0 / 256.0), 1)) {
    f = short_series(x0, x2, hh);
    pd = pd_series(x2 * x2);
    pj = pj_series(4.0 * hh);
  } else {   // each by the site's own angles
    f = general_series(x0, x2, hh);
    const double y2 = x2 * x2;
    pd = fabs(x2) <= 0.1 ? pd_series(y2) : (f.s2 - fma(y2, f.c2, 1.0)) * rcp_t(y2);
    pj = hh <= 1.0 / 256.0 ? pj_series(4.0 * hh) : (1.0 - f.sh * f.ch) * rcp_t(4.0 * hh);
  }
  const cx<double> mu0{f.re0, -f.im0};
  const cx<double> cs{kappa * x2 * f.c2, -(kappa * f.s2)};        // c(n)
  Rot2<double> R;
  rot2(f.ch, f.sh * Hx, f.sh * Hy, f.sh * Hz, R);
  // both cotangents first: R's 25 entries are then free
  rotate_back(la, R, mu0);
  rotate_back(lb, R, mu0);
  stage_end();

  auto mac = [](cx<double> u, cx<double> w, cx<double> acc) {     // acc + u w
    return cx<double>{fma(u.re, w.re, fma(-u.im, w.im, acc.re)), fma(u.re, w.im, fma(u.im, w.re, acc.im))};
  };
  auto vdot = [&](const cx<double>(&x)[5]) {   // v^H x, conj(v_m) = (-1)^m psi_{-m}
    cx<double> s = p[4] * x[0];
    s = mac(cx<double>{-p[3].re, -p[3].im}, x[1], s);
    s = mac(p[2], x[2], s);
    s = mac(cx<double>{-p[1].re, -p[1].im}, x[3], s);
    return mac(p[0], x[4], s);
  };
  auto v_of = [&](int m) {   // v_m = (-1)^m conj(psi_{-m})
    const cx<double> z = p[4 - m];
    return (m == 1 || m == 3) ? cx<double>{-z.re, z.im} : cx<double>{z.re, -z.im};
  };
  cx<double> lpsi[5] = {};
  double t[5] = {0.0, 0.0, 0.0, 0.0, 0.0};               // Im(conj(m_i) y1_i), summed over a and b
  double io = 0.0, ii = 0.0, ro = 0.0, ri = 0.0;         // the f_x and f_y sums of outer and inner pairs
  cx<double> sw{0.0, 0.0};                               // s conj(w)
  // one 5-vector x; l holds m on entry and P^H m on exit
  auto one = [&](const cx<double>(&x)[5], cx<double>(&l)[5]) {
    const cx<double> s = vdot(x), w = vdot(l);
    const cx<double> k2 = cs * s, k1 = cmulc(cs, w);
    sw = sw + cmulc(w, s);
    cx<double> y[5];
    for (int m = 0; m < 5; ++m) y[m] = mac(k2, v_of(m), x[m]);
    for (int m = 0; m < 5; ++m) t[m] = fma(l[m].re, y[m].im, fma(-l[m].im, y[m].re, t[m]));
    for (int i = 0; i < 4; ++i) {
      // conj(m_i) y_{i+1} and conj(m_{i+1}) y_i: the sum of their imaginary parts, the difference of
      // their real parts
      double& im = (i == 0 || i == 3) ? io : ii;
      double& re = (i == 0 || i == 3) ? ro : ri;
      im = fma(l[i].re, y[i + 1].im, fma(-l[i].im, y[i + 1].re, im));
      im = fma(l[i + 1].re, y[i].im, fma(-l[i + 1].im, y[i].re, im));
      re = fma(l[i].re, y[i + 1].re, fma(l[i].im, y[i + 1].im, re));
      re = fma(-l[i + 1].re, y[i].re, fma(-l[i + 1].im, y[i].im, re));
    }
    for (int m = 0; m < 5; ++m) {
      // (S z)_m = (-1)^m z_{-m}
      const double sg = (m == 1 || m == 3) ? -1.0 : 1.0;
      const cx<double> xs{sg * x[4 - m].re, -sg * x[4 - m].im}, ls{sg * l[4 - m].re, -sg * l[4 - m].im};
      lpsi[m] = mac(k1, xs, mac(k2, ls, lpsi[m]));
    }
    for (int m = 0; m < 5; ++m) l[m] = mac(k1, v_of(m), l[m]);
  };
  one(a, la);
  stage_end();
  one(b, lb);
  const double A = ((t[0] + t[4]) + (t[1] + t[3])) + t[2];
  const double Tx = fma(0.5 * r6, ii, io), Ty = -fma(0.5 * r6, ri, ro), Tz = fma(2.0, t[0] - t[4], t[1] - t[3]);
  // c'(n) = kappa^2 (-(s + c) + i x2 pd), dc/dg2 = -i theta/5 e^{-i x2}
  const cx<double> dcn{-(kappa * kappa) * (f.s2 + f.c2), kappa * kappa * x2 * pd};
  const cx<double> ekn{fma(x2 * x2, f.c2, 1.0), -(x2 * f.s2)};
  const double dn = fma(theta * g0, A, fma(dcn.re, sw.re, -(dcn.im * sw.im)));
  dg[0] += theta * n * A;
  dg[1] += theta * fma(Fx, Tx, fma(Fy, Ty, Fz * Tz));
  dg[2] += (0.2 * theta) * fma(ekn.re, sw.im, ekn.im * sw.re);
  // dL/dF = tau J T with phi = 2 H
  const double jt = f.sh * f.ch, jx = f.sh * f.sh, jp = 4.0 * pj * fma(Hx, Tx, fma(Hy, Ty, Hz * Tz));
  const double LFx = tau * fma(jt, Tx, fma(jp, Hx, jx * fma(Hy, Tz, -(Hz * Ty))));
  const double LFy = tau * fma(jt, Ty, fma(jp, Hy, jx * fma(Hz, Tx, -(Hx * Tz))));
  const double LFz = tau * fma(jt, Tz, fma(jp, Hz, jx * fma(Hx, Ty, -(Hy * Tx))));
  // lambda_psi += 2 dn psi + 2 (LFz f_z + (LFx - i LFy)/2 f_+ + (LFx + i LFy)/2 f_-) psi
  const double d2 = 2.0 * dn, z2 = 2.0 * LFz;
  const cx<double> co{2.0 * LFx, -2.0 * LFy}, ci{r6 * LFx, -(r6 * LFy)};   // f_+ of outer and inner pairs
  const double dz[5] = {fma(2.0, z2, d2), d2 + z2, d2, d2 - z2, fma(-2.0, z2, d2)};
  for (int i = 0; i < 5; ++i) {
    cx<double> u = rfma(dz[i], p[i], lpsi[i]);
    if (i < 4) u = mac((i == 0 || i == 3) ? co : ci, p[i + 1], u);
    if (i > 0) u = mac(conj((i == 1 || i == 4) ? co : ci), p[i - 1], u);
    la[i] = la[i] + u;
    lb[i] = lb[i] + u;
  }
}

}  // namespace qlg

// Pointwise physics of the FP64 step in closed form: what the templates of
// physics.h, invert.h and implicit.h form from 4x4 contractions, from the
// 3 + 1 split instead.  With u~^i the velocity relative to the normal
// observer, gamma = sqrt(1 + g_ij u~^i u~^j), beta = alpha^2 g^{tr} (the
// shift, radial alone on Kerr-Schild, none in flat space):
//   u_i = g_ij u~^j,  u_t = -alpha gamma + beta u_r,  u^t = gamma/alpha;
//   B_i = g_ij B^j, B_t = beta B_r, bt = B^i u_i:  b^t = bt,
//   b_mu = (B_mu + bt u_mu)/u^t,  b^2 = (B^i B_i + bt^2)/(u^t)^2;
//   of two frames, u . r = -gamma_u gamma_r + u~^i r_i.
//
// What bounds it: FP64 issue.  A wavefront issues an FMA in 4.4 cycles and
// spends 64 on an IEEE division, 91 on sqrt (measured, independent chains of
// each); the template residual has 18 divisions and 12 square roots, half its
// time.  Here quotients share refined reciprocals (recip: 33 cycles), square
// roots skip the scaling of arguments that cannot be denormal (root: 60),
// and the reciprocal of a root comes out of the root's own iteration.
#pragma once
#include "implicit.h"

// 1/x to the last bit or two for normal x (up to 1e307); zero, an infinity or a
// denormal gives NaN.  So the callers' arguments are sums with a term that is
// bounded away from zero (1 + gamma, (1 - c^2) (u^t)^2 - c^2 g^tt, an enthalpy
// with its rest mass, a norm set to 1e-300 where it vanishes), bounded where
// they may overflow (an optical depth), or checked afterwards: an evaluation
// whose residual is not finite fails, as with the IEEE forms, except that a
// norm beyond 1e308 fails it too instead of passing for an error of zero.
DEV double recip(double x) {
#ifdef __HIP_DEVICE_COMPILE__
  double y = __builtin_amdgcn_rcp(x);
  y = __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
  return __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
#else
  return 1.0 / x;
#endif
}
// a/b, correctly rounded up to rare ties, from y = 1/b to a few bits
DEV double quot(double a, double b, double y) {
  const double q = a * y;
  return __builtin_fma(__builtin_fma(-b, q, a), y, q);
}
DEV double quot(double a, double b) { return quot(a, b, recip(b)); }
// sqrt(x) and its reciprocal for normal x (Goldschmidt's coupled iteration
// from the hardware's estimate, then the residual's correction); an infinity
// gives NaN.  The arguments are 1 + u~^2 and the limiter's polynomials.
DEV double root(double x, double& inv) {
#ifdef __HIP_DEVICE_COMPILE__
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  double r = __builtin_fma(-h, g, 0.5);
  g = __builtin_fma(g, r, g);
  h = __builtin_fma(h, r, h);
  r = __builtin_fma(-h, g, 0.5);
  g = __builtin_fma(g, r, g);
  h = __builtin_fma(h, r, h);
  g = __builtin_fma(__builtin_fma(-g, g, x), h, g);
  inv = h + h;
  return g;
#else
  const double g = ::sqrt(x);
  inv = 1.0 / g;
  return g;
#endif
}
DEV double root(double x) {
  double i;
  return root(x, i);
}
// the same where x may be zero or denormal: zero up to 1e-300.  These are
// norms, to which a larger term is added, and the discriminant of speeds, where
// 1e-150 of c is nothing
DEV double root0(double x) { return x > 1e-300 ? root(fmax(x, 1e-300)) : 0.0; }

// v_i = g_ij v^j
template <class M>
DEV void low3(const M& m, const double v[3], double o[3]) {
  if constexpr (M::diagonal) {
#pragma unroll
    for (int i = 0; i < 3; i++) o[i] = v[i];
  } else {
    o[0] = m.g11 * v[0] + m.g13 * v[2];
    o[1] = m.g22 * v[1];
    o[2] = m.g13 * v[0] + m.g33 * v[2];
  }
}
// gamma^{ij} v_j
template <class M>
DEV void up3(const M& m, const double v[3], double o[3]) {
  if constexpr (M::diagonal) {
#pragma unroll
    for (int i = 0; i < 3; i++) o[i] = v[i];
  } else {
    o[0] = m.gam11 * v[0] + m.u13 * v[2];
    o[1] = m.u22 * v[1];
    o[2] = m.u13 * v[0] + m.u33 * v[2];
  }
}
DEV double dot3(const double a[3], const double b[3]) {
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}
// gamma^{ij} v_i v_j
template <class M>
DEV double norm3sq(const M& m, const double v[3]) {
  double o[3];
  up3(m, v, o);
  return dot3(v, o);
}

// ---------------------------------------------------------------------------
// The PMHD residual of the implicit solve (Sec. 4.8) and its Jacobian.
// ---------------------------------------------------------------------------
// One cell's constants: the explicit state per sqrt(-g) and what every
// evaluation would form anew from it.
template <class M>
struct PCell {
  M m;
  double ia, beta;                // 1/alpha, the shift
  double D, iD, B[3], Bl[3], Bt, B2;  // rho u^t, its reciprocal, B^i, B_i, B_t, B^i B_i
  double Tgi[4], Ri[4];
  double nTs, nRs;                // norms of the spatial parts of Tgi, Ri
  double w[3];                    // sqrt(gamma^{ii})
  double dt, ca, ce;
};

template <class M>
DEV void pcell_setup(const M& m, const double Ui[12], double dt, double ca, double ce, PCell<M>& c) {
  c.m = m;
  const double igd = 1.0 / m.gdet;
  c.ia = 1.0 / m.alpha;
  c.beta = M::diagonal ? 0.0 : m.alpha * m.alpha * m.up(0, 1);
  c.D = Ui[0] * igd;
  c.iD = 1.0 / c.D;
#pragma unroll
  for (int i = 0; i < 3; i++) c.B[i] = Ui[5 + i] * igd;
  low3(m, c.B, c.Bl);
  c.Bt = c.beta * c.Bl[0];
  c.B2 = dot3(c.B, c.Bl);
#pragma unroll
  for (int k = 0; k < 4; k++) {
    c.Tgi[k] = Ui[1 + k] * igd;
    c.Ri[k] = Ui[8 + k] * igd;
  }
  c.nTs = root0(norm3sq(m, c.Tgi + 1));
  c.nRs = root0(norm3sq(m, c.Ri + 1));
#pragma unroll
  for (int i = 0; i < 3; i++) c.w[i] = ::sqrt(m.gam(i, i));
  c.dt = dt;
  c.ca = ca;
  c.ce = ce;
}

// Result of one evaluation: the gas residual, the total error, the dependent
// primitives.
struct PEval {
  double Eg[4], eT;
  double rho, Eb, ur[3];
  int radflags, ok;
};

// M1 inversion of R^t_nu with the TYPE2 limiter (Sec. 4.6): p_rad = Ebar/3,
// the frame's gamma_r, u~_r^i = f U~^i, and their derivatives with respect
// to E = E_rad and U = U~^2 (f_d: f for the derivatives, which at zero flux
// keep their limit).  gamma_r^2 = a/b with a = 2 - y + sqrt(4 - 3y),
// b = 4(1 - y); p_rad = E b/(4a - b); f = (4a - b)/(4 E sqrt(a b)).
struct RadState {
  double p, gr, f, fd;
  double pE, pU, gE, gU, fE, fU;
  int flags;
};
template <bool JAC>
DEV void rad_state(const Phys& ph, double E, double U, RadState& s) {
  s.flags = 0;
  const bool small = !(E > 1e-140);
  double iE = 0.0, y = 0.0;
  if (small) {
    y = (E != 0.0) ? U / (E * E) : 0.0;
    iE = 1.0 / E;
  } else {
    iE = recip(E);
    y = quot(U, E * E, iE * iE);
  }
  s.flags = (E <= 0.0) ? 1 : (y >= ph.ymax ? 2 : 0);
  if (JAC) s.pE = s.pU = s.gE = s.gU = s.fE = s.fU = 0.0;
  if (s.flags) {
    const double G2 = ph.gamma_max * ph.gamma_max;
    s.p = 1e-150 * (1.0 / 3.0);
    s.gr = 1.0;
    s.f = s.fd = 0.0;
    if (U > 0.0) {
      const double ip = 1.0 / (4.0 * G2 - 1.0), q = ::sqrt(U * (1.0 / ph.ymax));
      s.p = (1e-150 + q) * ip;
      s.gr = ph.gamma_max;
      s.f = s.fd = ::sqrt((G2 - 1.0) / U);
      if (JAC) {
        s.pU = 0.5 * q / U * ip;
        s.fU = -0.5 * s.f / U;
      }
    }
  } else if (y <= 0.0) {
    s.p = E * (1.0 / 3.0);
    s.gr = 1.0;
    s.f = 0.0;
    s.fd = 0.75 * iE;
    if (JAC) s.pE = 1.0 / 3.0;
  } else {
    double is, iab;
    const double q = root(4.0 - 3.0 * y, is);
    const double a = 2.0 - y + q, b = 4.0 * (1.0 - y), c4 = 4.0 * a - b;
    root(a * b, iab);
    const double ic = recip(c4);
    s.p = E * b * ic;
    s.gr = a * iab;
    s.f = s.fd = 0.25 * c4 * iE * iab;
    if (JAC) {
      const double ay = -1.0 - 1.5 * is;          // da/dy; db/dy = -4
      const double yU = iE * iE, yE = -2.0 * y * iE;
      const double py = E * ic * (-4.0 - b * ic * (4.0 * ay + 4.0));
      const double ib = a * iab * iab;            // 1/b
      const double gy = 0.5 * (a * iab) * (ay * iab * iab * b + 4.0 * ib);
      s.pE = b * ic + py * yE;
      s.pU = py * yU;
      s.gE = gy * yE;
      s.gU = gy * yU;
      // f = 1/(4 p gamma_r)
      const double lp = c4 * iE * ib, lg = iab * b;   // 1/p, 1/gamma_r
      s.fE = -s.f * (s.pE * lp + s.gE * lg);
      s.fU = -s.f * (s.pU * lp + s.gU * lg);
    }
  }
}

// The gas at x = (u_g, u~^i): velocity, field, T^t_nu (+ rho u^t in the energy
// slot).
struct GasState {
  double g, ig, u0, iu0, ul[3], utl;   // gamma, u^t, their reciprocals, u_i, u_t
  double rho, p, bt, bsq, bl[4], wg, Dw;
  double T[4];
};
template <class M>
DEV void gas_state(const PCell<M>& c, double gam, const double x[4], GasState& s) {
  const double al = c.m.alpha;
  const double* ut = x + 1;
  low3(c.m, ut, s.ul);
  const double q = dot3(ut, s.ul);
  s.g = root(1.0 + q, s.ig);
  s.u0 = M::diagonal ? s.g : quot(s.g, al, c.ia);
  s.iu0 = M::diagonal ? s.ig : al * s.ig;
  const double bu = M::diagonal ? 0.0 : c.beta * s.ul[0];
  s.utl = M::diagonal ? -s.g : bu - al * s.g;
  // 1 + u_t, free of the rest-mass cancellation
  const double opu = ((1.0 - al) - quot(al * q, 1.0 + s.g)) + bu;
  s.rho = quot(c.D, s.u0, s.iu0);
  s.bt = dot3(c.B, s.ul);
  s.bsq = (c.B2 + s.bt * s.bt) * (s.iu0 * s.iu0);
  s.bl[0] = (c.Bt + s.bt * s.utl) * s.iu0;
#pragma unroll
  for (int i = 0; i < 3; i++) s.bl[1 + i] = (c.Bl[i] + s.bt * s.ul[i]) * s.iu0;
  s.p = (gam - 1.0) * x[0];
  s.wg = x[0] + s.p + s.bsq;
  const double wu = s.wg * s.u0;
  s.Dw = c.D + wu;
  s.T[0] = (c.D * opu + wu * s.utl - s.bt * s.bl[0]) + (s.p + 0.5 * s.bsq);
#pragma unroll
  for (int i = 0; i < 3; i++) s.T[1 + i] = s.Dw * s.ul[i] - s.bt * s.bl[1 + i];
}

// Residual at x = (u_g, u~^i) and, with JAC, J[nu][k] = dE_nu/dx_k.
template <bool JAC, class M>
DEV void pmhd_eval(const PCell<M>& c, const Phys& ph, const double x[4], PEval& e, double J[4][4]) {
  const M& m = c.m;
  const double al = m.alpha, gm1 = ph.gam - 1.0;
  const double* ut = x + 1;
  GasState gs;
  gas_state(c, ph.gam, x, gs);
  const double(&ul)[3] = gs.ul, (&bl)[4] = gs.bl, (&T)[4] = gs.T;
  const double g = gs.g, ig = gs.ig, u0 = gs.u0, iu0 = gs.iu0, utl = gs.utl, rho = gs.rho;
  const double p = gs.p, bt = gs.bt, bsq = gs.bsq, wg = gs.wg, Dw = gs.Dw;
  double R[4];
#pragma unroll
  for (int k = 0; k < 4; k++) R[k] = c.Ri[k] - (T[k] - c.Tgi[k]);
  // radiation
  const double Er = M::diagonal ? -R[0] : c.beta * R[1] - R[0];
  double Ut[3];
  up3(m, R + 1, Ut);
  if (!M::diagonal) {
#pragma unroll
    for (int i = 0; i < 3; i++) Ut[i] *= al;
  }
  const double U2 = al * dot3(Ut, R + 1);
  RadState s;
  rad_state<JAC>(ph, Er, U2, s);
  double rl[4];
  const double fa = s.f * al;
#pragma unroll
  for (int i = 0; i < 3; i++) rl[1 + i] = fa * R[1 + i];
  rl[0] = M::diagonal ? -s.gr : c.beta * rl[1] - al * s.gr;
  const double w = dot3(ut, rl + 1) - g * s.gr;
  const double c43 = 4.0 * s.p * w;
  const double Eh = c43 * w - s.p;
  // 4-force: G_nu = -(P1 r_nu + P2 u_nu)
  const double Tg = (p * c.iD) * u0;   // p/rho, 1/rho = u^t/D
  const double T2 = Tg * Tg;
  const double ka = c.ca * rho, ke = c.ce * rho, kt = ka + ke;
  const double lam = ka * ph.arad * (T2 * T2);
  const double P1 = kt * c43, P2 = kt * s.p + lam + ke * Eh;
  double Gd[4], Rr[4];
  Gd[0] = -c.dt * (P1 * rl[0] + P2 * utl);
#pragma unroll
  for (int i = 0; i < 3; i++) Gd[1 + i] = -c.dt * (P1 * rl[1 + i] + P2 * ul[i]);
  const double r43 = 4.0 * s.p * (s.gr * c.ia);
#pragma unroll
  for (int k = 0; k < 4; k++) Rr[k] = r43 * rl[k];
  Rr[0] += s.p;
  double Ee[4];
#pragma unroll
  for (int k = 0; k < 4; k++) {
    e.Eg[k] = (T[k] - c.Tgi[k]) - Gd[k];
    Ee[k] = (Rr[k] - c.Ri[k]) + Gd[k];
  }
  // errors (Sec. 4.8), as norm_errors
  {
    const double g0 = ::fabs(Gd[0]), gn = root0(norm3sq(m, Gd + 1));
    double ntg = ::fabs(T[0]) + ::fabs(c.Tgi[0]) + g0;
    double ntr = ::fabs(Rr[0]) + ::fabs(c.Ri[0]) + g0;
    if (!(ntg > 0.0)) ntg = 1e-300;
    if (!(ntr > 0.0)) ntr = 1e-300;
    const double nsg = root0(norm3sq(m, T + 1)) + c.nTs + gn + ntg;
    const double nsr = root0(norm3sq(m, Rr + 1)) + c.nRs + gn + ntr;
    double t = (s.flags & 1) ? 0.0 : fmax(::fabs(e.Eg[0]) * recip(ntg), ::fabs(Ee[0]) * recip(ntr));
    const double ig3 = recip(nsg), ir3 = recip(nsr);
#pragma unroll
    for (int i = 0; i < 3; i++)
      t += c.w[i] * fmax(::fabs(e.Eg[1 + i]) * ig3, ::fabs(Ee[1 + i]) * ir3);
    e.eT = 0.25 * t;
    e.ok = 1;
    // an overflow or an invalid operation anywhere ends up in the sum (fmax
    // alone would drop a NaN)
    const double sum = e.eT + (e.Eg[0] + Ee[0]) + (e.Eg[1] + Ee[1]) + (e.Eg[2] + Ee[2]) +
                       (e.Eg[3] + Ee[3]);
    if (!isfinite(sum)) {
      e.eT = INFINITY;
      e.ok = 0;
    }
  }
  e.rho = rho;
  e.Eb = 3.0 * s.p;
#pragma unroll
  for (int i = 0; i < 3; i++) e.ur[i] = s.f * Ut[i];
  e.radflags = s.flags;
  if constexpr (JAC) {
    // lambda's derivative along u_g (4 lambda/u_g, finite at u_g = 0)
    const double lug = 4.0 * ka * ph.arad * (T2 * Tg) * (gm1 * c.iD * u0);
#pragma unroll
    for (int k = 0; k < 4; k++) {
      // gas: A[nu] = dT_nu/dx_k, du_nu, dgamma, d(ln rho)
      double A[4], dul[3] = {0.0, 0.0, 0.0}, dutl = 0.0, dg = 0.0, dlr = 0.0, dlam;
      if (k == 0) {
        const double gu = ph.gam * u0;
        A[0] = gu * utl + gm1;
#pragma unroll
        for (int i = 0; i < 3; i++) A[1 + i] = gu * ul[i];
        dlam = lug;
      } else {
        const int v = k - 1;
#pragma unroll
        for (int i = 0; i < 3; i++) dul[i] = m.lo(k, 1 + i);
        dg = ul[v] * ig;
        const double du0 = M::diagonal ? dg : dg * c.ia;
        dutl = M::diagonal ? -dg : c.beta * dul[0] - al * dg;
        dlr = -iu0 * du0;
        const double dbsq = 2.0 * (bt * c.Bl[v] * (iu0 * iu0) + bsq * dlr);
        const double dwu = dbsq * u0 + wg * du0;
        const double dbl0 = (c.Bl[v] * utl + bt * dutl) * iu0 + bl[0] * dlr;
        A[0] = Dw * dutl + dwu * utl + 0.5 * dbsq - c.Bl[v] * bl[0] - bt * dbl0;
#pragma unroll
        for (int i = 0; i < 3; i++) {
          const double db = (c.Bl[v] * ul[i] + bt * dul[i]) * iu0 + bl[1 + i] * dlr;
          A[1 + i] = dwu * ul[i] + Dw * dul[i] - c.Bl[v] * bl[1 + i] - bt * db;
        }
        dlam = -3.0 * lam * dlr;
      }
      // radiation along dR = -A
      const double dE = M::diagonal ? A[0] : A[0] - c.beta * A[1];
      const double dU = -2.0 * al * dot3(Ut, A + 1);
      const double dp = s.pE * dE + s.pU * dU, dgr = s.gE * dE + s.gU * dU;
      const double df = al * (s.fE * dE + s.fU * dU), fda = s.fd * al;
      double drl[4];
#pragma unroll
      for (int i = 0; i < 3; i++) drl[1 + i] = df * R[1 + i] - fda * A[1 + i];
      drl[0] = M::diagonal ? -dgr : c.beta * drl[1] - al * dgr;
      double dw = dot3(ut, drl + 1) - (g * dgr + dg * s.gr);
      if (k > 0) dw += rl[k];
      const double dc43 = 4.0 * (dp * w + s.p * dw);
      const double dEh = dc43 * w + c43 * dw - dp;
      const double dP1 = kt * (dc43 + c43 * dlr);
      const double dP2 = kt * (dp + s.p * dlr) + dlam + ke * (dEh + Eh * dlr);
      J[0][k] = A[0] + c.dt * (dP1 * rl[0] + P1 * drl[0] + dP2 * utl + P2 * dutl);
#pragma unroll
      for (int i = 0; i < 3; i++)
        J[1 + i][k] = A[1 + i] + c.dt * (dP1 * rl[1 + i] + P1 * drl[1 + i] + dP2 * ul[i] + P2 * dul[i]);
    }
  }
}

// ---------------------------------------------------------------------------
// First PMHD attempt of a cell (Sec. 4.10), as newton<M_PMHD>.
// ---------------------------------------------------------------------------
// LU with partial pivoting; inv[k] = 1/A[k][k] of the factors
DEV bool lu4f(double A[4][4], double inv[4], int& piv) {
  bool ok = true;
  piv = 0;
#pragma unroll
  for (int k = 0; k < 4; k++) {
    int p = k;
    double best = ::fabs(A[k][k]);
#pragma unroll
    for (int i = k + 1; i < 4; i++)
      if (::fabs(A[i][k]) > best) { best = ::fabs(A[i][k]); p = i; }
    ok = ok && best > 0.0 && isfinite(best);
    piv |= p << (2 * k);
#pragma unroll
    for (int i = k + 1; i < 4; i++) {
      const bool sw = i == p;
#pragma unroll
      for (int j = k; j < 4; j++) {
        const double a = A[k][j], b = A[i][j];
        A[k][j] = sw ? b : a;
        A[i][j] = sw ? a : b;
      }
    }
    inv[k] = recip(A[k][k]);
#pragma unroll
    for (int i = k + 1; i < 4; i++) {
      const double f = A[i][k] * inv[k];
#pragma unroll
      for (int j = k + 1; j < 4; j++) A[i][j] -= f * A[k][j];
      A[i][k] = f;
    }
  }
  return ok;
}

// x of A x = b from the factors; false when it is not finite.  The
// multipliers sit in the row positions of their own step, so the swaps run
// along with the elimination.
DEV bool lu_solve4f(const double A[4][4], const double inv[4], int piv, double b[4], double x[4]) {
#pragma unroll
  for (int k = 0; k < 4; k++) {
    const int p = piv >> (2 * k) & 3;
#pragma unroll
    for (int i = k + 1; i < 4; i++) {
      const bool sw = i == p;
      const double t = b[k];
      b[k] = sw ? b[i] : t;
      b[i] = sw ? t : b[i];
    }
#pragma unroll
    for (int i = k + 1; i < 4; i++) b[i] -= A[i][k] * b[k];
  }
#pragma unroll
  for (int i = 3; i >= 0; i--) {
    double s = b[i];
#pragma unroll
    for (int j = i + 1; j < 4; j++) s -= A[i][j] * x[j];
    x[i] = quot(s, A[i][i], inv[i]);
  }
  return isfinite((x[0] + x[1]) + (x[2] + x[3]));
}

// The best iterate of an attempt.
struct PBest {
  double x[4], rho, Eb, ur[3], eT;
  int radflags, ok;
};
DEV void keep(PBest& b, const double x[4], const PEval& e) {
#pragma unroll
  for (int k = 0; k < 4; k++) b.x[k] = x[k];
  b.rho = e.rho;
  b.Eb = e.Eb;
#pragma unroll
  for (int i = 0; i < 3; i++) b.ur[i] = e.ur[i];
  b.eT = e.eT;
  b.radflags = e.radflags;
  b.ok = e.ok;
}

// State of the attempt between trips.
struct PNewton {
  double x[4], Eg[4], eT;
  double A[4][4], inv[4];   // the last Jacobian's factors
  double h[5];              // the last five e_T, h[4] newest
  int piv, lu, it, nrise, extra, conv, iters;
};

// Stopping rules and the Newton step; true when the attempt ends here.
DEV bool pnewton_step(const Opts& o, PNewton& n, double xn[4]) {
  if (n.it >= o.max_iter) return true;
  if (n.eT < o.tol_pmhd) n.conv = 1;
  if (n.conv) {
    if (!o.roundoff || n.extra >= 3) return true;
    n.extra++;
  }
  if (!n.conv && n.it >= 5 && n.eT > 0.5 * (n.h[0] + n.h[1] + n.h[2]) * (1.0 / 3.0)) return true;
  double r[4] = {n.Eg[0], n.Eg[1], n.Eg[2], n.Eg[3]}, dx[4];
  if (!n.lu || !lu_solve4f(n.A, n.inv, n.piv, r, dx)) return true;
#pragma unroll
  for (int i = 0; i < 4; i++) xn[i] = n.x[i] - dx[i];
  if (xn[0] < 0.0) xn[0] = 0.5 * ::fabs(xn[0]);            // one-sided bisection of u_g
  return false;
}

// After the evaluation at xn; true when the attempt ends here.
DEV bool pnewton_take(const double xn[4], const PEval& e, PNewton& n, PBest& b) {
  n.iters++;
  bool small = true;
#pragma unroll
  for (int i = 0; i < 4; i++)
    if (::fabs(xn[i] - n.x[i]) > 10.0 * DBL_EPSILON * ::fabs(n.x[i])) small = false;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    n.x[i] = xn[i];
    n.Eg[i] = e.Eg[i];
  }
  const double prev = n.h[4];
#pragma unroll
  for (int k = 0; k < 4; k++) n.h[k] = n.h[k + 1];
  n.h[4] = n.eT = e.eT;
  if (e.eT < b.eT) keep(b, xn, e);
  if (n.it >= 5 && e.eT > prev && ++n.nrise >= 5) return true;
  n.it++;
  return small;
}

// The attempt.  A wavefront first runs the trips that need a Jacobian until
// no lane does, then the trips on the last factors (chord steps, near the
// root): lanes in different phases would otherwise each pay for both kinds
// of evaluation in every trip.
template <class M>
DEV void pnewton(const PCell<M>& c, const Phys& ph, const Opts& o, const double x0[4], PBest& b,
                 int& iters) {
  PNewton n;
  bool done;
  {
    PEval e;
    pmhd_eval<true>(c, ph, x0, e, n.A);
    keep(b, x0, e);
    done = !e.ok;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      n.x[i] = x0[i];
      n.Eg[i] = e.Eg[i];
      n.h[i] = INFINITY;
    }
    n.h[4] = n.eT = e.eT;
    n.lu = lu4f(n.A, n.inv, n.piv);
    n.it = n.nrise = n.extra = n.conv = n.iters = 0;
  }
  while (!done) {
    while (!done && !(n.eT < GRRMHD_CHORD_TOL)) {
      double xn[4];
      done = pnewton_step(o, n, xn);
      if (!done) {
        PEval e;
        pmhd_eval<true>(c, ph, xn, e, n.A);
        n.lu = lu4f(n.A, n.inv, n.piv);
        done = pnewton_take(xn, e, n, b);
      }
    }
    while (!done && n.eT < GRRMHD_CHORD_TOL) {
      double xn[4];
      done = pnewton_step(o, n, xn);
      if (!done) {
        PEval e;
        pmhd_eval<false>(c, ph, xn, e, n.A);
        done = pnewton_take(xn, e, n, b);
      }
    }
  }
  iters = n.iters;
}

// implicit_fast on the closed forms.
template <class M>
DEV bool implicit_first(const M& m, const Phys& ph, const Opts& o, const double Ui[12],
                        const double Pg[12], double dt, double chi_abs, double chi_es,
                        CellOut& out, Best& bo, int& iters, bool& extreme, int& trips) {
  PCell<M> c;
  pcell_setup(m, Ui, dt, chi_abs, chi_es, c);
  int status = 0;
  {
    // extreme radiation sub-dominance, as prepare()
    double ul[3], rl[3];
    low3(m, Pg + 2, ul);
    low3(m, Pg + 9, rl);
    const double w = dot3(Pg + 2, rl) -
                     root(1.0 + dot3(Pg + 2, ul)) * root(1.0 + dot3(Pg + 9, rl));
    const double Eh = (4.0 / 3.0) * Pg[8] * w * w - Pg[8] * (1.0 / 3.0);
    const double tenEps = 10.0 * DBL_EPSILON;
    extreme = (::fabs(c.Ri[0]) <= tenEps * (::fabs(c.Tgi[0]) + ::fabs(c.Ri[0]))) ||
              (::fabs(Eh) <= tenEps * (::fabs(Pg[1]) + ::fabs(Eh)));
  }
  bo.eT = INFINITY;
  bo.ok = 0;
  iters = 0;
  trips = 0;
  if (extreme) return false;
  double x0[4] = {Pg[1], Pg[2], Pg[3], Pg[4]};
  if (dt * (chi_abs + chi_es) * Pg[0] < 2.0 / 3.0) {
    double rho = Pg[0], ug = Pg[1], ut[3] = {Pg[2], Pg[3], Pg[4]};
    if (mhd_invert(m, ph.gam, c.D, c.Tgi[0], c.Tgi + 1, c.B, rho, ug, ut) == 0) {
      x0[0] = ug; x0[1] = ut[0]; x0[2] = ut[1]; x0[3] = ut[2];
    } else {
      status |= GRRMHD_ST_C2P_FAIL;
    }
  }
  PBest b;
  pnewton(c, ph, o, x0, b, iters);
  trips = iters + 1;
  bo.eT = b.eT;
  bo.ok = b.ok;
  bo.radflags = b.radflags;
  bo.P[0] = b.rho;
  bo.P[8] = b.Eb;
#pragma unroll
  for (int k = 0; k < 4; k++) bo.x[k] = bo.P[1 + k] = b.x[k];
#pragma unroll
  for (int i = 0; i < 3; i++) {
    bo.P[5 + i] = c.B[i];
    bo.P[9 + i] = b.ur[i];
  }
  if (!(b.ok && b.eT < accept_threshold(o))) return false;
  if (b.radflags || !(b.x[0] > 0.0)) {   // a limiter acted: radiation from its primitives
    CellT<M> g;
    cell_setup(m, Ui, dt, chi_abs, chi_es, g);
    finalize(g, ph, o, bo, M_PMHD, status, iters, Ui, out);
    return true;
  }
  status |= GRRMHD_ST_PMHD;
  if (b.eT > o.tol_fail) status |= GRRMHD_ST_FAIL;
  else if (b.eT > o.tol_accept) status |= GRRMHD_ST_NOT_ACCEPT;
  GasState gs;
  gas_state(c, ph.gam, b.x, gs);
#pragma unroll
  for (int q = 0; q < 12; q++) out.P[q] = bo.P[q];
  const double gd = m.gdet;
#pragma unroll
  for (int k = 0; k < 4; k++) {
    out.U[1 + k] = gd * gs.T[k];
    out.U[8 + k] = gd * (c.Ri[k] - (gs.T[k] - c.Tgi[k]));
  }
  out.U[0] = Ui[0];
#pragma unroll
  for (int i = 0; i < 3; i++) out.U[5 + i] = Ui[5 + i];
  out.status = status;
  out.iters = iters;
  out.err = b.eT;
  return true;
}
DEV bool implicit_first(const Metric& m, const Phys& ph, const Opts& o, const double Ui[12],
                        const double Pg[12], double dt, double chi_abs, double chi_es,
                        CellOut& out, Best& b, int& iters, bool& extreme, int& trips) {
  return implicit_fast(m, ph, o, Ui, Pg, dt, chi_abs, chi_es, out, b, iters, extreme, trips);
}

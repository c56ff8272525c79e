// Derivatives of the test-particle map: forward (tangent) and reverse
// (adjoint) mode, by hand, for gfx950.
//
// One step of the map is kick(h) o drift(dt) o kick(h) with h = dt/2.
//  * Kick: v' = v + h a(r), a(r) = h0 - sum_j mu_j d_j/|d_j|^3, d_j = r - r_j.
//    Its Jacobian is [[I, 0], [h A, I]] with the symmetric
//    A = da/dr = sum_j mu_j (3 d_j d_j^T/|d_j|^5 - I/|d_j|^3); h0 and the planet
//    positions do not depend on the particle.
//  * Drift: the f-g Kepler drift (see kepler.hpp).  The change x of eccentric
//    anomaly is an implicit function of (ec, es, dM) through
//    x - ec sin x + es (1 - cos x) = dM, so by the implicit-function theorem
//    dx = (sin x dec - (1 - cos x) des + d dM) / F'(x).  Every other quantity
//    is an explicit expression; they are differentiated in order (tangent) or
//    in reverse order (adjoint).
// The fixed-count Newton iterate x_k stands for the root (its residual is
// below the Kepler-failure threshold), so derivatives are those of the exact
// drift at the computed state.  A particle removed at step n keeps its state,
// so nothing after step n contributes to its derivative.
#pragma once
#include "particle.hpp"

namespace tpm {

// Values of one drift that its derivatives need: r0 = |r|, alpha = 1/a,
// sa = sqrt(alpha), ms = sqrt(mu) sa, ar = a/r0, y = 1/F', m = cos x - 1, and
//   f = 1 + ar m,  g = dte + (s - x)/n,  fdot = -(ms/r0)(s y),  gdot = 1 + y m.
struct DriftVals {
  double u, r0, rinv, alpha, sa, rsa, a, ar, ms, ninv, ec, es, dM, x, s, m, y, f, g, fd, gd;
  bool turns;                // whole periods were taken off dM
};

// The values of the drift whose Kepler root x, with its sine s and cosine minus
// one m, an evaluation of the particles' drift found (drift_lanes).
TPM_DEV DriftVals drift_vals(const KepConst& K, double dt, const double r[3], const double v[3],
                             double x, double s, double m) {
  DriftVals D;
  const double r2 = fma_(r[0], r[0], fma_(r[1], r[1], r[2] * r[2]));
  const double v2 = fma_(v[0], v[0], fma_(v[1], v[1], v[2] * v[2]));
  D.u = fma_(r[0], v[0], fma_(r[1], v[1], r[2] * v[2]));
  sqrt_rsqrt(r2, D.r0, D.rinv);
  D.alpha = fma_(-v2, K.inv_mu, 2.0 * D.rinv);
  sqrt_rsqrt(D.alpha, D.sa, D.rsa);
  D.a = D.rsa * D.rsa;
  D.ms = K.sqrt_mu * D.sa;
  D.ninv = K.inv_sqrt_mu * D.rsa * D.a;
  D.ec = fma_(-D.r0, D.alpha, 1.0);
  D.es = D.u * D.sa * K.inv_sqrt_mu;
  const double M = D.ms * D.alpha * dt;
  const double q = __builtin_rint(M * INV_TWO_PI);
  D.dM = fma_(-q, TWO_PI_LO, fma_(-q, TWO_PI_HI, M));
  D.turns = q != 0.0;
  D.x = x; D.s = s; D.m = m;
  D.y = rcp(fma_(-D.ec, m, fma_(D.es, s, 1.0 - D.ec)));
  D.ar = D.a * D.rinv;
  D.f = fma_(D.ar, m, 1.0);
  D.g = fma_(s - x, D.ninv, D.turns ? D.dM * D.ninv : dt);
  D.fd = -((D.ms * D.rinv) * (s * D.y));
  D.gd = fma_(D.y, m, 1.0);
  return D;
}

TPM_DEV double dot3(const double a[3], const double b[3]) {
  return fma_(a[0], b[0], fma_(a[1], b[1], a[2] * b[2]));
}

// Tangent of the drift: (dr, dv) at (r, v) -> (dr', dv').
TPM_DEV void drift_jvp(const KepConst& K, double dt, const DriftVals& D, const double r[3],
                       const double v[3], const double dr[3], const double dv[3], double odr[3],
                       double odv[3]) {
  const double dr0 = dot3(r, dr) * D.rinv;
  const double drinv = -dr0 * (D.rinv * D.rinv);
  const double dalpha = 2.0 * fma_(-dot3(v, dv), K.inv_mu, drinv);
  const double du = dot3(r, dv) + dot3(v, dr);
  const double dsa = 0.5 * dalpha * D.rsa;
  const double da = -(D.a * D.a) * dalpha;
  const double dms = K.sqrt_mu * dsa;
  const double dn = fma_(dms, D.alpha, D.ms * dalpha);
  const double dninv = -dn * (D.ninv * D.ninv);
  const double dec = -fma_(dr0, D.alpha, D.r0 * dalpha);
  const double des = fma_(du, D.sa, D.u * dsa) * K.inv_sqrt_mu;
  const double ddM = dn * dt;
  const double ddte = D.turns ? fma_(ddM, D.ninv, D.dM * dninv) : 0.0;
  const double dx = fma_(D.s, dec, fma_(D.m, des, ddM)) * D.y;
  const double c = 1.0 + D.m;
  const double ds = c * dx, dm = -D.s * dx;
  const double dFp = fma_(-dec, c, fma_(-D.ec, dm, fma_(des, D.s, D.es * ds)));
  const double dy = -(D.y * D.y) * dFp;
  const double df = fma_(fma_(da, D.rinv, D.a * drinv), D.m, D.ar * dm);
  const double dg = fma_(ds - dx, D.ninv, fma_(D.s - D.x, dninv, ddte));
  const double t1 = D.ms * D.rinv, t2 = D.s * D.y;
  const double dfd = -fma_(fma_(dms, D.rinv, D.ms * drinv), t2, t1 * fma_(ds, D.y, D.s * dy));
  const double dgd = fma_(dy, D.m, D.y * dm);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    odr[k] = fma_(df, r[k], fma_(D.f, dr[k], fma_(dg, v[k], D.g * dv[k])));
    odv[k] = fma_(dfd, r[k], fma_(D.fd, dr[k], fma_(dgd, v[k], D.gd * dv[k])));
  }
}

// Adjoint of the drift: given (lr', lv') = dL/d(r', v'), return dL/d(r, v).
// The expressions of drift_vals are walked backwards (b<name> = dL/d<name>).
TPM_DEV void drift_vjp(const KepConst& K, double dt, const DriftVals& D, const double r[3],
                       const double v[3], const double lr1[3], const double lv1[3], double lr[3],
                       double lv[3]) {
  // r' = f r + g v, v' = fd r + gd v
  const double bf = dot3(lr1, r), bg = dot3(lr1, v), bfd = dot3(lv1, r), bgd = dot3(lv1, v);
  // gd = 1 + y m, f = 1 + ar m, fd = -t1 t2 with t1 = ms rinv, t2 = s y
  const double t1 = D.ms * D.rinv, t2 = D.s * D.y;
  const double bt1 = -bfd * t2, bt2 = -bfd * t1;
  const double bar = bf * D.m;
  double bm = fma_(bgd, D.y, bf * D.ar);
  const double by = fma_(bgd, D.m, bt2 * D.s);
  double bms = bt1 * D.rinv;
  double brinv = fma_(bt1, D.ms, bar * D.a);
  const double ba = bar * D.rinv;
  // g = dte + (s - x) ninv
  double bs = fma_(bt2, D.y, bg * D.ninv);
  double bninv = bg * (D.s - D.x);
  // y = 1/F', F' = 1 - ec c + es s
  const double bFp = -by * (D.y * D.y);
  const double c = 1.0 + D.m;
  bm = fma_(-bFp, D.ec, bm);
  bs = fma_(bFp, D.es, bs);
  // s and m of x, x(ec, es, dM)
  const double bx = fma_(bs, c, fma_(-bm, D.s, -bg * D.ninv)) * D.y;
  const double bec = fma_(bx, D.s, -bFp * c);
  const double bes = fma_(bx, D.m, bFp * D.s);
  double bdM = bx;
  // dte = dM ninv where whole periods were taken off (else dt itself)
  if (D.turns) {
    bdM = fma_(bg, D.ninv, bdM);
    bninv = fma_(bg, D.dM, bninv);
  }
  // dM = n dt (minus a constant), ninv = 1/n, n = ms alpha
  const double bn = fma_(bdM, dt, -bninv * (D.ninv * D.ninv));
  bms = fma_(bn, D.alpha, bms);
  // ms = sqrt(mu) sa, es = u sa/sqrt(mu), ec = 1 - r0 alpha, a = 1/alpha
  const double beu = bes * K.inv_sqrt_mu;
  const double bu = beu * D.sa;
  const double bsa = fma_(beu, D.u, bms * K.sqrt_mu);
  double balpha = fma_(bn, D.ms, fma_(-bec, D.r0, fma_(-ba, D.a * D.a, 0.5 * bsa * D.rsa)));
  // alpha = 2 rinv - v2/mu, rinv = 1/r0, r0 = sqrt(r2)
  brinv = fma_(2.0, balpha, brinv);
  const double bv2 = -2.0 * balpha * K.inv_mu;                  // d/d(v^2/2)
  const double br0 = fma_(-brinv, D.rinv * D.rinv, -bec * D.alpha);
  const double br2 = br0 * D.rinv;                              // d/d(r^2/2)
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    lr[k] = fma_(br2, r[k], fma_(bu, v[k], fma_(D.f, lr1[k], D.fd * lv1[k])));
    lv[k] = fma_(bv2, v[k], fma_(bu, r[k], fma_(D.g, lr1[k], D.gd * lv1[k])));
  }
}

// A w with A = da/dr at position r for one table row (symmetric, so it also
// serves the adjoint): sum_j k_j (3 (d_j.w)/|d_j|^2 d_j - w), k_j = mu_j/|d_j|^3,
// with k_j and 1/|d_j|^2 from one reciprocal square root and its residual.
template <int NP, typename RowT>
TPM_DEV void accel_jac(const RowT& row, const PlanetConst<NP>& P, const double r[3],
                       const double w[3], double out[3]) {
  out[0] = out[1] = out[2] = 0.0;
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    const double d[3] = {r[0] - row[3 * j + 0], r[1] - row[3 * j + 1], r[2] - row[3 * j + 2]};
    const double d2 = dot3(d, d);
    const double y = __builtin_amdgcn_rsq(d2);
    const double y2 = y * y;
    const double e = fma_(-d2, y2, 1.0);
    const double mm = P.mu[j] * (y2 * y);
    const double k = fma_(mm * e, fma_(e, 1.875, 1.5), mm);
    const double inv2 = fma_(y2, fma_(e, e, e), y2);
    const double c = 3.0 * k * (inv2 * dot3(d, w));
#pragma unroll
    for (int q = 0; q < 3; ++q) out[q] = fma_(c, d[q], fma_(-k, w[q], out[q]));
  }
}

}  // namespace tpm

// Kepler drift with the f and g functions (Zhang & Gladman 2021, sec. 2.2,
// drift step and the difference form of Kepler's equation), FP64, gfx950.
//
// With r0 = |r|, u = r.v and alpha = 2/r0 - v^2/mu = 1/a, the mean motion is
// n = sqrt(mu alpha) alpha, ec = 1 - r0 alpha = e cos E0 and
// es = u sqrt(alpha/mu) = e sin E0.  The change x of eccentric anomaly over a
// step dt solves F(x) = x - ec sin x + es (1 - cos x) - n dt = 0, and
//   f = 1 + (a/r0)(cos x - 1),      g = dt + (sin x - x)/n,
//   fdot = -a^2 n sin x / (r1 r0),  gdot = 1 + (a/r1)(cos x - 1),
// with r1 = a F'(x), give r' = f r + g v and v' = fdot r + gdot v.
//
// Particle version (drift_fixed): at most k Newton steps from a fixed
// starting guess (sec. 2.2: a fixed iteration count, since the slowest lane of
// a group sets the group's time).  A lane stops early only once its iterate
// has converged to rounding (kepler_newton), so the result is the k-step
// result up to an ulp or two, and the wavefront leaves the loop when every
// lane has stopped.  The starter is the third-order series root of F = 0 in
// t = dM/(1-ec) (kepler_starter), clamped to dM +- 2(|ec|+|es|) (a bracket of
// the root).  The drift is refused (returns false) when the orbit is unbound
// or |F(x_k)| > ftol; mean anomaly steps beyond pi are reduced by whole
// periods.
#pragma once
#include "dmath.hpp"
#include "internal.h"
#include "universal.hpp"

namespace tpm {

constexpr double TWO_PI_HI = 0x1.921fb54442d18p+2;
constexpr double TWO_PI_LO = 0x1.1a62633145c07p-52;
constexpr double INV_TWO_PI = 0x1.45f306dc9c883p-3;


// sin and cos - 1 of an iterate; SHORT when every argument of the solve is
// known to lie within +-0.78 (see short_args), so the pi/2 reduction is
// skipped (the values are those of the full path up to the polynomial's
// evaluation order); otherwise each call checks by itself.  Only the planet
// map takes the SHORT form, evaluated by Horner's rule (see
// sincos_poly_horner).  The solve and the f and g functions use cos x - 1
// (m below) rather than cos x: F = x - ec sin x - es m - dM,
// F' = (1 - ec) - ec m + es sin x, f = 1 + (a/r0) m, gdot = 1 + (a/r1) m, all
// free of the cancellation 1 - cos x would bring for small x.
template <bool SHORT>
TPM_DEV void sincos_it(double x, double& s, double& m) {
  if (SHORT) sincos_poly_horner(x, s, m);
  else sincosm1(x, s, m);
}

// A lane's starter (clamped to dM +- w, w = 2(|ec| + |es|)), root and Newton
// iterates stay within 0.66 of zero when |dM| <= 0.45 and w <= 0.2: then
// e <= 0.1, the root lies within 2e of dM, F' >= 1 - e and |F''| <= e, so one
// Newton step from the starter (at most 0.4 from the root) lands within 0.01
// of the root and later steps closer still.
TPM_DEV bool short_args(double dM, double w) {
  return __builtin_fabs(dM) <= 0.45 && w <= 0.2;
}

// Newton steps on F(x) = x - ec sin x + es (1 - cos x) - dM from xk.  With
// e <= |ec| + |es| = eb, |F''| <= e and 1 - e <= F' <= 1 + e, so a step
// x -> x - d, whose d = F(x)/F'(x) is at least (1-e)/(1+e) times the error of
// x, leaves an error of at most Q d^2 with
//   Q = eb (1 + eb)^2 / (2 (1 - eb)^3)      (kepler_bound; +inf for eb > 0.75).
// A lane stops after the first step with Q d^2 <= 2^-54 |x - d| and
// |d| <= 2^-28 (a quarter ulp at most is left), or with |d| <= 2^-30 |x - d|
// (the error then is below e/(2(1-e)) (2^-30 |x|)^2, under one ulp for
// e <= 0.99, |x| <= 4).  The stop is each lane's own decision, so the result of
// a particle does not depend on which particles share its wavefront; the
// wavefront leaves the loop once all its lanes have stopped.  Lanes with a
// NaN state (unbound orbits) never stop; lanes that start with done set take
// no part.
//
// The method's fixed count kiters decides failure: Fk receives F(x_k) of a
// lane still iterating after kiters steps (0 for a lane that stopped before;
// the drift is refused where |Fk| > ftol).  Such a lane's state is taken from
// up to KEPLER_EXTRA further steps: a lane that passes the failure rule has
// |x_k - root| <= |F(x_k)|/(1-e), inside Newton's quadratic range, so two
// steps bring it to rounding (at e = 0.9999, 1e-9 -> 5e-15 -> 1e-25).  The
// state is then the root, as the converged reference has it, rather than x_k,
// whose phase may be off by up to ftol/(1-e) per drift.
//
// Returns the root and, in (s, m), its sine and cosine minus one.  A lane's
// (s, m) are fixed in the step where it stops, like its root: from the values
// at the point x of that step (c = 1 + m) and the step's correction d (the
// root is x - d), the first-order rotation
//   sin(x - d) = s - c d,  cos(x - d) - 1 = m + s d
// leaves out s d^2/2 and c d^3/6 (and their cosine counterparts): with
// |d| <= 2^-28 and Q >= 2^-24 (kepler_bound's floor) these stay below 0.05 ulp
// of the values and of x.  Lanes still iterating when the step budget runs
// out get sin/cos of their last iterate afresh; lanes that start with done
// set get (0, 0) (their xk is 0).  Each lane's values depend only on its own
// iterates, whichever lanes share its wavefront.  om = 1 - ec.
constexpr int KEPLER_EXTRA = 2;

template <bool SHORT>
TPM_DEV double kepler_newton(double ec, double es, double om, double dM, int kiters, double Q,
                             bool done, double xk, double& s, double& m, double& Fk) {
  bool converged = false;   // wave-uniform: every lane stopped
  s = 0.0;
  m = 0.0;
  Fk = 0.0;
  for (int it = 0; it < kiters + KEPLER_EXTRA; ++it) {
    if (it >= 1 && wave_all(done)) {
      converged = true;
      break;
    }
    double sv, mv;
    sincos_it<SHORT>(xk, sv, mv);
    double F = fma_(-ec, sv, fma_(-es, mv, xk - dM));
    if (it == kiters) Fk = done ? 0.0 : F;
    double Fp = fma_(-ec, mv, fma_(es, sv, om));
    double xn = fma_(-F, rcp_newton(Fp), xk);
    const double d = xk - xn;
    const double ad = __builtin_fabs(d), ax = __builtin_fabs(xn);
    bool small = (ad <= 0x1p-30 * ax) |
                 ((ad <= 0x1p-28) & (fma_(Q * ad, ad, -0x1p-54 * ax) <= 0.0));
    const double sn = fma_(-(1.0 + mv), d, sv), mn = fma_(sv, d, mv);
    s = done ? s : sn;
    m = done ? m : mn;
    xk = done ? xk : xn;
    done = done | small;
  }
  if (!converged) {
    double sf, mf;
    sincos_it<SHORT>(xk, sf, mf);
    s = done ? s : sf;
    m = done ? m : mf;
  }
  return xk;
}

// Newton for the planet map: as kepler_newton, but no lane freezes.  The
// planet map's wavefront always holds the same bodies in the same lanes, so
// its results cannot depend on which lanes share it.  Every lane iterates
// until the last step of each non-idle lane was a correction of at most
// 2^-30 |x|, and its sin/cos come from that last step's rotation (as in
// kepler_newton); at most 40 steps, after which sin/cos are evaluated afresh.
// Idle lanes (dM = 0, x = 0) stay at x = 0.  Lanes beyond the bodies may
// carry NaN (their central-body term sits at zero distance), so idle lanes
// enter every wave-wide test through their idle flag.
template <bool SHORT>
TPM_DEV double planet_newton(double ec, double es, double om, double dM, bool idle, double xk,
                             double& s, double& m) {
  bool done = idle;
  for (int it = 0; it < 40; ++it) {
    if (it >= 2 && wave_all(done)) return xk;
    double sv, mv;
    sincos_it<SHORT>(xk, sv, mv);
    const double F = fma_(-ec, sv, fma_(-es, mv, xk - dM));
    const double Fp = fma_(-ec, mv, fma_(es, sv, om));
    const double xn = fma_(-F, rcp_newton(Fp), xk);
    const double d = xk - xn;
    done = idle | (__builtin_fabs(d) <= 0x1p-30 * __builtin_fabs(xn));
    s = fma_(-(1.0 + mv), d, sv);
    m = fma_(sv, d, mv);
    xk = xn;
  }
  sincos_it<SHORT>(xk, s, m);
  return xk;
}

// Starter of the particles' Newton solve: with p = 1 - ec and t = dM/p, the
// series root of F = 0 through third order in t,
//   x0 = t - (es/(2p)) t^2 + (es^2/(2p^2) - ec/(6p)) t^3
// (F = p x + (es/2) x^2 + (ec/6) x^3 - dM + O(x^4)), clamped to dM +- w,
// w = 2(|ec| + |es|) (a bracket of the root).  Its error is O(e t^4): on
// near-circular orbits one Newton step from it is converged to rounding.
TPM_DEV double kepler_starter(double ec, double es, double om, double dM, double w) {
  const double oinv = rcp_newton(om);   // a first guess only (om = 1 - ec)
  const double t = dM * oinv;
  const double h = 0.5 * es * oinv;
  const double c3 = oinv * fma_(es, h, ec * (-1.0 / 6.0));
  const double x0 = t * fma_(t, fma_(c3, t, -h), 1.0);
  return __builtin_fmin(__builtin_fmax(x0, dM - w), dM + w);
}

// Q of kepler_newton's stopping rule from w = 2(|ec| + |es|): rounded up (the
// hardware reciprocal is good to 2^-24) and at least 2^-24; +inf where
// eb = w/2 > 0.75 (or NaN), which leaves those lanes the relative rule alone.
TPM_DEV double kepler_bound(double w) {
  const double eb = 0.5 * w;
  const double om = 1.0 - eb, op = 1.0 + eb;
  const double Q = (0.5 + 0x1p-20) * eb * (op * op) * __builtin_amdgcn_rcp(om * om * om);
  return eb <= 0.75 ? __builtin_fmax(Q, 0x1p-24) : __builtin_inf();
}

// The particles' Newton solve from the starter xk, with sin/cos of its result
// and F(x_k) of the fixed count (see kepler_newton).  (Each sin/cos decides its
// short path by itself: one copy of the loop keeps the particle kernel's
// registers within budget.)
TPM_DEV double kepler_solve(double ec, double es, double om, double dM, int kiters, double w,
                            double xk, double& s, double& m, double& Fk) {
  return kepler_newton<false>(ec, es, om, dM, kiters, kepler_bound(w), false, xk, s, m, Fk);
}

// Drift (x, v) by dt about mass mu with k fixed Newton iterations.  Writes the
// drifted state into (x, v) on every lane; where the return value is false
// (the drift is refused) that state is meaningless and the caller keeps its
// own copy of the old one.
// (xk, s, m) receive the root, its sine and its cosine minus one.
TPM_DEV bool drift_fixed(const KepConst& K, double dt, int kiters, double ftol,
                         double& x, double& y, double& z,
                         double& vx, double& vy, double& vz, double& xk, double& s, double& m) {
  double r2 = fma_(x, x, fma_(y, y, z * z));
  double v2 = fma_(vx, vx, fma_(vy, vy, vz * vz));
  double u = fma_(x, vx, fma_(y, vy, z * vz));
  double r0, rinv;
  sqrt_rsqrt(r2, r0, rinv);
  double alpha = fma_(-v2, K.inv_mu, 2.0 * rinv);
  bool bound = alpha > 0.0;
  double sa, rsa;
  sqrt_rsqrt(alpha, sa, rsa);            // NaN for unbound lanes, never selected
  double a = rsa * rsa;                  // 1/alpha
  a = fma_(a, fma_(-alpha, a, 1.0), a);  // one correction to ~1 ulp
  double n = K.sqrt_mu * sa * alpha;
  double ninv = K.inv_sqrt_mu * rsa * a; // 1/n
  double ec = fma_(-r0, alpha, 1.0);
  double es = u * sa * K.inv_sqrt_mu;
  double dM = n * dt;
  // reduce dM to (-pi, pi]; keep dt itself when no whole period is removed
  double q = __builtin_rint(dM * INV_TWO_PI);
  double dMr = fma_(-q, TWO_PI_HI, dM);
  dMr = fma_(-q, TWO_PI_LO, dMr);
  double dte = (q == 0.0) ? dt : dMr * ninv;
  dM = dMr;
  const double w = 2.0 * (__builtin_fabs(ec) + __builtin_fabs(es));
  const double om = 1.0 - ec;
  xk = kepler_starter(ec, es, om, dM, w);
  double Fk;
  xk = kepler_solve(ec, es, om, dM, kiters, w, xk, s, m, Fk);
  double F = fma_(-ec, s, fma_(-es, m, xk - dM));
  double Fp = fma_(-ec, m, fma_(es, s, om));
  // one compare: an unbound orbit counts as an infinite residual; the larger
  // of the fixed count's residual and the final one decides
  const double Fm = __builtin_fmax(__builtin_fabs(F), __builtin_fabs(Fk));
  const bool ok = (bound ? Fm : __builtin_inf()) <= ftol;
  double r1 = a * Fp;
  double r1inv = rcp(r1);
  double f = fma_(a * rinv, m, 1.0);
  double g = fma_(s - xk, ninv, dte);
  double fd = -(a * a) * n * s * rinv * r1inv;
  double gd = fma_(a * r1inv, m, 1.0);
  double nx = fma_(f, x, g * vx), ny = fma_(f, y, g * vy), nz = fma_(f, z, g * vz);
  double nvx = fma_(fd, x, gd * vx), nvy = fma_(fd, y, gd * vy), nvz = fma_(fd, z, gd * vz);
  x = nx; y = ny; z = nz;
  vx = nvx; vy = nvy; vz = nvz;
  return ok;
}

// The short drift: the particle drift where the arc and the eccentricity are
// moderate, |t| = |dM|/(1 - ec) <= 1/4 and eb = |ec| + |es| <= 3/4, in the
// fewest instructions (a particle step is bound by their number).
//  * No whole periods to remove and no bracket for the starter.  The failure
//    rule of five Newton steps from the third-order starter always holds in
//    these ranges (|F(x_5)| stays below 6e-17 over two million draws of them), so
//    for thresholds from 1e-14 up it needs no evaluation.
//  * 1/(1 - ec) = a/r0 is at hand, and the starter goes one order further
//    (c4 = h (5 (h^2 - c3) + 1/12) by reversion of the series): one Newton step
//    then is converged for arcs up to a hundredth of an orbit at
//    eccentricities up to 0.5, where the third-order one left 2% of the lanes,
//    and with them seven wavefronts in ten, to a second step.
//  * |x| <= 0.3 leaves the last terms of the sine and cosine series below
//    2^-55 of the sum.  sin x - x enters g as summed, not as a difference.
//  * |r| and sqrt(alpha) are one product each, without the correction of
//    sqrt_rsqrt: an error of theirs meets the result through the arc x, or, |r| in
//    1 - ec = |r| alpha, shifts the orbit by as much as a rounding of r would.
//    (1 - ec must come from the same alpha: from v^2 directly the velocities
//    lose a tenth to a fifth at arcs of 0.1 to 0.25.)  |r|^2 is the step before's.
//  * gdot = 1 + m/F', fdot = -(n a)(sin x / r0)/F' and n a = sqrt(mu alpha), all
//    without r1; 1/F' at the root continues the step's reciprocal (F' has moved
//    by less than 2^-26).
// A Newton step from x to x - d leaves an error of |F''| d^2 / (2 F'(x)) where d
// is so small that F' hardly changes, and |F''| <= eb: a lane is `fine` with
// |d| <= 2^-28 and eb d^2 / F'(x) <= 2^-54 |x - d|, half of which is left at
// most.  The few lanes in the ranges that are not after one step take a second
// one, and a lane still not fine (or out of the ranges, or unbound: NaN) is left
// to drift_wide and drift_fixed.  All of it is the lane's own decision; the branches only skip
// what no lane of act needs.  Lane predicates are kept as lane masks: as
// booleans the compiler carries them through vector registers.
// With it a lone wavefront's step of four planets takes about 0.52 us (0.78 with
// drift_fixed; the planet map 0.49); 10,000 steps of 13,313 particles 5.3 ms
// (9.5 with drift_fixed and the map of then), of 200,000 15.0 (22.1).  Rounding
// errors of one drift are no larger than drift_fixed's (rms 5.7e-17 in position;
// in velocity 7.4e-17 to 8.6e-17 against 7.4e-17 to 8.7e-17).
constexpr double QUICK_FTOL = 1e-14;   // smallest failure threshold it may serve

// sin x - x and cos x - 1 for |x| <= 0.31.
TPM_DEV void sinm_short(double x, double& sx, double& m) {
  const double z = x * x;
  const double z2 = z * z;
  const double z4 = z2 * z2;
  const double s01 = fma_(S5, z, S3), s23 = fma_(S9, z, S7), s45 = fma_(S13, z, S11);
  sx = (x * z) * fma_(z4, s45, fma_(z2, s23, s01));
  const double c01 = fma_(C6, z, C4), c23 = fma_(C10, z, C8);
  m = fma_(z2, fma_(z4, C12, fma_(z2, c23, c01)), -0.5 * z);
}

// r2: |r|^2.  Returns the fine lanes; the others' states mean nothing.
TPM_DEV uint64_t drift_quick(const KepConst& K, double dt, uint64_t act, double r2, double& x,
                             double& y, double& z, double& vx, double& vy, double& vz, double& xk,
                             double& s, double& m) {
  const double v2 = fma_(vx, vx, fma_(vy, vy, vz * vz));
  const double u = fma_(x, vx, fma_(y, vy, z * vz));
  const double rinv = rsqrt(r2), r0 = r2 * rinv;
  const double alpha = fma_(-v2, K.inv_mu, 2.0 * rinv);
  const double rsa = rsqrt(alpha), sa = alpha * rsa;   // NaN for unbound lanes: not fine
  const double a = rsa * rsa;             // meets cos x - 1 and sin x - x only
  const double ms = K.sqrt_mu * sa;       // n a
  const double dM = ms * alpha * dt;
  const double ninv = K.inv_sqrt_mu * rsa * a;
  const double ec = fma_(-r0, alpha, 1.0);
  const double es = u * sa * K.inv_sqrt_mu;
  const double eb = __builtin_fabs(ec) + __builtin_fabs(es);
  const double om = 1.0 - ec;
  const double ar = a * rinv;             // 1/om
  const double t = dM * ar;
  const double h = (0.5 * es) * ar;
  const double c3 = ar * fma_(es, h, ec * (-1.0 / 6.0));
  const double c4 = h * fma_(5.0, fma_(h, h, -c3), 1.0 / 12.0);
  xk = t * fma_(t, fma_(t, fma_(t, c4, c3), -h), 1.0);
  const uint64_t range = lanes(__builtin_fabs(t) <= 0.25) & lanes(eb <= 0.75);
  double iFp, smx;                        // smx: sin x - x
  auto newton = [&](double x0, double& xn, double& sxn, double& mn, double& yn) {
    double sx, mv;
    sinm_short(x0, sx, mv);
    const double sv = x0 + sx;
    const double F = fma_(-ec, sv, fma_(-es, mv, x0 - dM));
    yn = rcp_newton(fma_(-ec, mv, fma_(es, sv, om)));
    xn = fma_(-F, yn, x0);
    const double d = x0 - xn;
    sxn = fma_(-mv, d, sx);
    mn = fma_(sv, d, mv);
    const double ad = __builtin_fabs(d);
    return range & lanes(ad <= 0x1p-28) &
           lanes(eb * yn * (ad * ad) <= 0x1p-54 * __builtin_fabs(xn));
  };
  uint64_t fine = newton(xk, xk, smx, m, iFp);
  if (act & range & ~fine) {
    double xn, sxn, mn, yn;
    const uint64_t f2 = newton(xk, xn, sxn, mn, yn);
    // (lanes out of the ranges keep their first iterate, whoever shares the
    // wavefront: drift_wide goes on from it)
    const bool mine = lane_in(fine | ~range);
    xk = mine ? xk : xn;
    smx = mine ? smx : sxn;
    m = mine ? m : mn;
    iFp = mine ? iFp : yn;
    fine |= f2;
  }
  s = xk + smx;
  {
    const double e = fma_(-fma_(-ec, m, fma_(es, s, om)), iFp, 1.0);
    iFp = fma_(iFp, fma_(e, e, e), iFp);
  }
  const double f = fma_(ar, m, 1.0);
  const double g = fma_(smx, ninv, dt);
  const double fd = -((ms * rinv) * (s * iFp));
  const double gd = fma_(iFp, m, 1.0);
  const double nx = fma_(f, x, g * vx), ny = fma_(f, y, g * vy), nz = fma_(f, z, g * vz);
  vx = fma_(fd, x, gd * vx); vy = fma_(fd, y, gd * vy); vz = fma_(fd, z, gd * vz);
  x = nx; y = ny; z = nz;
  return fine;
}

// The wide drift: a converged solve where drift_quick does not serve but the
// fixed-count solve cannot refuse either, t^2 <= (1 - e^2) max(1, 4 (1 - e^2)) with
// t = dM/(1 - ec) as in drift_quick (arcs up to two radians on circular orbits, half a
// radian at e = 0.87, 0.14 at e = 0.99).  There F after five Newton steps from the
// third-order starter is at rounding, below 7e-16 over twenty million draws up to
// the edge (the first refusals come with t 1.2 times larger, at e = 0.94), so
// thresholds from QUICK_FTOL up need no evaluation, and |dM| < 2.4 has no whole
// period.  drift_quick has left an iterate xk (its start and one Newton step); full-range
// Newton steps go on from there, with drift_quick's stopping rule: one to three at
// moderate arcs, where the fixed-count solve takes three to five and its
// bookkeeping; four at the most, and a lane that has not stopped by then is left to
// that solve.  The elements are drift_fixed's, to rounding (at these arcs the
// shortcuts of drift_quick would show), f, g, fdot and gdot drift_quick's forms.
// `low`: the lanes of small eccentricity (e^2 <= 0.28).
// Without it every lane out of drift_quick's ranges costs its wavefront that
// attempt and the fixed-count solve: 2,000 steps of 64 particles at 15 steps an
// orbit, planets from a table, 2.46 ms (1.94 with the fixed-count solve alone), with
// it 1.76; of 100,000 particles at e = 0.6 to 0.9, 60 steps an orbit, 4.9 (4.4) and 4.2.
// Where the lanes of a wavefront lie on both sides of its edge, both solves run: 250
// steps of 4,096 particles at e = 0.5 to 0.9999 0.82 ms, 0.80 without it.
TPM_DEV uint64_t drift_wide(const KepConst& K, double dt, uint64_t act, double r2, double& x,
                            double& y, double& z, double& vx, double& vy, double& vz, double& xk,
                            double& s, double& m, uint64_t& low) {
  const double v2 = fma_(vx, vx, fma_(vy, vy, vz * vz));
  const double u = fma_(x, vx, fma_(y, vy, z * vz));
  double r0, rinv, sa, rsa;
  sqrt_rsqrt(r2, r0, rinv);
  const double alpha = fma_(-v2, K.inv_mu, 2.0 * rinv);
  sqrt_rsqrt(alpha, sa, rsa);             // NaN for unbound lanes: not served
  double a = rsa * rsa;
  a = fma_(a, fma_(-alpha, a, 1.0), a);
  const double ms = K.sqrt_mu * sa;       // n a
  const double dM = ms * alpha * dt;
  const double ninv = K.inv_sqrt_mu * rsa * a;
  const double ec = fma_(-r0, alpha, 1.0);
  const double es = u * sa * K.inv_sqrt_mu;
  const double eb = __builtin_fabs(ec) + __builtin_fabs(es);
  const double om = 1.0 - ec;
  const double ar = a * rinv;             // 1/om
  const double t = dM * ar;
  const double q = fma_(-es, es, fma_(-ec, ec, 1.0));   // 1 - e^2
  low = lanes(q >= 0.72);
  const uint64_t wide = act & lanes(t * t <= q * __builtin_fmax(1.0, 4.0 * q));
  if (wide == 0) return 0;
  uint64_t todo = wide;
  double iFp = 0.0;
  for (int it = 0; it < 4; ++it) {
    double sv, cv, mv;
    if (todo & ~lanes(__builtin_fabs(xk) <= 0.78)) sincos3_reduced(xk, sv, cv, mv);
    else sincos_poly(xk, sv, mv);
    const double F = fma_(-ec, sv, fma_(-es, mv, xk - dM));
    const double yn = rcp_newton(fma_(-ec, mv, fma_(es, sv, om)));
    const double xn = fma_(-F, yn, xk);
    const double d = xk - xn;
    const double ad = __builtin_fabs(d);
    const bool go = lane_in(todo);
    xk = go ? xn : xk;
    s = go ? fma_(-(1.0 + mv), d, sv) : s;
    m = go ? fma_(sv, d, mv) : m;
    iFp = go ? yn : iFp;
    todo &= ~(lanes(ad <= 0x1p-28) &
              lanes(eb * yn * (ad * ad) <= 0x1p-54 * __builtin_fabs(xn)));
    if (todo == 0) break;
  }
  {
    const double e = fma_(-fma_(-ec, m, fma_(es, s, om)), iFp, 1.0);
    iFp = fma_(iFp, fma_(e, e, e), iFp);
  }
  const double f = fma_(ar, m, 1.0);
  const double g = fma_(s - xk, ninv, dt);
  const double fd = -((ms * rinv) * (s * iFp));
  const double gd = fma_(iFp, m, 1.0);
  const double nx = fma_(f, x, g * vx), ny = fma_(f, y, g * vy), nz = fma_(f, z, g * vz);
  vx = fma_(fd, x, gd * vx); vy = fma_(fd, y, gd * vy); vz = fma_(fd, z, gd * vz);
  x = nx; y = ny; z = nz;
  return wide & ~todo;
}

// The particles' drift of the lanes of act: where `quick` is set, drift_quick where
// it serves, then drift_wide where that does, and with `univ` (a refused drift is
// then taken in universal variables, so whether the fixed-count solve refuses does
// not matter) drift_universal_quick where that serves, but for orbits of small
// eccentricity, which are left by their arcs alone (long ones, that it does not
// reach: at six steps an orbit its attempt took half the time of a step);
// drift_fixed elsewhere, and with univ drift_universal where it refuses.  Returns
// the lanes of act whose drift is refused in the end (their state, and that of
// lanes outside act, means nothing).
__host__ TPM_DEV bool quick_serves(int kiters, double ftol) {
  return kiters == 5 && ftol >= QUICK_FTOL;
}

TPM_DEV uint64_t drift_lanes(const KepConst& K, double dt, int kiters, double ftol, bool quick,
                             bool univ, uint64_t act, double r2, double& x, double& y, double& z,
                             double& vx, double& vy, double& vz, double& xk, double& s,
                             double& m) {
  const double ox = x, oy = y, oz = z, ux = vx, uy = vy, uz = vz;
  uint64_t rest = act, low = 0;
  if (quick) rest = act & ~drift_quick(K, dt, act, r2, x, y, z, vx, vy, vz, xk, s, m);
  // (said to be likely, so that what follows lies behind the step loop and not within it:
  // within it the loop of a step was ten times its length, and runs that drift_quick
  // serves took 2 to 10% longer, a fifth longer with univ; 0.6 to 0.9999 are alike but
  // for 4,096 particles at e above 0.5, 2 to 3% longer at 0.9999 than at 0.9)
  if (__builtin_expect_with_probability(rest == 0, 1, 0.9)) return 0;
  // (drift_wide behind drift_quick rather than in it: values that may come from either,
  // carried through one common end, made its own lanes' step 20% longer)
  if (quick) {
    double px = ox, py = oy, pz = oz, qx = ux, qy = uy, qz = uz;
    double wk = xk, ws = 0.0, wm = 0.0;
    const uint64_t wide = drift_wide(K, dt, rest, r2, px, py, pz, qx, qy, qz, wk, ws, wm, low);
    if (lane_in(wide)) {
      x = px; y = py; z = pz;
      vx = qx; vy = qy; vz = qz;
      xk = wk; s = ws; m = wm;
    }
    rest &= ~wide;
    if (rest == 0) return 0;
  }
  if (quick && univ && (rest & ~low)) {
    double px = ox, py = oy, pz = oz, qx = ux, qy = uy, qz = uz;
    const uint64_t served = drift_universal_quick(K, dt, rest & ~low, px, py, pz, qx, qy, qz);
    if (lane_in(served)) {
      x = px; y = py; z = pz;
      vx = qx; vy = qy; vz = qz;
    }
    rest &= ~served;
    if (rest == 0) return 0;
  }
  bool ok = true;
  if (lane_in(rest)) {
    x = ox; y = oy; z = oz;
    vx = ux; vy = uy; vz = uz;
    ok = drift_fixed(K, dt, kiters, ftol, x, y, z, vx, vy, vz, xk, s, m);
    if (!ok && univ) {
      x = ox; y = oy; z = oz;
      vx = ux; vy = uy; vz = uz;
      ok = drift_universal(K.mu, dt, x, y, z, vx, vy, vz);
    }
  }
  return lanes(!ok);
}

// The same from the state alone.
TPM_DEV uint64_t drift_lanes(const KepConst& K, double dt, int kiters, double ftol, bool quick,
                             bool univ, uint64_t act, double& x, double& y, double& z, double& vx,
                             double& vy, double& vz, double& xk, double& s, double& m) {
  return drift_lanes(K, dt, kiters, ftol, quick, univ, act, fma_(x, x, fma_(y, y, z * z)), x, y, z,
                     vx, vy, vz, xk, s, m);
}

// f, g, fdot and gdot of a planet's converged Kepler drift from r^2, v^2 and
// r.v (a handful of lanes in one wavefront): Newton until every lane has made a
// step whose correction is at most 2^-30 |x| (converged to rounding;
// planet_newton), at most 40 steps.  A lane that holds no body, or whose body
// is found unbound (the return value is then false), drifts for no time on a
// stand-in bound orbit (alpha = 1): dM = 0, x = 0, f = gdot = 1 and
// g = fdot = 0 exactly, so its state is left as it was without any select on
// the result.
TPM_DEV bool planet_fg(const KepConst& K, double dt, bool lane_on, double r2, double v2, double u,
                       double& f, double& g, double& fd, double& gd) {
  double r0, rinv;
  sqrt_rsqrt(lane_on ? r2 : 1.0, r0, rinv);
  double alpha = fma_(-v2, K.inv_mu, 2.0 * rinv);
  const bool bound = alpha > 0.0;
  const bool idle = !(lane_on && bound);
  alpha = idle ? 1.0 : alpha;
  dt = idle ? 0.0 : dt;
  double sa, rsa;
  sqrt_rsqrt(alpha, sa, rsa);
  double a = rsa * rsa;
  a = fma_(a, fma_(-alpha, a, 1.0), a);
  double n = K.sqrt_mu * sa * alpha;
  double ninv = K.inv_sqrt_mu * rsa * a;
  double ec = fma_(-r0, alpha, 1.0);
  double es = u * sa * K.inv_sqrt_mu;
  double dM = n * dt;
  double q = __builtin_rint(dM * INV_TWO_PI);
  double dMr = fma_(-q, TWO_PI_HI, dM);
  dMr = fma_(-q, TWO_PI_LO, dMr);
  double dte = (q == 0.0) ? dt : dMr * ninv;
  dM = dMr;
  const double om = 1.0 - ec;
  double oinv = rcp_newton(om);   // a first guess only: one refinement is enough
  double t = dM * oinv;
  double xk = t * fma_(-0.5 * es * t, oinv, 1.0);
  double w = 2.0 * (__builtin_fabs(ec) + __builtin_fabs(es));
  xk = __builtin_fmin(__builtin_fmax(xk, dM - w), dM + w);
  double s, m;
  if (wave_all(idle | short_args(dM, w)))
    xk = planet_newton<true>(ec, es, om, dM, idle, xk, s, m);
  else
    xk = planet_newton<false>(ec, es, om, dM, idle, xk, s, m);
  double Fp = fma_(-ec, m, fma_(es, s, om));
  double r1 = a * Fp;
  double r1inv = rcp(r1);
  f = fma_(a * rinv, m, 1.0);
  g = fma_(s - xk, ninv, dte);
  fd = -(a * a) * n * s * rinv * r1inv;
  gd = fma_(a * r1inv, m, 1.0);
  return bound;
}

// f, g, fdot and gdot of a planet's drift in the fewest instructions (the planet
// map's lone wavefront is bound by their number), for arcs up to three quarters
// of a radian and eccentricities up to 0.4: one step of fourth order from the
// third-order series start (see drift_quick, whose quantities these are), and
// the sine and cosine carried over to the root by the rotation, where a second
// Newton step would evaluate them again.  With y = 1/F', u = F y, A = F'' y/2 and
// B = (y - 1)/6 (the third derivative is 1 - F') the step is -u (1 + u (A + u (2 A^2 -
// B))), the inverse series of F.  What it leaves is at most eb y d^4 (the next
// term, 5 A^3 - 5 A B + y/24 of the fourth derivative, is below 0.6 eb y for eb <= 0.4): a lane is
// served where that is below 2^-54 |x| and |d| <= 2^-14, from where on the
// rotation's first term left out, d^4/24, would show.  sin x - x is summed from
// small terms and enters g as such, where sin x minus x would bring in half
// an ulp of x.  Where it is not
// served (or out of the ranges, or unbound: NaN) planet_fg takes the lane; the
// choice is the lane's own, so it does not depend on the map's blocks.  A lane
// without a body holds a stand-in (r^2 = v^2 = mu = 1, u = 0, dt = 0), which
// comes out as f = gdot = 1, g = fdot = 0.
TPM_DEV bool planet_quick(const KepConst& K, double dt, double r2, double v2, double u, double& f,
                          double& g, double& fd, double& gd) {
  const double rinv = rsqrt(r2), r0 = r2 * rinv;
  const double alpha = fma_(-v2, K.inv_mu, 2.0 * rinv);
  double sa, rsa;
  sqrt_rsqrt(alpha, sa, rsa);
  const double a = rsa * rsa;             // meets cos x - 1 and sin x - x only
  const double ms = K.sqrt_mu * sa;       // n a
  const double dM = ms * alpha * dt;
  const double ninv = K.inv_sqrt_mu * rsa * a;
  const double ec = fma_(-r0, alpha, 1.0);
  const double es = u * sa * K.inv_sqrt_mu;
  const double eb = __builtin_fabs(ec) + __builtin_fabs(es);
  const double om = 1.0 - ec;
  const double ar = a * rinv;             // 1/om
  const double t = dM * ar;
  const double h = (0.5 * es) * ar;
  const double c3 = ar * fma_(es, h, ec * (-1.0 / 6.0));
  const double x0 = t * fma_(t, fma_(t, c3, -h), 1.0);
  const double z = x0 * x0;
  double ps, pc;
  series_horner(z, ps, pc);
  const double sx = (x0 * z) * ps;        // sin x0 - x0
  const double sv = x0 + sx;
  const double mv = fma_(z * z, pc, -0.5 * z);
  const double F = fma_(-ec, sv, fma_(-es, mv, x0 - dM));
  const double y = rcp_newton(fma_(-ec, mv, fma_(es, sv, om)));
  const double U = F * y;
  const double A = fma_(ec, sv, fma_(es, mv, es)) * (0.5 * y);
  const double B = fma_(y, 1.0 / 6.0, -1.0 / 6.0);
  const double d = U * fma_(U, fma_(U, fma_(A + A, A, -B), A), 1.0);
  const double x = x0 - d;
  const double d2 = d * d, q = 0.5 * d2;
  const double e3 = (d * d2) * (1.0 / 6.0);
  const double sd = d - e3;               // sin d
  const double smx = sx + fma_(-mv, sd, fma_(-sv, q, e3));   // sin x - x
  const double s = x + smx;
  const double m = fma_(sv, sd, fma_(-(1.0 + mv), q, mv));
  const double iFp = rcp(fma_(-ec, m, fma_(es, s, om)));
  f = fma_(ar, m, 1.0);
  g = fma_(smx, ninv, dt);
  fd = -((ms * rinv) * (s * iFp));
  gd = fma_(iFp, m, 1.0);
  return (__builtin_fabs(x0) <= 0.75) & (eb <= 0.4) & (__builtin_fabs(d) <= 0x1p-14) &
         ((eb * y) * (d2 * d2) <= 0x1p-54 * __builtin_fabs(x));
}

// The drift of a planet held as three components on one lane (nb: 0 there, 1 on a
// lane without a body, whose state is zero and whose dt is 0: it stays).  FAST:
// `bad` is set on a lane that planet_quick does not serve; else such a lane
// takes planet_fg.  Returns false on a body found unbound.
template <bool FAST>
TPM_DEV bool planet_drift(const KepConst& K, double dt, bool lane_on, double nb, double& x,
                          double& y, double& z, double& vx, double& vy, double& vz, bool& bad) {
  const double r2 = fma_(x, x, fma_(y, y, fma_(z, z, nb)));
  const double v2 = fma_(vx, vx, fma_(vy, vy, fma_(vz, vz, nb)));
  const double u = fma_(x, vx, fma_(y, vy, z * vz));
  double f, g, fd, gd;
  const bool served = planet_quick(K, dt, r2, v2, u, f, g, fd, gd) | !lane_on;
  bool bound = true;
  bad = FAST & !served;
  if (!FAST && !wave_all(served)) {
    double f1, g1, fd1, gd1;
    const bool b = planet_fg(K, dt, lane_on, r2, v2, u, f1, g1, fd1, gd1);
    bound = served | b;
    f = served ? f : f1;
    g = served ? g : g1;
    fd = served ? fd : fd1;
    gd = served ? gd : gd1;
  }
  const double nx = fma_(f, x, g * vx), ny = fma_(f, y, g * vy), nz = fma_(f, z, g * vz);
  vx = fma_(fd, x, gd * vx); vy = fma_(fd, y, gd * vy); vz = fma_(fd, z, gd * vz);
  x = nx; y = ny; z = nz;
  return bound;
}

}  // namespace tpm

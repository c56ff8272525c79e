// The planet map of up to four planets on matrix instructions, one wavefront.
//
// A serial chain in time, so its cost is the number of instructions one
// wavefront issues per step.  With a body per lane and three components in
// each (the form for more planets, ephemeris_body) every lane goes through all
// its partners in turn, and 24 lane reads a step bring the positions and 24
// more the accelerations.  Here each lane holds one component of one body, and
// v_mfma_f64_4x4x4f64 does what couples bodies: four independent 4x4 products
// D = A B, with lane 16 i + 4 q + c holding element (i, c) of B and of D in
// block q, and lane 16 k + 4 q + i element (i, k) of A.  So lane 16 b + 4 q + c
// holds component c (3: zero) of Jacobi body b + 1, the same in every block q,
// and a step is
//  * half kick, one FMA;
//  * drift: r^2, v^2 and r.v as sums over the quad, a block each, broadcast
//    along the row; f, g, fdot, gdot by planet_quick; two FMA pairs;
//  * one product gives sixteen difference vectors d, four a block: block 0 the
//    planets' heliocentric positions, block 2 their Jacobi positions, blocks 1
//    and 3 the planet pairs.  g = d/|d|^3 then costs one evaluation for all;
//  * a second product sums the g with their weights per block, and two row
//    rotations add the blocks: the interaction acceleration, in place in every
//    block; a third gives h0 from block 0.
// Weights, with g_p = d_p/|d_p|^3 (a_k the Newtonian acceleration of body k,
// a'_b = a_b - (sum_{k<b} mu_k a_k)/eta_{b-1} + mu'_b r'_b/|r'_b|^3): a central
// pair enters a'_b with -mu'_b if it is b's own, -mu_0 mu_j/eta_{b-1} if
// planet j lies outside b, else 0; the Kepler term with +mu'_b, so the two
// cancel to the difference of their vectors with one and the same factor, and
// for the innermost planet, whose vectors are the same, both are left out; a
// pair i < j with mu_j in a'_i, -mu_i - mu_i mu_j/eta_{j-1} in a'_j and
// -mu_i mu_j/eta_{b-1} between them.
//
// Bound by the instructions of the one wavefront (by the counters 209 vector ones a
// step, its three products of 20 cycles among them, against 405 of the other form when
// it held four planets; 5 to 6 cycles each).  Four
// giant planets: 0.49 us a step, 0.887 in the other form (0.56 with planet_fg's
// two Newton steps for the drift); the error against extended precision over 240
// starts is that of the other form (2.27e-13 rms after 1,000 steps against
// 2.25e-13).  With more than four planets the vectors no longer fit one product
// per lane, and the other form stays.
#pragma once
#include "kepler.hpp"

namespace tpm {

// Value of v on lane SRC of each row of 16, on every lane of the row.
template <int SRC>
TPM_DEV double row_lane(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x150 + SRC, 0xF,
                                                             0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32),
                                                             0x150 + SRC, 0xF, 0xF, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// v plus its value on the lane that the DPP control CTRL names.
template <int CTRL>
TPM_DEV double dpp_sum(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xF, 0xF,
                                                             false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xF,
                                                             0xF, false);
  return v + __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// Sums over a quad and over the four quads of a row; every lane gets the same
// bits (each stage adds the same two numbers on both sides).
TPM_DEV double quad_sum(double v) { return dpp_sum<0x4E>(dpp_sum<0xB1>(v)); }
TPM_DEV double block_sum(double v) { return dpp_sum<0x124>(dpp_sum<0x128>(v)); }

TPM_DEV double mfma4(double a, double b) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, 0.0, 0, 0, 0);
}

// One lane's constants.  NP planets, 1..4.
struct EphQuad {
  int body, col;            // body index (0-based) and component of the lane's state
  bool on;                  // a planet, not a stand-in
  bool dot_v, dot_r;        // which product of the drift's sums the lane's block takes
  double pos;               // A of the difference vectors
  double acc;               // A of the interaction accelerations
  double ind;               // A of h0
  double guard;             // 1 in the fourth component of a vector that is not there
  double hill2;             // squared mutual Hill radius of the lane's pair, -1 if none
  double dt;                // the step, 0 for a stand-in
  KepConst K;
};

// The pair i < j (1-based) of slot i in block 1 or 3; j = 0: none.
TPM_DEV void quad_pair(int blk, int slot, int& i, int& j) {
  i = blk == 1 ? (slot < 3 ? 1 : 2) : (slot == 0 ? 2 : 3);
  j = blk == 1 ? (slot < 3 ? slot + 2 : 3) : (slot < 2 ? 4 : 0);
}

// EP: pointer to the constants, read with per-lane indices.
template <int NP, typename EP>
TPM_DEV EphQuad eph_quad(EP E, double dt, int lane) {
  static_assert(NP >= 1 && NP <= 4, "one to four planets");
  const int row = lane >> 4, blk = (lane >> 2) & 3, col = lane & 3;
  EphQuad Q;
  Q.body = row;
  Q.col = col;
  Q.on = row < NP;
  Q.dot_v = blk == 1;
  Q.dot_r = blk == 0;
  const bool pairs = blk & 1;
  // A of the difference vectors: weight of body row + 1 in vector (blk, col)
  {
    const int k = row + 1, b = col + 1;
    int i, j;
    quad_pair(blk, col, i, j);
    const double ck = E->cj[min(k, NP)];
    double w;
    if (pairs) w = k == j ? 1.0 : (k == i ? ck - 1.0 : (i < k && k < j ? ck : 0.0));
    else w = k == b ? 1.0 : (blk == 0 && k < b ? ck : 0.0);
    const bool there = pairs ? j >= 1 && j <= NP : b <= NP;
    Q.pos = there ? w : 0.0;
  }
  // this lane's vector (blk, row) in B and D, and its weight in a'_{col+1}
  int i, j;
  quad_pair(blk, row, i, j);
  const int v = row + 1, b = col + 1;
  const bool there = pairs ? j >= 1 && j <= NP : v <= NP;
  {
    const double ie = E->inv_eta[min(b, NP) - 1];
    double w = 0.0;
    if (pairs) {
      const double mi = E->mu[min(i, NP)], mj = E->mu[max(min(j, NP), 0)];
      const double mm = -(mi * mj) * ie;
      w = b == i ? mj : (b == j ? mm - mi : (i < b && b < j ? mm : 0.0));
    } else {
      const double mp = E->mup[min(v, NP)];
      const double own = v == b && b > 1 ? mp : 0.0;
      w = blk == 2 ? own : (v > b ? -(E->mu[0] * E->mu[min(v, NP)]) * ie : -own);
    }
    Q.acc = there && b <= NP ? w : 0.0;
  }
  Q.ind = blk == 0 && col == 0 && there ? -E->mu[min(v, NP)] : 0.0;
  Q.guard = !there && col == 3 ? 1.0 : 0.0;
  Q.hill2 = pairs && there ? E->hill2[i][j] : -1.0;
  Q.dt = Q.on ? dt : 0.0;
  const double mup = Q.on ? E->mup[min(v, NP)] : 1.0;
  double smu, rsmu;
  sqrt_rsqrt(mup, smu, rsmu);
  Q.K = KepConst{mup, rcp(mup), smu, rsmu};
  return Q;
}

// The difference vectors of the Jacobi positions j, the interaction
// acceleration a, h0 (lanes 0..2) and whether the lane's pair is closer than
// its mutual Hill radius.
TPM_DEV bool quad_accel(const EphQuad& Q, double j, double& d, double& a, double& h0) {
  d = mfma4(Q.pos, j);
  const double d2 = quad_sum(fma_(d, d, Q.guard));
  const double g = mul_rsqrt3(1.0, d2) * d;
  a = block_sum(mfma4(Q.acc, g));
  h0 = mfma4(Q.ind, g);
  return d2 < Q.hill2;
}

// Kepler drift of the state (j, w).  FAST: `bad` is set on a lane that
// planet_quick does not serve; else such a lane takes planet_fg.
template <bool FAST>
TPM_DEV bool quad_drift(const EphQuad& Q, double& j, double& w, bool& bad) {
  const double p = quad_sum((Q.dot_v ? w : j) * (Q.dot_r ? j : w));
  const double r2 = row_lane<0>(p), v2 = row_lane<4>(p), u = row_lane<8>(p);
  double f, g, fd, gd;
  const bool served = planet_quick(Q.K, Q.dt, r2, v2, u, f, g, fd, gd);
  bool bound = true;
  bad = FAST & !served;
  if (!FAST && !wave_all(served)) {
    double f1, g1, fd1, gd1;
    const bool b = planet_fg(Q.K, Q.dt, Q.on, r2, v2, u, f1, g1, fd1, gd1);
    bound = served | b;
    f = served ? f : f1;
    g = served ? g : g1;
    fd = served ? fd : fd1;
    gd = served ? gd : gd1;
  }
  const double nj = fma_(f, j, g * w);
  w = fma_(fd, j, gd * w);
  j = nj;
  return bound;
}

}  // namespace tpm

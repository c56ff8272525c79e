// Close-encounter hand-off (Zhang & Gladman 2021, sec. 5: particles in close
// encounters move off the main integration, so the bulk keeps its uniform,
// full-speed kernel).  The method of the encounter integration is this
// library's reading, applied identically by the oracle:
//
//  * at every step boundary a particle within the hand-off radius rcrit_j of
//    any planet takes its next step as an encounter step, any other particle
//    the plain map step;
//  * an encounter step is M equal substeps h = dt/M of the same kick - drift -
//    kick, with the planets between the two table rows on the cubic Hermite
//    interpolant of their heliocentric positions and velocities (the row
//    values themselves at the step's two ends) and h0 = -sum_j mu_j r_j/|r_j|^3
//    of the interpolated positions;
//  * removal within the removal radius rrem_j at any step or substep boundary
//    (lowest j; step n at a step boundary, n + 1 at a substep inside step n,
//    keeping that substep's state), beyond rmax at a step boundary, or on a
//    refused drift (the state at the start of the failing substep, step n).
//
// The particle kernel hands a lane off where it would otherwise record an
// encounter removal (hand-off radius = its rcrit) and leaves its state in the
// working set; handoff_gather moves such entries to the encounter list;
// encounter_run advances the list towards the end of a chunk, four lanes per
// entry (entries differ in their steps, which is why they left the main kernel);
// handoff_merge puts the survivors back into the working set at the end of
// an integrate call.  A lane may lag behind the main kernel: every launch
// gives it a budget of micro-steps, and where it stops (at a step or substep
// boundary) the next launch resumes it, with the planet rows of every chunk
// of the call still in place; the last launch of a call has no budget.
#include <hip/hip_runtime.h>

#include "internal.h"
#include "particle.hpp"
#include "universal.hpp"

namespace tpm {

constexpr int ENC_WAVE = 16;   // list entries per wavefront (encounter_run)

__global__ void __launch_bounds__(256)
handoff_gather(Work w, const int32_t* __restrict__ d_nactive, EncList L, int64_t step0) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= *d_nactive) return;
  const int32_t st = w.status[i];
  if (st < HANDOFF_BASE) return;
  const int k = atomicAdd(L.count, 1);
  L.x[k] = w.x[i]; L.y[k] = w.y[i]; L.z[k] = w.z[i];
  L.vx[k] = w.vx[i]; L.vy[k] = w.vy[i]; L.vz[k] = w.vz[i];
  L.slot[k] = w.slot[i];
  L.status[k] = ST_ACTIVE;
  L.step[k] = step0 + (st - HANDOFF_BASE);
  L.m[k] = -1;                            // not yet checked at its hand-off boundary
  w.status[i] = ST_HANDED;
}

__global__ void __launch_bounds__(64) handoff_snap(const int32_t* count, int32_t* snap) {
  if (threadIdx.x == 0) *snap = *count;
}

hipError_t launch_handoff_gather(Work w, const int32_t* d_nactive, int n_upper, EncList L,
                                 int64_t step0, int32_t* snap, hipStream_t st) {
  if (n_upper > 0)
    hipLaunchKernelGGL(handoff_gather, dim3((n_upper + 255) / 256), dim3(256), 0, st, w, d_nactive,
                       L, step0);
  hipLaunchKernelGGL(handoff_snap, dim3(1), dim3(64), 0, st, L.count, snap);
  return hipGetLastError();
}

template <int NP>
struct EncArgs {
  PlanetConst<NP> Prem;   // mu and the removal radii squared
  double renc2[NP > 0 ? NP : 1];
  KepConst K;
  double rmax2, ftol, dt;
  int kiters, M, universal;
  int64_t target;         // step (from the call's start) the lanes advance to
  int64_t budget;         // micro-steps per lane in this launch; 0 = no limit
};

// One particle of the list on four lanes of a wavefront, sixteen entries in
// all: lane 16 k + p works for entry p and holds the rows of planet k (and of
// planet k + 4 if there are more than four).  The state is the same on all
// four, which do the drift together; the planets' interpolation, their
// distances and forces are a lane's own, and the sums over the planets are
// v_mfma_f64_4x4x4f64 products.  In its layout lane 16 k + 4 q + i holds element
// (i, k) of A and (k, i) of B, and D's (i, i) is on lane 16 i + 4 q + i: with the
// factors -mu_j/|d_j|^3 in A and a component of d in B the diagonal is the FMA
// chain over the planets, in their order, of the particle kernel's accel
// (the other elements mix particles and are not used).  A second product, of
// ones with the diagonal and zeros elsewhere, brings it to the particle's four
// lanes.  Lanes without a planet carry a mass of zero.
//
// Each entry runs its own sequence of micro-steps, a plain step (one kick -
// drift - kick of dt) or one substep of an encounter step (of dt / M), so an
// entry in an encounter costs its wavefront M micro-steps per step and the
// others go on with their plain steps meanwhile: a wavefront takes the largest
// number of (plain steps + M x encounter steps) of its entries, not M per step
// whenever any is in an encounter.  The acceleration at the end of a plain step
// or of a step's last substep comes from the row itself (exactly the main
// kernel's arithmetic: at tau = 1 the interpolant is the closing row to the bit,
// and h0 is taken from the row), inside a step from the interpolated planets.
// The two rows of a step stay in registers through its substeps and the next
// closing row is fetched before the last one's drift.  An entry begins at a
// step boundary (its hand-off boundary, or where a launch left it) as the
// particle kernel enters a chunk: acceleration, removal-radius and escape
// checks from the row there; inside a step (a budget stopped it after a
// substep) with the acceleration of the interpolated planets there.  Either
// gives the values it had when it stopped, bit for bit.  Entries that are done
// or removed have left their results and ride along, so the loop has no
// divergent branch but the exits and the row change.  KIT > 0 fixes the Newton
// count at compile time, as in the particle kernel.
//
// Bound by the micro-steps of the longest encounter in the list, one after the
// other (thousands, on a lone wavefront): 0.64 us each with four planets and 16
// substeps, 1.25 with an entry per lane, which took a lane's eight
// distances one after the other, read the step's rows again in every substep,
// and made sixty-four entries wait for the longest.  20,000 particles, 800
// steps: 15.0 -> 8.3 ms for the whole call where one entry takes 9,000
// micro-steps; results are the same to the bit.  (A first chunk of 128 steps, to
// start earlier, gains 0.5 ms there and costs 0.3 where encounters are short.)
// encounter_run's parameters in order, for the offsets of the fields that are
// read where they are used (see karg_field).
template <int NP>
struct EncRunArgs {
  EncArgs<NP> A;
  EncList L;
  const int32_t* snap;
  EncRing R;
  Out out;
};

// a b + c of the 4x4 blocks.
TPM_DEV double mfma4_add(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// The lanes whose entry has any of its four lanes in the mask.
TPM_DEV uint64_t entry_lanes(uint64_t mask) {
  mask |= (mask >> 32) | (mask << 32);
  const uint32_t h = (uint32_t)mask;
  const uint32_t f = h | (h >> 16) | (h << 16);
  return ((uint64_t)f << 32) | f;
}

template <int NP, int KIT>
__global__ void __launch_bounds__(64, NP > 4 ? 1 : 2)
encounter_run(EncArgs<NP> A, EncList L_arg, const int32_t* __restrict__ snap, EncRing R,
              Out out_arg) {
  constexpr int ROW = 3 * NP + 3;
  constexpr int PL = NP > 4 ? 2 : 1;         // planets per lane
  // the list's and the results' pointers are read where they are used (the
  // entry, a removal, the exit), which leaves the micro-step loop's scalar
  // registers to its constants
  (void)L_arg;
  (void)out_arg;
  const KargPtr ka = (KargPtr)__builtin_amdgcn_kernarg_segment_ptr();
  auto list = [&]() { return karg_field<EncList>(ka, offsetof(EncRunArgs<NP>, L)); };
  const int count = *snap;
  const int first = blockIdx.x * ENC_WAVE;
  if (first >= count) return;
  const int lane = threadIdx.x, part = lane >> 4;
  const bool diag = part == (lane & 3);
  // chunk c covers steps [cb(c), cb(c + 1)) of the call, cut at its end
  auto cb = [&](int c) -> int64_t {
    const int64_t b = c == 0 ? 0 : R.k0 + (int64_t)(c - 1) * R.k;
    return b < R.nsteps ? b : R.nsteps;
  };
  auto chunk_of = [&](int64_t g) -> int { return g < R.k0 ? 0 : 1 + (int)((g - R.k0) / R.k); };

  // the entry: state, step g of the call, m substeps into it
  int i = first + (lane & 15);
  bool on = i < count;
  i = on ? i : first;
  int64_t g;
  int m, Ml;
  double x, y, z, vx, vy, vz;
  {
    const EncList L = list();
    g = L.step[i] - R.step0;
    m = L.m[i];
    Ml = L.Ml[i];
    x = L.x[i]; y = L.y[i]; z = L.z[i];
    vx = L.vx[i]; vy = L.vy[i]; vz = L.vz[i];
    // (a step outside the call is never the case)
    on = on && L.status[i] == ST_ACTIVE && g >= 0 && g <= R.nsteps && !(m > 0 && g >= R.nsteps);
  }
  uint64_t act = lanes(on);
  if (act == 0) return;
  if (!on) { g = 0; m = 0; }                 // rides along on the call's first step
  const bool inside = m > 0;
  if (!inside) { m = 0; Ml = 1; }

  // the lane's planets
  double mu[PL], rrem2[PL], renc2[PL];
  int off[PL];
#pragma unroll
  for (int q = 0; q < PL; ++q) {
    const int j = part + 4 * q;
    const bool there = j < NP;
    const int jj = there ? j : 0;
    const auto P = karg_pointer<double>(ka, offsetof(EncRunArgs<NP>, A));
    mu[q] = there ? P[offsetof(EncArgs<NP>, Prem.mu) / 8 + jj] : 0.0;
    rrem2[q] = there ? P[offsetof(EncArgs<NP>, Prem.rcrit2) / 8 + jj] : -1.0;
    renc2[q] = there ? P[offsetof(EncArgs<NP>, renc2) / 8 + jj] : -1.0;
    off[q] = 3 * jj;
  }
  // the step's opening and closing rows (positions, velocities) and the closing
  // row's h0; slot rows `row` of chunk c's slot
  struct Planets { double p[PL][3], v[PL][3]; };
  Planets a, b;
  double hx, hy, hz;
  auto row_at = [&](int c, int row) { return R.rows + ((size_t)c * R.ring_rows + row) * ROW; };
  auto vel_at = [&](int c, int row) {
    return R.vrows + ((size_t)c * R.vring_rows + row) * (3 * NP);
  };
  auto load = [&](Planets& P, const double* r, const double* v, bool with_h, double& h0,
                  double& h1, double& h2) {
#pragma unroll
    for (int q = 0; q < PL; ++q)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        P.p[q][k] = r[off[q] + k];
        P.v[q][k] = NP > 0 ? v[off[q] + k] : 0.0;
      }
    if (with_h) { h0 = r[3 * NP]; h1 = r[3 * NP + 1]; h2 = r[3 * NP + 2]; }
  };
  auto open = [&](const double* r, const double* v) { double t; load(a, r, v, false, t, t, t); };
  // the loop's constants, in vector registers: there are not scalar ones enough
  // for them, and a read of the argument segment at each use stalls a lone wave
  const KepConst K{vgpr_held(A.K.mu), vgpr_held(A.K.inv_mu), vgpr_held(A.K.sqrt_mu),
                   vgpr_held(A.K.inv_sqrt_mu)};
  const double dt = vgpr_held(A.dt), ftol = vgpr_held(A.ftol), rmax2 = vgpr_held(A.rmax2);
  const int M = A.M + opaque_zero_vgpr();
  const int64_t target = A.target + opaque_zero_vgpr();

  // Acceleration at (px, py, pz) with the planets at fraction tau of the step,
  // on the Hermite interpolants of their rows; h0 from the closing row on the
  // lanes of `ends` (tau = 1), elsewhere from the interpolated planets.  rem and
  // enc: the lanes whose planets are within their removal and hand-off radius.
  double ax, ay, az;
  uint64_t rem[PL], enc;
  auto accel_at = [&](uint64_t ends, double tau, double px, double py, double pz) {
    double p[PL][3];
    double cx = hx, cy = hy, cz = hz;
    if (act & ~ends) {
      const double t2 = tau * tau, t3 = t2 * tau;
      const double h00 = fma_(2.0, t3, fma_(-3.0, t2, 1.0));
      const double h10 = fma_(-2.0, t2, t3 + tau);
      const double h01 = fma_(-2.0, t3, 3.0 * t2);
      const double h11 = t3 - t2;
      const double d10 = h10 * dt, d11 = h11 * dt;
      double ix = 0.0, iy = 0.0, iz = 0.0;
#pragma unroll
      for (int q = 0; q < PL; ++q) {
#pragma unroll
        for (int k = 0; k < 3; ++k)
          p[q][k] = fma_(h00, a.p[q][k],
                         fma_(d10, a.v[q][k], fma_(h01, b.p[q][k], d11 * b.v[q][k])));
        // h0: -mu_j r_j / |r_j|^3
        const double k0 =
            -mul_rsqrt3(mu[q], fma_(p[q][0], p[q][0], fma_(p[q][1], p[q][1], p[q][2] * p[q][2])));
        ix = mfma4_add(k0, p[q][0], ix);
        iy = mfma4_add(k0, p[q][1], iy);
        iz = mfma4_add(k0, p[q][2], iz);
      }
      const bool e = lane_in(ends);
      cx = e ? cx : ix; cy = e ? cy : iy; cz = e ? cz : iz;
    } else {
#pragma unroll
      for (int q = 0; q < PL; ++q)
#pragma unroll
        for (int k = 0; k < 3; ++k) p[q][k] = b.p[q][k];
    }
    enc = 0;
#pragma unroll
    for (int q = 0; q < PL; ++q) {
      const double dx = px - p[q][0], dy = py - p[q][1], dz = pz - p[q][2];
      const double d2 = fma_(dx, dx, fma_(dy, dy, dz * dz));
      rem[q] = lanes(d2 < rrem2[q]);
      enc |= lanes(d2 < renc2[q]);
      const double k = -mul_rsqrt3(mu[q], d2);
      cx = mfma4_add(k, dx, cx);
      cy = mfma4_add(k, dy, cy);
      cz = mfma4_add(k, dz, cz);
    }
    ax = mfma4_add(1.0, diag ? cx : 0.0, 0.0);
    ay = mfma4_add(1.0, diag ? cy : 0.0, 0.0);
    az = mfma4_add(1.0, diag ? cz : 0.0, 0.0);
  };
  auto removing = [&]() {
    uint64_t r = rem[0];
    if (PL > 1) r |= rem[PL - 1];
    return act & entry_lanes(r);
  };
  auto remove = [&](uint64_t who, int32_t why, int64_t step, double rx, double ry, double rz,
                    double ux, double uy, double uz) {
    act &= ~who;
    if (!lane_in(who) || part != 0) return;
    int pl = -1;
    if (why == ST_ENCOUNTER) {
      // the lowest planet; scanning downwards, the last hit wins
#pragma unroll
      for (int q = PL - 1; q >= 0; --q)
        for (int k = 3; k >= 0; --k)
          pl = (rem[q] >> (16 * k + lane)) & 1 ? 4 * q + k : pl;
    }
    const EncList L = list();
    const Out out = karg_field<Out>(ka, offsetof(EncRunArgs<NP>, out));
    const int k = L.slot[i];
    out.r[3 * k + 0] = rx; out.r[3 * k + 1] = ry; out.r[3 * k + 2] = rz;
    out.v[3 * k + 0] = ux; out.v[3 * k + 1] = uy; out.v[3 * k + 2] = uz;
    out.step[k] = R.step0 + step;
    out.reason[k] = why;
    out.planet[k] = pl;
    L.status[i] = why;
  };
  // the state of entries that stop here for this launch
  auto leave = [&](uint64_t who) {
    act &= ~who;
    if (!lane_in(who) || part != 0) return;
    const EncList L = list();
    L.x[i] = x; L.y[i] = y; L.z[i] = z;
    L.vx[i] = vx; L.vy[i] = vy; L.vz[i] = vz;
    L.step[i] = R.step0 + g;
    L.m[i] = m;
    L.Ml[i] = Ml;
  };
  const double inv_M = 1.0 / M;
  // k / M to rounding (the correction step makes it the quotient of an IEEE
  // division: checked for every k <= M <= 4096)
  auto fraction = [&](int k) -> double {
    if (Ml == 1) return 1.0;
    const double q = k * inv_M;
    return fma_(fma_(-q, (double)Ml, (double)k), inv_M, q);
  };

  // An entry inside step g (a budget stopped it after a substep) is in the
  // chunk that holds the step; one at the boundary g in the chunk that ends at
  // or holds it: at a chunk's end it begins with that chunk's last row (the
  // next chunk's rows may not exist yet when g is the launch's target).
  int c = inside ? chunk_of(g) : (g == 0 ? 0 : chunk_of(g - 1));
  int s = (int)(g - cb(c));
  open(row_at(c, s), vel_at(c, s));
  load(b, row_at(c, s + inside), vel_at(c, s + inside), true, hx, hy, hz);
  uint64_t near;                             // within a hand-off radius at the step's boundary
  {
    const uint64_t at = ~lanes(inside);
    accel_at(at, inside ? fraction(m) : 1.0, x, y, z);
    near = entry_lanes(enc);
    const uint64_t hit = removing() & at;
    if (hit) remove(hit, ST_ENCOUNTER, g, x, y, z, vx, vy, vz);
    const uint64_t far = act & at & lanes(fma_(x, x, fma_(y, y, z * z)) > rmax2);
    if (far) remove(far, ST_ESCAPE, g, x, y, z, vx, vy, vz);
    const uint64_t there = act & lanes(g >= target);
    if (there) leave(there);
  }
  if (act == 0) return;
  int ks = (int)(cb(c + 1) - cb(c));
  if (!lane_in(act)) {
    c = s = 0;
    ks = 1;
  } else if (s == ks) {
    ++c;
    s = 0;
    ks = (int)(cb(c + 1) - cb(c));
  }
  const double* row = row_at(c, s);          // the step's closing row, the slot's row s + 1
  const double* vel = vel_at(c, s);
  open(row, vel);
  row += ROW;
  vel += 3 * NP;
  load(b, row, vel, true, hx, hy, hz);

  const double hM = dt / M;
  int64_t left = A.budget > 0 ? A.budget : INT64_MAX;
  for (; left > 0; --left) {
    // the mode of a step is decided at its first boundary
    if (m == 0) Ml = lane_in(near) ? M : 1;
    const uint64_t ends = lanes(m + 1 == Ml);
    // the closing row of the entry's next step
    Planets n;
    double nhx, nhy, nhz;
    const uint64_t next = act & ends & lanes(g + 1 < target);
    if (lane_in(next)) {
      row += ROW;
      vel += 3 * NP;
      if (s + 1 == ks) {
        row = row_at(c + 1, 1);
        vel = vel_at(c + 1, 1);
      }
      load(n, row, vel, true, nhx, nhy, nhz);
    }
    const double h = Ml == 1 ? dt : hM;
    const double hh = 0.5 * h;
    double nx = x, ny = y, nz = z;
    double nvx = fma_(hh, ax, vx), nvy = fma_(hh, ay, vy), nvz = fma_(hh, az, vz);
    // the fixed-count elliptic solve, retried in universal variables where it
    // is refused and the option is on (the same arithmetic as the particle
    // kernel's step); the state at the start of a failing (sub)step
    double xk, sk, mk;
    const uint64_t refused =
        drift_lanes(K, h, KIT > 0 ? KIT : A.kiters, ftol, KIT == 5, A.universal != 0, act, nx,
                    ny, nz, nvx, nvy, nvz, xk, sk, mk);
    if (refused & act) remove(refused & act, ST_KEPLER, g, x, y, z, vx, vy, vz);
    accel_at(ends, fraction(m + 1), nx, ny, nz);
    x = nx; y = ny; z = nz;
    vx = fma_(hh, ax, nvx); vy = fma_(hh, ay, nvy); vz = fma_(hh, az, nvz);
    // step n + 1 at the step's end or at a substep inside it
    const uint64_t hit = removing();
    if (hit) remove(hit, ST_ENCOUNTER, g + 1, x, y, z, vx, vy, vz);
    ++m;
    if (act & ends) {
      const uint64_t e = entry_lanes(enc);
      near = (near & ~ends) | (e & ends);
      const uint64_t far = act & ends & lanes(fma_(x, x, fma_(y, y, z * z)) > rmax2);
      if (far) remove(far, ST_ESCAPE, g + 1, x, y, z, vx, vy, vz);
      if (lane_in(act & ends)) {
        m = 0;
        ++g;
      }
      const uint64_t there = act & ends & ~next;
      if (there) leave(there);
      if (lane_in(act & ends)) {
        a = b;
        b = n;
        hx = nhx; hy = nhy; hz = nhz;
        if (++s == ks) {
          ++c;
          s = 0;
          ks = (int)(cb(c + 1) - cb(c));
        }
      }
    }
    if (act == 0) return;
  }
  leave(act);
}

template <int NP>
static hipError_t enc_np(const SysConst& S, const double* rrem2, EncList L, const int32_t* snap,
                         int n_upper, const EncRing& R, int64_t target, int64_t budget, double dt,
                         int M, Out out, hipStream_t st) {
  EncArgs<NP> A;
  for (int j = 0; j < (NP > 0 ? NP : 1); ++j) {
    A.Prem.mu[j] = NP > 0 ? S.mu[j] : 0.0;
    A.Prem.rcrit2[j] = NP > 0 ? rrem2[j] : 0.0;
    A.renc2[j] = NP > 0 ? S.rcrit2[j] : 0.0;
  }
  A.K = KepConst{S.mu0, S.inv_mu0, S.sqrt_mu0, S.inv_sqrt_mu0};
  A.rmax2 = S.rmax2;
  A.ftol = S.ftol;
  A.dt = dt;
  A.kiters = S.kiters;
  A.M = M;
  A.universal = S.universal;
  A.target = target;
  A.budget = budget;
  if (quick_serves(S.kiters, S.ftol))
    hipLaunchKernelGGL((encounter_run<NP, 5>), dim3((n_upper + ENC_WAVE - 1) / ENC_WAVE), dim3(64), 0, st, A, L,
                       snap, R, out);
  else
    hipLaunchKernelGGL((encounter_run<NP, 0>), dim3((n_upper + ENC_WAVE - 1) / ENC_WAVE), dim3(64), 0, st, A, L,
                       snap, R, out);
  return hipGetLastError();
}

hipError_t launch_encounter_run(const SysConst& S, const double* rrem2, EncList L,
                                const int32_t* snap, int n_upper, const EncRing& R,
                                int64_t target, int64_t budget, double dt, int M, Out out,
                                hipStream_t st) {
  if (n_upper <= 0) return hipSuccess;
  if (M < 1 || R.k0 < 1 || R.k < 1 || target < 0 || target > R.nsteps)
    return hipErrorInvalidValue;
  switch (S.np) {
#define TPM_ENC(N) \
    case N: return enc_np<N>(S, rrem2, L, snap, n_upper, R, target, budget, dt, M, out, st);
    TPM_ENC(0) TPM_ENC(1) TPM_ENC(2) TPM_ENC(3) TPM_ENC(4) TPM_ENC(5) TPM_ENC(6) TPM_ENC(7)
    TPM_ENC(8)
#undef TPM_ENC
    default: return hipErrorInvalidValue;
  }
}

__global__ void __launch_bounds__(256)
handoff_merge(EncList L, int n_upper, Work w, int32_t* __restrict__ d_nactive) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_upper || i >= *L.count || L.status[i] != ST_ACTIVE) return;
  const int k = atomicAdd(d_nactive, 1);
  w.x[k] = L.x[i]; w.y[k] = L.y[i]; w.z[k] = L.z[i];
  w.vx[k] = L.vx[i]; w.vy[k] = L.vy[i]; w.vz[k] = L.vz[i];
  w.slot[k] = L.slot[i];
  w.status[k] = ST_ACTIVE;
}

__global__ void __launch_bounds__(64) handoff_clear(int32_t* count) {
  if (threadIdx.x == 0) *count = 0;
}

hipError_t launch_handoff_merge(EncList L, int n_upper, Work w, int32_t* d_nactive,
                                hipStream_t st) {
  if (n_upper > 0)
    hipLaunchKernelGGL(handoff_merge, dim3((n_upper + 255) / 256), dim3(256), 0, st, L, n_upper, w,
                       d_nactive);
  hipLaunchKernelGGL(handoff_clear, dim3(1), dim3(64), 0, st, L.count);
  return hipGetLastError();
}

}  // namespace tpm

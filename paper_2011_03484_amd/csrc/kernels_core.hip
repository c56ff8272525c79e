// Core kernels of the test-particle map on gfx950 (FP64 throughout).
//
//  * particle_queue  - one lane per particle; the particle stays in registers
//    for hundreds of steps (sec. 2.2: a single kernel loops over the planet
//    chunk so each particle is read and written once per chunk), with the
//    chunk's (tile, sub-chunk) items handed out dynamically to wavefronts and
//    the planet map of the chunk run by one more wavefront of the same launch.
//    Every lane reads the same planet-table row: broadcast vector loads into
//    VGPRs, one step ahead of its use.
//  * ephemeris_chunk (and planet_rows, inside particle_queue) - one wavefront,
//    each lane one component of one body (up to four planets, planet_quad.hpp)
//    or lane b Jacobi body b.  Wisdom-Holman kick-drift-kick of the planets
//    (sec. 2.2, planet integration) writing the heliocentric positions and the
//    indirect term h0 per step.
//  * compact_kernel  - stable partition of the working set so removed particles
//    stop occupying lanes (sec. 2.2, resync interval), by wave ballots and a
//    look-back over the tiles before.
//  * finalize        - scatter the active particles back to caller order.
#include <algorithm>
#include <climits>

#include "internal.h"
#include "particle.hpp"
#include "planet_quad.hpp"
#include "universal.hpp"

namespace tpm {

// ---------------------------------------------------------------- particles
template <int NP>
struct ChunkArgs {
  PlanetConst<NP> P;
  KepConst K;
  double rmax2, ftol, dt;
  int kiters, nsteps;
  int64_t step0;
  int handoff;   // within rcrit: hand off to the encounter integrator, not removal
  // sampled states (see QueueLaunch); every 0: none
  struct Samples {
    int first, every;
    int64_t stride;
    double* at;
  } samp;
};

// Work queue of one launch (see particle_queue).
struct QueueArgs {
  unsigned long long* ctr;     // monotonic item counter
  unsigned long long base;     // counter value at this launch's start
  uint32_t* progress;          // per tile: sub-chunks completed (monotonic over launches)
  uint32_t epoch;              // progress value of every tile at this launch's start
  int ntiles, nsub, sub_steps, nsteps;
  int32_t* error;
};

// The work-queue kernel's arguments as its argument segment lays them out
// (particle_queue); see karg_field.
struct QueueArgsHead {
  Work w;
  const int32_t* n;
  Out out;
  RowStream R;
};
template <int NP>
struct QueueKernelArgs {
  QueueArgsHead head;
  const double* rows;
  ChunkArgs<NP> A;
  QueueArgs Q;
  EphConst E;
};
TPM_DEV Work karg_work(KargPtr p) { return karg_field<Work>(p, offsetof(QueueArgsHead, w)); }
TPM_DEV Out karg_out(KargPtr p) { return karg_field<Out>(p, offsetof(QueueArgsHead, out)); }
template <typename T>
TPM_DEV T karg_stream(KargPtr p, size_t off) {
  return karg_field<T>(p, offsetof(QueueArgsHead, R) + off);
}

constexpr uint32_t SPIN_LIMIT = 1u << 22;   // about 4 s of polling

// What one wavefront of a launch hands to another that may run on another die
// (a tile's state between its items): stored through to memory and loaded from
// there, each value by itself.  An agent-scope release and acquire would do it
// for plain accesses, by writing back and invalidating the die's whole L2: 20 us
// an item with every wavefront of the die doing so, and nobody's planet rows
// stayed cached.  (shared_done: the stores before it have arrived.)
template <typename T>
TPM_DEV T shared_load(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
TPM_DEV void shared_store(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
TPM_DEV void shared_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

TPM_DEV unsigned long long wave_uniform(unsigned long long v) {
  uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
  return ((unsigned long long)hi << 32) | lo;
}

// Steps of the launch's chunk whose closing rows are published, once that is
// more than s (`have` already known to be): the planet map of the same launch
// writes the rows as the particles follow (planet_rows).  The whole wavefront
// polls the count with relaxed loads.  The rows behind it need no acquire: a
// count ends with a cache line (ROW_GROUP), so no line that holds a published
// row was read, by anyone in this launch, before all of it was written.
// A wait ends when the map, which always runs (see particle_queue), publishes
// its next block; one in which it publishes nothing for the spin limit flags
// an error and returns s.
TPM_DEV int wait_rows(KargPtr ka, int s, int nsteps) {
  const int64_t* cnt = karg_stream<const int64_t*>(ka, offsetof(RowStream, done));
  const int64_t begin = karg_stream<int64_t>(ka, offsetof(RowStream, begin));
  for (uint32_t spins = 0; spins <= SPIN_LIMIT; ++spins) {
    const int64_t p = (int64_t)wave_uniform((unsigned long long)__hip_atomic_load(
                          cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) - begin;
    if (p > s) {
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");   // (orders the code only)
      return p < nsteps ? (int)p : nsteps;
    }
    __builtin_amdgcn_s_sleep(16);
  }
  atomicOr(karg_stream<int32_t*>(ka, offsetof(RowStream, error)), 1);
  return s;
}

// Advance particle i of the working set through steps [s_begin, s_end) of a
// chunk whose rows start at `rows` (row k = step step0 + k).  KIT = 5 serves
// failure thresholds from QUICK_FTOL up (drift_quick).  The rows are
// written before the launch, or (KA with a row stream) by the launch's own
// planet map as the particles follow: `have` counts the steps whose closing
// rows are published, and the wavefront waits for more where it runs out
// (wait_rows).  The step loop is uniform across the
// wavefront (s_begin, s_end are wave-uniform); removed lanes are masked off
// and the wavefront leaves early once none is active.  KIT > 0 fixes the
// Newton count at compile time; AHEAD fetches each planet row a step ahead into
// VGPRs (for launches with a few wavefronts per SIMD; else scalar loads at the
// point of use, for many).
//
// UNIV: a drift the fixed-iteration solve refuses is taken in universal
// variables instead (drift_lanes); the particle is removed as KEPLER only if
// that gives no finite result either.
// KA: w and out are read from the work-queue kernel's argument segment ka
// where they are used (the item's start and end, a record), which leaves the
// step loop's scalar registers to its constants.
template <int NP, int KIT, bool AHEAD, bool UNIV = false, bool KA = false>
TPM_DEV void advance(Work w, Out out, const double* rows, const ChunkArgs<NP>& A, int i,
                     bool valid, int s_begin, int s_end, KargPtr ka, int& have) {
  constexpr int ROW = 3 * NP + 3;
  const int kiters = KIT > 0 ? KIT : A.kiters;
  if (KA) w = karg_work(ka);
  double x = 0, y = 0, z = 0, vx = 0, vy = 0, vz = 0;
  if (valid) {
    x = shared_load(w.x + i); y = shared_load(w.y + i); z = shared_load(w.z + i);
    vx = shared_load(w.vx + i); vy = shared_load(w.vy + i); vz = shared_load(w.vz + i);
    valid = shared_load(w.status + i) == ST_ACTIVE;
  }
  // A lane's removal record (the state it keeps, step, reason, planet) is
  // written out in the step that removes it.  `act` holds the lanes still
  // integrated: the others ride along, their states mean nothing and enter no
  // test (masking them out of the step would cost every step an exec mask and
  // a branch).  With the hand-off on, a lane within a planet's radius is
  // handed off instead: its state stays in the working set, marked with its
  // local step, for the encounter integrator.
  uint64_t act = lanes(valid);
  auto record = [&](int32_t why, int64_t st, int32_t pl, double rx, double ry, double rz,
                    double ux, double uy, double uz) {
    const Work wr = KA ? karg_work(ka) : w;
    if (A.handoff && why == ST_ENCOUNTER) {
      wr.x[i] = rx; wr.y[i] = ry; wr.z[i] = rz;
      wr.vx[i] = ux; wr.vy[i] = uy; wr.vz[i] = uz;
      shared_store(wr.status + i, HANDOFF_BASE + (int32_t)(st - A.step0));
      return;
    }
    const Out o = KA ? karg_out(ka) : out;
    const int k = wr.slot[i];
    o.r[3 * k + 0] = rx; o.r[3 * k + 1] = ry; o.r[3 * k + 2] = rz;
    o.v[3 * k + 0] = ux; o.v[3 * k + 1] = uy; o.v[3 * k + 2] = uz;
    o.step[k] = st;
    o.reason[k] = why;
    o.planet[k] = pl;
    shared_store(wr.status + i, why);
  };
  double ax, ay, az, r2;
  if (KA && have <= s_begin) {
    have = wait_rows(ka, s_begin, A.nsteps);
    if (have <= s_begin) return;            // the wait gave up (flagged)
  }
  {
    const int hit = accel<NP>(rows + (size_t)s_begin * ROW, A.P, x, y, z, ax, ay, az);
    r2 = fma_(x, x, fma_(y, y, z * z));
    const bool far = r2 > A.rmax2;
    if (valid) {
      if (hit >= 0) record(ST_ENCOUNTER, A.step0 + s_begin, hit, x, y, z, vx, vy, vz);
      else if (far) record(ST_ESCAPE, A.step0 + s_begin, -1, x, y, z, vx, vy, vz);
    }
    act &= ~lanes((hit >= 0) | far);
  }
  const double h = 0.5 * A.dt;
  // one step s -> s + 1, with the row that ends it (row s + 1)
  auto step = [&](int s, const auto& row) {
    double nx = x, ny = y, nz = z;
    double nvx = fma_(h, ax, vx), nvy = fma_(h, ay, vy), nvz = fma_(h, az, vz);
    double xk, sk, mk;
    const uint64_t bad = drift_lanes(A.K, A.dt, kiters, A.ftol, KIT == 5, UNIV, act, r2, nx, ny,
                                     nz, nvx, nvy, nvz, xk, sk, mk);
    double bx, by, bz;
    uint64_t near;
    const auto hit_of = accel_near<NP>(row, A.P, nx, ny, nz, bx, by, bz, near);
    r2 = fma_(nx, nx, fma_(ny, ny, nz * nz));
    const uint64_t far = lanes(r2 > A.rmax2);
    nvx = fma_(h, bx, nvx); nvy = fma_(h, by, nvy); nvz = fma_(h, bz, nvz);
    const uint64_t gone = act & (bad | near | far);
    if (gone) {
      if (lane_in(gone)) {
        // a Kepler failure keeps the state at the start of the step
        if (lane_in(bad)) record(ST_KEPLER, A.step0 + s, -1, x, y, z, vx, vy, vz);
        else if (lane_in(near))
          record(ST_ENCOUNTER, A.step0 + s + 1, hit_of(), nx, ny, nz, nvx, nvy, nvz);
        else record(ST_ESCAPE, A.step0 + s + 1, -1, nx, ny, nz, nvx, nvy, nvz);
      }
      act &= ~gone;
    }
    x = nx; y = ny; z = nz;
    vx = nvx; vy = nvy; vz = nvz;
    ax = bx; ay = by; az = bz;
  };
  // the item's first sampled step (after s_begin: a state at s_begin is the
  // item's before)
  int next = INT_MAX;
  using Samples = typename ChunkArgs<NP>::Samples;
  constexpr size_t SAMPLES = offsetof(QueueKernelArgs<NP>, A) + offsetof(ChunkArgs<NP>, samp);
  if (KA) {
    const Samples q = karg_field<Samples>(ka, SAMPLES);
    if (q.every > 0) {
      next = q.first;
      if (next <= s_begin) next += ((s_begin - next) / q.every + 1) * q.every;
    }
  }
  for (int s0 = s_begin;;) {
    if (KA && have <= s0) {
      have = wait_rows(ka, s0, A.nsteps);
      if (have <= s0) break;                // the wait gave up (flagged)
    }
    const int lim = KA ? min(min(s_end, have), next) : s_end;
    if (AHEAD) {
      // The row that ends step s is fetched during step s - 1, into the one of
      // two alternating VGPR buffers that step s - 1 does not use: with few
      // wavefronts per SIMD nothing else hides that load's latency.
      const int zero = opaque_zero_vgpr();
      Row<NP> ra, rb;
      load_row<NP>(ra, rows + (size_t)(s0 + 1) * ROW, zero);
      for (int s = s0; s < lim; s += 2) {
        if (act == 0) break;
        load_row<NP>(rb, rows + (size_t)min(s + 2, lim) * ROW, zero);
        step(s, ra.v);
        if (s + 1 >= lim) break;
        load_row<NP>(ra, rows + (size_t)min(s + 3, lim) * ROW, zero);
        step(s + 1, rb.v);
      }
    } else {
      // many wavefronts per SIMD: rows by scalar loads at their use
      for (int s = s0; s < lim; ++s) {
        if (act == 0) break;
        step(s, rows + (size_t)(s + 1) * ROW);
      }
    }
    s0 = lim;
    if (KA && s0 == next) {
      const Samples q = karg_field<Samples>(ka, SAMPLES);
      if (lane_in(act)) {
        const int64_t k = q.stride;
        double* p = q.at + 6 * k * ((s0 - q.first) / q.every) + i;
        p[0] = x; p[k] = y; p[2 * k] = z;
        p[3 * k] = vx; p[4 * k] = vy; p[5 * k] = vz;
      }
      next += q.every;
    }
    if (!KA || s0 >= s_end || act == 0) break;
  }
  if (lane_in(act)) {
    const Work we = KA ? karg_work(ka) : w;
    shared_store(we.x + i, x); shared_store(we.y + i, y); shared_store(we.z + i, z);
    shared_store(we.vx + i, vx); shared_store(we.vy + i, vy); shared_store(we.vz + i, vz);
  }
}

// Work queue of one chunk: item = (sub-chunk s, tile t) in s-major order,
// tile = 64 consecutive working-set entries (one wavefront).  Wavefronts take
// items from a monotonic counter, so a wavefront that shares its SIMD with
// other work (or sits alone on one) simply takes fewer items.  Item (s, t)
// waits for item (s-1, t) through a per-tile progress counter; that item was
// taken earlier by a running wavefront, so the wait always ends.  A wait
// longer than the spin limit flags an error and drops the item.
//
// With a row stream (R.on) the queue's first item is the planet map itself:
// the wavefront that takes it writes the chunk's planet rows (planet_rows)
// while the others follow it through them, a block of steps behind.  That
// wavefront runs by definition and waits for nobody, whichever order the
// launch's workgroups start in, so every wait for rows ends.  As launches of
// its own the map had to finish a chunk before the particles could start on
// it, so a call of one or two chunks took the sum of both: 10,000 steps of
// 13,313 particles 16.7 ms, then 9.5; 1,000 steps of 16,384 particles on one
// stream 1.74 ms, then 1.01; 10,000 steps of 200,000 particles 29.2 ms, then 21.8
// (5.3, 0.57 and 15.0 with the shorter steps since).
//
// No part of the item loop runs on a subset of the lanes: the grab, the wait
// and the publish are executed by the whole wavefront (lane 0 alone adds 1 to
// the counter), so the readfirstlane that makes their results wave-uniform
// always sees the full wavefront and the loop's branches stay scalar.
template <int NP>
TPM_DEV void run_planet_rows(KargPtr ka);

template <int NP, int KIT, bool UNIV>
__global__ void __launch_bounds__(256, 2)
particle_queue(Work w, const int32_t* __restrict__ d_nactive, Out out, RowStream R,
               const double* rows, ChunkArgs<NP> A, QueueArgs Q, EphConst E) {
  (void)E;                             // read by planet_rows from the argument segment
  const KargPtr ka = (KargPtr)__builtin_amdgcn_kernarg_segment_ptr();
  const int lane = threadIdx.x & 63;
  const int n = *d_nactive;
  const unsigned long long map_item = R.on ? 1ull : 0ull;
  int have = R.on ? 0 : Q.nsteps;
  const unsigned long long total = (unsigned long long)Q.ntiles * Q.nsub;
  const unsigned long long one = lane == 0 ? 1ull : 0ull;
  unsigned long long grab = wave_uniform(atomicAdd(Q.ctr, one) - Q.base);
  if (grab < map_item) {
    // the launch's first grab; this wavefront does nothing else (so that no
    // value of the item loop has to outlive the call)
    run_planet_rows<NP>(ka);
    return;
  }
  for (;; grab = wave_uniform(atomicAdd(Q.ctr, one) - Q.base)) {
    const unsigned long long item = grab - map_item;
    if (item >= total) break;
    const int s = (int)(item / Q.ntiles);
    const int t = (int)(item % Q.ntiles);
    bool go = true;
    if (s > 0) {
      const uint32_t target = Q.epoch + (uint32_t)s;
      uint32_t spins = 0;
      for (;;) {
        const uint32_t p = (uint32_t)__builtin_amdgcn_readfirstlane(
            (int)__hip_atomic_load(Q.progress + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        if ((int32_t)(p - target) >= 0) break;
        if (++spins > SPIN_LIMIT) {
          atomicOr(Q.error, 1);
          go = false;
          break;
        }
        __builtin_amdgcn_s_sleep(2);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");   // (orders the code only)
    }
    const int s_begin = s * Q.sub_steps;
    const int s_end = min(Q.nsteps, s_begin + Q.sub_steps);
    if (go && s_begin < s_end) {       // the last sub-chunks of a short chunk may be empty
      const int i = t * 64 + lane;
      advance<NP, KIT, true, UNIV, true>(w, out, rows, A, i, i < n, s_begin, s_end, ka, have);
    }
    // publish completion, after the state has arrived
    shared_done();
    shared_store(Q.progress + t, Q.epoch + (uint32_t)s + 1u);
  }
}

// ---------------------------------------------------------- many systems
// Item (s, t) of the batched queue: tile t (64 particles of one system, so the
// planet row stays wave-uniform) through sub-chunk s; the tile's system picks
// the planet count, constants, time step and table rows.
template <int NP>
TPM_DEV void batch_item(const SysDev& S, Work w, Out out, const double* __restrict__ ring,
                        const BatchQueueArgs& Q, const TileDesc& T, int s_begin, int s_end,
                        int lane) {
  ChunkArgs<NP> A;
#pragma unroll
  for (int j = 0; j < (NP > 0 ? NP : 1); ++j) {
    A.P.mu[j] = NP > 0 ? S.mu[j] : 0.0;
    A.P.rcrit2[j] = NP > 0 ? S.rcrit2[j] : 0.0;
  }
  A.K = S.K;
  A.rmax2 = S.rmax2;
  A.ftol = S.ftol;
  A.dt = S.dt;
  A.kiters = S.kiters;
  A.nsteps = Q.nsteps;
  A.step0 = Q.step0;
  A.handoff = 0;
  A.samp = {};
  const double* rows = ring + S.ring_off + (int64_t)Q.slot * Q.slot_rows * (3 * NP + 3);
  const int i = T.first + lane;
  const bool valid = lane < T.count;
  int have = s_end;                    // the rows are written before the launch
  if (quick_serves(S.kiters, S.ftol))
    advance<NP, 5, false>(w, out, rows, A, i, valid, s_begin, s_end, nullptr, have);
  else
    advance<NP, 0, false>(w, out, rows, A, i, valid, s_begin, s_end, nullptr, have);
}

__global__ void __launch_bounds__(256)
particle_batch_queue(const SysDev* __restrict__ sys, const TileDesc* __restrict__ tiles, Work w,
                     Out out, const double* __restrict__ ring, BatchQueueArgs Q) {
  const int lane = threadIdx.x & 63;
  // the tile count of a run that compacts lives on the device (batch_tiles)
  const int ntiles = Q.ntiles_dev ? *Q.ntiles_dev : Q.ntiles;
  const unsigned long long total = (unsigned long long)ntiles * Q.nsub;
  const unsigned long long one = lane == 0 ? 1ull : 0ull;
  for (;;) {
    const unsigned long long item = wave_uniform(atomicAdd(Q.ctr, one) - Q.base);
    if (item >= total) break;
    const int s = (int)(item / ntiles);
    const int t = (int)(item % ntiles);
    bool go = true;
    if (s > 0) {
      const uint32_t target = Q.epoch + (uint32_t)s;
      uint32_t spins = 0;
      for (;;) {
        const uint32_t p = (uint32_t)__builtin_amdgcn_readfirstlane(
            (int)__hip_atomic_load(Q.progress + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        if ((int32_t)(p - target) >= 0) break;
        if (++spins > SPIN_LIMIT) {
          atomicOr(Q.error, 1);
          go = false;
          break;
        }
        __builtin_amdgcn_s_sleep(2);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");   // (orders the code only)
    }
    const int s_begin = s * Q.sub_steps;
    const int s_end = min(Q.nsteps, s_begin + Q.sub_steps);
    if (go && s_begin < s_end) {
      const TileDesc T = tiles[t];
      const SysDev& S = sys[T.sys];
      switch (S.np) {
        case 0: batch_item<0>(S, w, out, ring, Q, T, s_begin, s_end, lane); break;
        case 1: batch_item<1>(S, w, out, ring, Q, T, s_begin, s_end, lane); break;
        case 2: batch_item<2>(S, w, out, ring, Q, T, s_begin, s_end, lane); break;
        case 3: batch_item<3>(S, w, out, ring, Q, T, s_begin, s_end, lane); break;
        case 4: batch_item<4>(S, w, out, ring, Q, T, s_begin, s_end, lane); break;
        case 5: batch_item<5>(S, w, out, ring, Q, T, s_begin, s_end, lane); break;
        case 6: batch_item<6>(S, w, out, ring, Q, T, s_begin, s_end, lane); break;
        case 7: batch_item<7>(S, w, out, ring, Q, T, s_begin, s_end, lane); break;
        default: batch_item<8>(S, w, out, ring, Q, T, s_begin, s_end, lane); break;
      }
    }
    shared_done();
    shared_store(Q.progress + t, Q.epoch + (uint32_t)s + 1u);
  }
}

hipError_t launch_particle_batch(const SysDev* sys, const TileDesc* tiles, Work w, Out out,
                                 const double* ring, const BatchQueueArgs& Q, int workers,
                                 int block, hipStream_t st) {
  if (Q.ntiles <= 0) return hipSuccess;
  const int wpb = block / 64;
  const int nblocks = (workers + wpb - 1) / wpb;
  hipLaunchKernelGGL(particle_batch_queue, dim3(nblocks), dim3(block), 0, st, sys, tiles, w, out,
                     ring, Q);
  return hipGetLastError();
}

// ---- compaction inside a batched run (captured in its graph)
// After a stable partition of the whole working set (launch_compact), each
// system's active particles are still contiguous and in order, so the tiles
// are rebuilt from each system's range [start, end) in the new working set:
// batch_bounds finds the ranges from the slots' systems, batch_tiles lays the
// systems' tiles out in the queue's order (most planets first) and stores the
// new tile count for the next particle launch.
__global__ void __launch_bounds__(256) batch_bounds_clear(int nsys, int32_t* start, int32_t* end) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < nsys) { start[s] = 0; end[s] = 0; }
}

__global__ void __launch_bounds__(256)
batch_bounds(const int32_t* __restrict__ slot, const int32_t* __restrict__ d_nactive,
             const int32_t* __restrict__ psys, int32_t* __restrict__ start,
             int32_t* __restrict__ end) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int n = *d_nactive;
  if (i >= n) return;
  const int s = psys[slot[i]];
  if (i == 0 || psys[slot[i - 1]] != s) start[s] = i;
  if (i == n - 1 || psys[slot[i + 1]] != s) end[s] = i + 1;
}

__global__ void __launch_bounds__(1024)
batch_tiles(const int32_t* __restrict__ sorder, int nsys, const int32_t* __restrict__ start,
            const int32_t* __restrict__ end, TileDesc* __restrict__ tiles,
            int32_t* __restrict__ ntiles_dev) {
  __shared__ int buf[1024];
  __shared__ int carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int base = 0; base < nsys; base += 1024) {
    const int k = base + threadIdx.x;
    const int s = k < nsys ? sorder[k] : 0;
    const int cnt = k < nsys ? end[s] - start[s] : 0;
    const int nt = (cnt + 63) / 64;
    buf[threadIdx.x] = nt;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
      const int t = threadIdx.x >= off ? buf[threadIdx.x - off] : 0;
      __syncthreads();
      buf[threadIdx.x] += t;
      __syncthreads();
    }
    const int first = carry + buf[threadIdx.x] - nt;
    for (int j = 0; j < nt; ++j)
      tiles[first + j] = TileDesc{s, start[s] + 64 * j, min(64, cnt - 64 * j), 0};
    __syncthreads();
    if (threadIdx.x == 1023) carry += buf[1023];
    __syncthreads();
  }
  if (threadIdx.x == 0) *ntiles_dev = carry;
}

// Workgroup b: tile b, and system b.
__global__ void __launch_bounds__(64)
batch_reset(const TileDesc* __restrict__ tiles0, TileDesc* __restrict__ tiles, int ntiles,
            int32_t* ntiles_dev, int32_t* __restrict__ psys, const double* __restrict__ rj0,
            const double* __restrict__ vj0, double* __restrict__ rj, double* __restrict__ vj,
            int64_t* __restrict__ flag, int nsys, unsigned long long* acc, int32_t* scratch,
            int nscratch) {
  const int b = blockIdx.x, lane = threadIdx.x;
  for (int k = b * 64 + lane; k < nscratch; k += 64 * gridDim.x) scratch[k] = 0;
  if (b < ntiles) {
    const TileDesc T = tiles0[b];
    if (lane < T.count) psys[T.first + lane] = T.sys;
    if (lane == 0) tiles[b] = T;
  }
  if (b < nsys) {
    if (lane < 3 * MAX_NP) {
      rj[3 * MAX_NP * b + lane] = rj0[3 * MAX_NP * b + lane];
      vj[3 * MAX_NP * b + lane] = vj0[3 * MAX_NP * b + lane];
    }
    if (lane == 0) flag[b] = -1;
  }
  if (b == 0 && lane == 0) {
    *ntiles_dev = ntiles;
    *acc = 0;
  }
}

hipError_t launch_batch_reset(const TileDesc* tiles0, TileDesc* tiles, int ntiles,
                              int32_t* ntiles_dev, int32_t* psys, const double* rj0,
                              const double* vj0, double* rj, double* vj, int64_t* flag, int nsys,
                              unsigned long long* acc, int32_t* scratch, int nscratch,
                              hipStream_t st) {
  hipLaunchKernelGGL(batch_reset, dim3(std::max(std::max(ntiles, nsys), 1)), dim3(64), 0, st,
                     tiles0, tiles, ntiles, ntiles_dev, psys, rj0, vj0, rj, vj, flag, nsys, acc,
                     scratch, nscratch);
  return hipGetLastError();
}

__global__ void __launch_bounds__(64) queue_reset(unsigned long long* ctr) {
  if (threadIdx.x == 0) *ctr = 0ull;
}

hipError_t launch_batch_retile(Work w, const int32_t* d_nactive, int n_upper, const int32_t* psys,
                               const int32_t* sorder, int nsys, int32_t* start, int32_t* end,
                               TileDesc* tiles, int32_t* ntiles_dev, hipStream_t st) {
  hipLaunchKernelGGL(batch_bounds_clear, dim3((nsys + 255) / 256), dim3(256), 0, st, nsys, start,
                     end);
  if (n_upper > 0)
    hipLaunchKernelGGL(batch_bounds, dim3((n_upper + 255) / 256), dim3(256), 0, st, w.slot,
                       d_nactive, psys, start, end);
  hipLaunchKernelGGL(batch_tiles, dim3(1), dim3(1024), 0, st, sorder, nsys, start, end, tiles,
                     ntiles_dev);
  return hipGetLastError();
}

hipError_t launch_queue_reset(unsigned long long* ctr, hipStream_t st) {
  hipLaunchKernelGGL(queue_reset, dim3(1), dim3(64), 0, st, ctr);
  return hipGetLastError();
}

template <int NP>
static hipError_t launch_np(const SysConst& S, Work w, const int32_t* d_nactive, int grid_n,
                            Out out, const double* rows, int nsteps, double dt, int64_t step0,
                            const QueueLaunch& QL, hipStream_t st) {
  ChunkArgs<NP> A;
  for (int j = 0; j < NP; ++j) { A.P.mu[j] = S.mu[j]; A.P.rcrit2[j] = S.rcrit2[j]; }
  if (NP == 0) { A.P.mu[0] = 0.0; A.P.rcrit2[0] = 0.0; }
  A.K = KepConst{S.mu0, S.inv_mu0, S.sqrt_mu0, S.inv_sqrt_mu0};
  A.rmax2 = S.rmax2;
  A.ftol = S.ftol;
  A.dt = dt;
  A.kiters = S.kiters;
  A.nsteps = nsteps;
  A.step0 = step0;
  A.handoff = S.handoff;
  A.samp = {QL.samp_first, QL.samp ? QL.samp_every : 0, QL.samp_stride, QL.samp};
  QueueArgs Q;
  Q.ctr = QL.ctr;
  Q.base = QL.base;
  Q.progress = QL.progress;
  Q.epoch = QL.epoch;
  Q.ntiles = (grid_n + 63) / 64;
  Q.nsub = QL.nsub;
  Q.sub_steps = (nsteps + QL.nsub - 1) / QL.nsub;
  Q.nsteps = nsteps;
  Q.error = QL.error;
  RowStream R{};
  EphConst E{};
  if (QL.stream) {
    R = *QL.stream;
    E = *QL.eph;
  }
  R.error = QL.error;
  R.ctr = QL.ctr;
  R.ctr_base = QL.base;
  R.ctr_alone = QL.grabs(Q.ntiles);
  if (Q.ntiles <= 0 && !R.on) return hipSuccess;
  const int nblocks = QL.blocks();
#define TPM_PQ(KIT, UNIV)                                                                     \
  hipLaunchKernelGGL((particle_queue<NP, KIT, UNIV>), dim3(nblocks), dim3(QL.block), 0, st, w, \
                     d_nactive, out, R, rows, A, Q, E)
  const bool quick = quick_serves(S.kiters, S.ftol);
  if (quick) {
    if (S.universal) TPM_PQ(5, true);
    else TPM_PQ(5, false);
  } else {
    if (S.universal) TPM_PQ(0, true);
    else TPM_PQ(0, false);
  }
#undef TPM_PQ
  return hipGetLastError();
}

hipError_t launch_particle_chunk(const SysConst& S, Work w, const int32_t* d_nactive, int grid_n,
                                 Out out, const double* rows, int nsteps, double dt, int64_t step0,
                                 const QueueLaunch& QL, hipStream_t st) {
  switch (S.np) {
    case 0: return launch_np<0>(S, w, d_nactive, grid_n, out, rows, nsteps, dt, step0, QL, st);
    case 1: return launch_np<1>(S, w, d_nactive, grid_n, out, rows, nsteps, dt, step0, QL, st);
    case 2: return launch_np<2>(S, w, d_nactive, grid_n, out, rows, nsteps, dt, step0, QL, st);
    case 3: return launch_np<3>(S, w, d_nactive, grid_n, out, rows, nsteps, dt, step0, QL, st);
    case 4: return launch_np<4>(S, w, d_nactive, grid_n, out, rows, nsteps, dt, step0, QL, st);
    case 5: return launch_np<5>(S, w, d_nactive, grid_n, out, rows, nsteps, dt, step0, QL, st);
    case 6: return launch_np<6>(S, w, d_nactive, grid_n, out, rows, nsteps, dt, step0, QL, st);
    case 7: return launch_np<7>(S, w, d_nactive, grid_n, out, rows, nsteps, dt, step0, QL, st);
    case 8: return launch_np<8>(S, w, d_nactive, grid_n, out, rows, nsteps, dt, step0, QL, st);
    default: return hipErrorInvalidValue;
  }
}

// ---------------------------------------------------------------- ephemeris
// The planet map is a serial chain in time, so this kernel is written for
// latency: one wavefront, lane b (1..NP) holds Jacobi body b, lane 0 the
// central body.  Values every lane needs are broadcast with v_readlane into
// scalar registers (no LDS round trip), and everything per step is branch-free
// except the general form of the planets' Kepler drifts.

// Value of v on lane `src` (a compile-time constant), returned wave-uniform
// in an SGPR pair.
TPM_DEV double bcast(double v, int src) {
  uint64_t u = __builtin_bit_cast(uint64_t, v);
  uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, src);
  uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), src);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Value of v on lane SRC (below 16) on every lane of each row of 16, by a DPP
// row broadcast (row_newbcast) into a VGPR.  The planet map's bodies sit in
// lanes 0..8, and its other lanes' values are never used: lanes 16..63 then
// carry garbage (NaN included), which every wave-wide test of the planet map
// masks by the lane's idle flag.
template <int SRC>
TPM_DEV double bcast_row(double v) {
  static_assert(SRC >= 0 && SRC < 16, "row broadcast source");
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x150 + SRC, 0xF,
                                                             0xF, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32),
                                                             0x150 + SRC, 0xF, 0xF, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// The planet map's broadcast of lane src's value.  The single-system map (a
// lone wavefront) reads it into SGPRs, since its FMAs run faster with a scalar
// operand; the many-system map, one wavefront per system, broadcasts it in
// VGPRs, which frees the SGPRs it otherwise spills (3% faster there).
template <bool ROWB>
TPM_DEV double eph_bcast(double v, int src) {
  if (!ROWB) return bcast(v, src);
  switch (src) {
    case 0: return bcast_row<0>(v);
    case 1: return bcast_row<1>(v);
    case 2: return bcast_row<2>(v);
    case 3: return bcast_row<3>(v);
    case 4: return bcast_row<4>(v);
    case 5: return bcast_row<5>(v);
    case 6: return bcast_row<6>(v);
    case 7: return bcast_row<7>(v);
    default: return bcast_row<8>(v);
  }
}

// Heliocentric positions of bodies 0..NP (body 0 at the origin) from the
// Jacobi positions held by lanes 1..NP.  The barycentre of bodies 0..b is
// R_b = R_{b-1} + (mu_b/eta_b) r'_b, so
//   r_b = r'_b + R_{b-1} = r'_b + sum_{k<b} (mu_k/eta_k) r'_k:
// the broadcasts are independent and the chain is one FMA per body.  The
// results are wave-uniform.
template <int NP>
TPM_DEV void helio_all(const EphConst& E, double jx, double jy, double jz,
                       double (&hx)[NP + 1], double (&hy)[NP + 1], double (&hz)[NP + 1]) {
  double Rx = 0.0, Ry = 0.0, Rz = 0.0;
  hx[0] = 0.0; hy[0] = 0.0; hz[0] = 0.0;
#pragma unroll
  for (int b = 1; b <= NP; ++b) {
    const double px = bcast(jx, b), py = bcast(jy, b), pz = bcast(jz, b);
    hx[b] = px + Rx; hy[b] = py + Ry; hz[b] = pz + Rz;
    Rx = fma_(E.cj[b], px, Rx);
    Ry = fma_(E.cj[b], py, Ry);
    Rz = fma_(E.cj[b], pz, Rz);
  }
}

// Per-lane constants of the planet map.
struct EphLane {
  int lane;
  bool body;
  double mup, ie_prev;            // mu'_b, 1/eta_{b-1} (0 on lanes that hold no body)
  double kc;                      // coefficient of the kick's Kepler term (see eph_accel)
  double cw;                      // weight of the central term in the lane's own kick
  double nb;                      // 0 on body lanes, 1 elsewhere (keeps an rsqrt finite)
  double c15;                     // 1.5 (held in a VGPR by the single-system map)
  double dt;                      // the step, 0 on lanes that hold no body
  KepConst K;                     // Kepler constant mu'_b for the drift
};

// Per-lane weights that turn the lane-dependent parts of a step into plain
// FMAs (no selects on the lane index inside the step loop).
template <int NP>
struct EphW {
  double cjv[NP + 1];    // mu_k/eta_k on every lane (see eph_weights)
  double wr[NP + 1];     // mu_k/eta_k for 1 <= k < lane, else 0 (own heliocentric position)
  double wa[NP + 1];     // mu_k for k < lane, else 0 (sum_{k<b} mu_k a_k)
  double mul[NP + 1];    // mu_l, 0 for the lane's own body
  double self[NP + 1];   // 1 for the lane's own body, else 0
  double hill2[NP + 1];  // squared mutual Hill radius with body j > lane, else 0
};

// HOLD: the constants that meet a broadcast in one instruction are held in
// VGPRs (the single-system map, whose broadcasts are scalar); the many-system
// map broadcasts into VGPRs and keeps them as they are.
template <int NP, bool HOLD>
TPM_DEV EphW<NP> eph_weights(const EphConst& E, int lane) {
  EphW<NP> W;
#pragma unroll
  for (int k = 0; k <= NP; ++k) {
    W.cjv[k] = HOLD ? vgpr_held(E.cj[k]) : E.cj[k];
    W.wr[k] = (k >= 1 && k < lane) ? E.cj[k] : 0.0;
    W.wa[k] = (k < lane) ? E.mu[k] : 0.0;
    W.mul[k] = (k == lane) ? 0.0 : E.mu[k];
    W.self[k] = (k == lane) ? 1.0 : 0.0;
    W.hill2[k] = 0.0;
  }
#pragma unroll
  for (int b = 1; b <= NP; ++b)
#pragma unroll
    for (int j = b + 1; j <= NP; ++j)
      if (lane == b) W.hill2[j] = E.hill2[b][j];
  return W;
}

// The lane's own heliocentric position r'_b + R_{b-1} from the broadcast
// Jacobi positions (the same bits as helio_all's entry for body b; 0 on lane
// 0).
template <int NP>
TPM_DEV void own_helio(const EphW<NP>& W, double jx, double jy, double jz,
                       const double (&px)[NP + 1], const double (&py)[NP + 1],
                       const double (&pz)[NP + 1], double& ox, double& oy, double& oz) {
  double Rx = 0.0, Ry = 0.0, Rz = 0.0;
#pragma unroll
  for (int k = 1; k <= NP; ++k) {
    Rx = fma_(W.wr[k], px[k], Rx);
    Ry = fma_(W.wr[k], py[k], Ry);
    Rz = fma_(W.wr[k], pz[k], Rz);
  }
  ox = jx + Rx; oy = jy + Ry; oz = jz + Rz;
}

// Heliocentric positions of all bodies and the lane's own one, from the Jacobi
// positions held by lanes 1..NP (see helio_all).
template <int NP, bool ROWB>
TPM_DEV void helio_step(const EphConst& E, const EphW<NP>& W, double jx, double jy, double jz,
                        double (&hx)[NP + 1], double (&hy)[NP + 1], double (&hz)[NP + 1],
                        double& ox, double& oy, double& oz) {
  double px[NP + 1], py[NP + 1], pz[NP + 1];
  double Rx = 0.0, Ry = 0.0, Rz = 0.0;
  hx[0] = 0.0; hy[0] = 0.0; hz[0] = 0.0;
  px[0] = 0.0; py[0] = 0.0; pz[0] = 0.0;
#pragma unroll
  for (int b = 1; b <= NP; ++b) {
    px[b] = eph_bcast<ROWB>(jx, b); py[b] = eph_bcast<ROWB>(jy, b); pz[b] = eph_bcast<ROWB>(jz, b);
    hx[b] = px[b] + Rx; hy[b] = py[b] + Ry; hz[b] = pz[b] + Rz;
    Rx = fma_(W.cjv[b], px[b], Rx);
    Ry = fma_(W.cjv[b], py[b], Ry);
    Rz = fma_(W.cjv[b], pz[b], Rz);
  }
  own_helio<NP>(W, jx, jy, jz, px, py, pz, ox, oy, oz);
}

// Interaction acceleration of the lane's Jacobi body (lanes 1..NP):
//   a'_b = a_b - (sum_{k<b} mu_k a_k)/eta_{b-1} + mu'_b r'_b/|r'_b|^3,
// with a_k the Newtonian acceleration of body k; lane 0 gets a_0 (h0 = -a_0).
// (ox, oy, oz) is the lane's own heliocentric position.  For the innermost
// body the heliocentric and Jacobi vectors are the same (bit for bit), so its
// central term -mu_0 r/|r|^3 and the Kepler term combine into
// (mu'_1 - mu_0) r/|r|^3: kc holds that difference (exact in floating point,
// the two coefficients being within a factor two) and cw = 0 drops the
// central term from the lane's own sum.  The two terms would otherwise cancel
// to about mu_1/mu_0 of their size and amplify their rounding by mu_0/mu_1.
// The broadcast a_1 keeps its central term.
template <int NP, bool ROWB>
TPM_DEV void eph_accel(const EphConst& E, const EphLane& L, const EphW<NP>& W, double jx,
                       double jy, double jz, const double (&hx)[NP + 1],
                       const double (&hy)[NP + 1], const double (&hz)[NP + 1], double ox,
                       double oy, double oz, double& ax, double& ay, double& az) {
  // the planets' pulls (l >= 1), then the central body's (l = 0, at the origin)
  double px = 0.0, py = 0.0, pz = 0.0;
#pragma unroll
  for (int l = 1; l <= NP; ++l) {
    double dx = ox - hx[l], dy = oy - hy[l], dz = oz - hz[l];
    double d2 = fma_(dx, dx, fma_(dy, dy, dz * dz));
    double k = mul_rsqrt3(W.mul[l], d2 + W.self[l], L.c15);
    px = fma_(-k, dx, px);
    py = fma_(-k, dy, py);
    pz = fma_(-k, dz, pz);
  }
  const double k0 = mul_rsqrt3(W.mul[0], fma_(ox, ox, fma_(oy, oy, oz * oz)) + W.self[0], L.c15);
  const double nx = fma_(-k0, ox, px), ny = fma_(-k0, oy, py), nz = fma_(-k0, oz, pz);
  // sum_{k<b} mu_k a_k from the broadcast Newtonian accelerations
  double sx = 0.0, sy = 0.0, sz = 0.0;
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    sx = fma_(W.wa[k], eph_bcast<ROWB>(nx, k), sx);
    sy = fma_(W.wa[k], eph_bcast<ROWB>(ny, k), sy);
    sz = fma_(W.wa[k], eph_bcast<ROWB>(nz, k), sz);
  }
  double r2 = fma_(jx, jx, fma_(jy, jy, jz * jz));
  double kk = mul_rsqrt3(L.kc, r2 + L.nb, L.c15);
  const double kw = k0 * L.cw;
  // lane 0: jx = ie_prev = 0, so a = n
  ax = fma_(kk, jx, fma_(-sx, L.ie_prev, fma_(-kw, ox, px)));
  ay = fma_(kk, jy, fma_(-sy, L.ie_prev, fma_(-kw, oy, py)));
  az = fma_(kk, jz, fma_(-sz, L.ie_prev, fma_(-kw, oz, pz)));
}

// Any pair (lane, j > lane) closer than their mutual Hill radius.
template <int NP>
TPM_DEV bool hill_violation(const EphW<NP>& W, double ox, double oy, double oz,
                            const double (&hx)[NP + 1], const double (&hy)[NP + 1],
                            const double (&hz)[NP + 1]) {
  bool bad = false;
#pragma unroll
  for (int j = 2; j <= NP; ++j) {
    double dx = ox - hx[j], dy = oy - hy[j], dz = oz - hz[j];
    double d2 = fma_(dx, dx, fma_(dy, dy, dz * dz));
    bad = bad || (d2 < W.hill2[j]);
  }
  return bad;
}

// The planet map's kernels keep the two-address FP64 FMA (v_fmac_f64), which
// the library's build otherwise turns off: its lone wavefront runs faster with
// the shorter encoding, the particle kernels without the copies it costs.
// (A device-code attribute: the host pass of the same source does not know it.)
#if defined(__HIP_DEVICE_COMPILE__)
#define TPM_PLANET_KERNEL __attribute__((target("fmacf64-inst")))
#else
#define TPM_PLANET_KERNEL
#endif

// Heliocentric velocities of the planets (internal order, [NP][3]) from the
// Jacobi velocities held by lanes 1..NP: the same linear map as the
// positions'.  Wave-uniform call.
template <int NP, bool ROWB>
TPM_DEV void write_helio_velocities(const EphConst& E, const EphW<NP>& W, bool body, int lane,
                                    double wx, double wy, double wz, double* __restrict__ out) {
  double hx[NP + 1], hy[NP + 1], hz[NP + 1];
  double ox, oy, oz;
  helio_step<NP, ROWB>(E, W, wx, wy, wz, hx, hy, hz, ox, oy, oz);
  if (body) {
    out[3 * (lane - 1) + 0] = ox;
    out[3 * (lane - 1) + 1] = oy;
    out[3 * (lane - 1) + 2] = oz;
  }
}

// One step of the planet map (sec. 2.2, planet integration: kick, Jacobi
// drift, kick), from the Jacobi state (j, w) and the interaction acceleration
// a at it; writes table row `row` (this lane's entry).  key1 = 2t for step
// t of the launch: the general form (FAST false) keeps the first event as a
// key ordered in time (see ephemeris_body); the fast form returns instead
// whether the lane would have taken another path than its own (the general
// drift's branches), or, with events on, met an event at all.
template <int NP, bool ROWB, bool FAST, bool VEL>
TPM_DEV bool eph_step(const EphConst& E, const EphLane& L, const EphW<NP>& W, double h, double dt,
                      double& jx, double& jy, double& jz, double& wx, double& wy, double& wz,
                      double& ax, double& ay, double& az, bool writer, double rsign,
                      double* __restrict__ row, double* __restrict__ vrow, uint32_t key1,
                      bool events, uint32_t& first_ev) {
  double hx[NP + 1], hy[NP + 1], hz[NP + 1];
  double ox, oy, oz;
  wx = fma_(h, ax, wx); wy = fma_(h, ay, wy); wz = fma_(h, az, wz);
  bool bad;
  const bool bound =
      planet_drift<FAST>(L.K, L.dt, L.body, L.nb, jx, jy, jz, wx, wy, wz, bad);
  if (!FAST) first_ev = __builtin_elementwise_min(first_ev, (L.body && !bound) ? key1 : UINT32_MAX);
  helio_step<NP, ROWB>(E, W, jx, jy, jz, hx, hy, hz, ox, oy, oz);
  eph_accel<NP, ROWB>(E, L, W, jx, jy, jz, hx, hy, hz, ox, oy, oz, ax, ay, az);
  wx = fma_(h, ax, wx); wy = fma_(h, ay, wy); wz = fma_(h, az, wz);
  if (writer) {
    row[0] = fma_(rsign, ax, ox);
    row[1] = fma_(rsign, ay, oy);
    row[2] = fma_(rsign, az, oz);
  }
  if (NP > 1) {
    const bool close = hill_violation<NP>(W, ox, oy, oz, hx, hy, hz);
    if (FAST) bad = bad | (events & close);
    else first_ev = __builtin_elementwise_min(first_ev, close ? key1 + 1u : UINT32_MAX);
  }
  if (VEL) write_helio_velocities<NP, ROWB>(E, W, L.body, L.lane, wx, wy, wz, vrow);
  return bad;
}

// Steps of one fast block (see ephemeris_body), and what ephemeris_body calls
// after each block of steps: here nothing to do, go on.
constexpr int EPH_BLOCK = 64;
struct EphNoBlockEnd {
  TPM_DEV int block(int, int left) const { return min(left, EPH_BLOCK); }
  TPM_DEV bool operator()(int) const { return true; }
};

// vside (may be null): receives the planets' heliocentric velocities at the
// chunk's first and last rows, [2][NP][3] (for the sampled diagnostics).
// VEL: vrows receives them at every row, [nsteps+1][NP][3] (for the
// encounter integrator).
// resumed: row 0 (and vside's first entry) was written by the call that
// stopped there and is left alone.  block_end(t) is called once rows 1..t are
// final and says whether to go on; the return value is the steps carried out
// (vside's second entry is written only if that is all of them).
template <int NP, bool ROWB, bool VEL = false, typename BlockEnd = EphNoBlockEnd>
TPM_DEV int ephemeris_body(const EphConst& E, double* __restrict__ rj, double* __restrict__ vj,
                           double* __restrict__ rows, int nsteps, double dt, int64_t step0,
                           int64_t* __restrict__ flag, double* __restrict__ vside = nullptr,
                           double* __restrict__ vrows = nullptr, bool resumed = false,
                           BlockEnd block_end = BlockEnd()) {
  constexpr int ROW = 3 * NP + 3;
  // This wave is a serial chain that shares its SIMD with particle waves:
  // let it issue first.
  __builtin_amdgcn_s_setprio(3);
  EphLane L;
  L.lane = threadIdx.x & 63;
  L.body = L.lane >= 1 && L.lane <= NP;
  L.mup = 1.0; L.ie_prev = 0.0; L.nb = L.body ? 0.0 : 1.0;
  L.dt = L.body ? dt : 0.0;
#pragma unroll
  for (int b = 1; b <= NP; ++b)
    if (L.lane == b) { L.mup = E.mup[b]; L.ie_prev = E.inv_eta[b - 1]; }
  L.kc = L.mup;
  L.cw = 1.0;
  L.c15 = ROWB ? 1.5 : vgpr_held(1.5);
  if (NP >= 1 && L.lane == 1) {
    L.kc = E.mup[1] - E.mu[0];
    L.cw = 0.0;
  }
  const EphW<NP> W = eph_weights<NP, !ROWB>(E, L.lane);
  {
    double smu, rsmu;
    sqrt_rsqrt(L.mup, smu, rsmu);
    L.K = KepConst{L.mup, rcp(L.mup), smu, rsmu};
  }
  double jx = 0, jy = 0, jz = 0, wx = 0, wy = 0, wz = 0;
  double hx[NP + 1], hy[NP + 1], hz[NP + 1];
  double ox, oy, oz, ax, ay, az;
  // the state from and to memory, and the acceleration at it (the same bits as
  // the one carried on)
  auto get_state = [&]() {
    jx = jy = jz = wx = wy = wz = 0.0;
    if (L.body) {
      jx = rj[3 * (L.lane - 1) + 0]; jy = rj[3 * (L.lane - 1) + 1]; jz = rj[3 * (L.lane - 1) + 2];
      wx = vj[3 * (L.lane - 1) + 0]; wy = vj[3 * (L.lane - 1) + 1]; wz = vj[3 * (L.lane - 1) + 2];
    }
    helio_step<NP, ROWB>(E, W, jx, jy, jz, hx, hy, hz, ox, oy, oz);
    eph_accel<NP, ROWB>(E, L, W, jx, jy, jz, hx, hy, hz, ox, oy, oz, ax, ay, az);
  };
  auto put_state = [&]() {
    if (L.body) {
      rj[3 * (L.lane - 1) + 0] = jx; rj[3 * (L.lane - 1) + 1] = jy; rj[3 * (L.lane - 1) + 2] = jz;
      vj[3 * (L.lane - 1) + 0] = wx; vj[3 * (L.lane - 1) + 1] = wy; vj[3 * (L.lane - 1) + 2] = wz;
    }
  };
  get_state();
  // Row entries: lane b writes planet b's heliocentric position, lane 0 (the
  // central body, whose own position is the origin) writes h0 = -a_0, both as
  // fma(rsign, a, o) with rsign = 0 on body lanes and -1 on lane 0.
  const bool writer = L.lane <= NP;
  const int roff = L.body ? 3 * (L.lane - 1) : 3 * NP;
  const double rsign = L.body ? 0.0 : -1.0;
  // row 0: the current state
  if (writer && !resumed) {
    rows[roff + 0] = fma_(rsign, ax, ox);
    rows[roff + 1] = fma_(rsign, ay, oy);
    rows[roff + 2] = fma_(rsign, az, oz);
  }
  const double h = 0.5 * dt;
  // Per lane, the first event as a key ordered in time, counted from step0: a
  // close pair seen at step step0 + t has key 2t+1; an orbit found unbound
  // while drifting from step0 + t - 1 to step0 + t has key 2t, so it wins a tie
  // with a close pair at that step (it is found first).  Keys grow with t, so
  // the first event is the smallest key.
  uint32_t first_ev = UINT32_MAX;
  if (NP > 1 && hill_violation<NP>(W, ox, oy, oz, hx, hy, hz)) first_ev = 1u;
  if (vside && !resumed)
    write_helio_velocities<NP, ROWB>(E, W, L.body, L.lane, wx, wy, wz, vside);
  if (VEL && !resumed) write_helio_velocities<NP, ROWB>(E, W, L.body, L.lane, wx, wy, wz, vrows);
  // Blocks of steps.  Planets on near-circular orbits are served by planet_quick
  // every time and meet no event; the fast form runs exactly that, with none of
  // the general form's wave-uniform branches, and only notes on each lane
  // whether the general form would have done otherwise.  A block in which any
  // lane did is restored from its start and run again in the general form, as is
  // the rest of the launch.  Either way the rows and the state are the general
  // form's bit for bit.  Once the run's first event is on record (*flag != -1) a
  // close pair cannot change it and no longer stops the fast form.  (The
  // many-system map keeps the general form: its wavefronts share SIMDs with the
  // particles, which hide its branches.)
  // A block's start is kept in memory: in registers it took eighteen more
  // through the fast loop, which with eight planets then no longer fits the 256
  // of a particle launch's wavefront (nine reloads a step: 1.83 us a step where
  // the map as a kernel of its own took 1.35).  So and with planet_quick 0.95, 1.06,
  // 1.11 and 1.26 us a step at five to eight planets (1.03, 1.13, 1.32, 1.83 before).
  const bool events = *flag == -1;
  bool fast = !ROWB;
  int done = 0;
  while (done < nsteps) {
    const int s0 = done;
    const int nb = ROWB ? nsteps : block_end.block(s0, nsteps - s0);
    done = s0 + nb;
    if (!ROWB && fast) {
      put_state();
      bool bad = false;
      for (int t = 0; t < nb; ++t) {
        const int s = s0 + t;
        bad = bad | eph_step<NP, ROWB, true, VEL>(
                        E, L, W, h, dt, jx, jy, jz, wx, wy, wz, ax, ay, az, writer, rsign,
                        rows + (size_t)(s + 1) * ROW + roff,
                        VEL ? vrows + (size_t)(s + 1) * 3 * NP : nullptr, 2u * (uint32_t)(s + 1),
                        events, first_ev);
      }
      if (wave_all(!bad)) {
        if (!block_end(done)) break;
        continue;
      }
      get_state();
      fast = false;
    }
    for (int t = 0; t < nb; ++t) {
      const int s = s0 + t;
      eph_step<NP, ROWB, false, VEL>(E, L, W, h, dt, jx, jy, jz, wx, wy, wz, ax, ay, az, writer,
                                     rsign, rows + (size_t)(s + 1) * ROW + roff,
                                     VEL ? vrows + (size_t)(s + 1) * 3 * NP : nullptr,
                                     2u * (uint32_t)(s + 1), events, first_ev);
    }
    if (!block_end(done)) break;
  }
  if (vside && done == nsteps)
    write_helio_velocities<NP, ROWB>(E, W, L.body, L.lane, wx, wy, wz, vside + 3 * NP);
  put_state();
  // earliest event over the wavefront: unbound -> -2, a close pair -> its step
  uint32_t ev = first_ev;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    uint32_t o = __shfl_xor(ev, off, 64);
    ev = o < ev ? o : ev;
  }
  if (L.lane == 0 && *flag == -1 && ev != UINT32_MAX)
    *flag = (ev & 1u) ? step0 + (int64_t)(ev >> 1) : -2;
  return done;
}

template <bool FAST>
struct FormTag { static constexpr bool value = FAST; };

// ephemeris_body for one to four planets, in the layout of planet_quad.hpp
// (same arguments and results to rounding; E is read per lane, once).  Blocks
// as there: the fast form, or the general form from the first block a lane
// could not take fast.  A body found unbound stays out of the fast form.
template <int NP, bool VEL, typename EP, typename BlockEnd = EphNoBlockEnd>
TPM_DEV int ephemeris_quad(EP E, double* __restrict__ rj, double* __restrict__ vj,
                           double* __restrict__ rows, int nsteps, double dt, int64_t step0,
                           int64_t* __restrict__ flag, double* __restrict__ vside = nullptr,
                           double* __restrict__ vrows = nullptr, bool resumed = false,
                           BlockEnd block_end = BlockEnd()) {
  constexpr int ROW = 3 * NP + 3;
  __builtin_amdgcn_s_setprio(3);   // a serial chain among particle wavefronts
  const int lane = threadIdx.x & 63;
  const EphQuad Q = eph_quad<NP>(E, dt, lane);
  // block 0 holds the state and the heliocentric positions, component 3 none
  const bool writer = Q.on && (lane & 12) == 0 && Q.col < 3;
  const bool writer0 = lane < 3;
  const int at = 3 * Q.body + Q.col;
  double j = 0.0, w = 0.0;
  if (Q.on && Q.col < 3) {
    j = rj[at];
    w = vj[at];
  } else if (!Q.on) {
    j = Q.col == 0 ? 1.0 : 0.0;      // the stand-in orbit of planet_fg
    w = Q.col == 1 ? 1.0 : 0.0;
  }
  auto put_row = [&](double* row, double d, double h0) {
    if (writer) row[at] = d;
    if (writer0) row[3 * NP + lane] = h0;
  };
  auto put_velocities = [&](double* out) {
    const double hv = mfma4(Q.pos, w);
    if (writer) out[at] = hv;
  };
  double d, a, h0;
  const bool close0 = quad_accel(Q, j, d, a, h0);
  if (!resumed) {
    put_row(rows, d, h0);
    if (vside) put_velocities(vside);
    if (VEL) put_velocities(vrows);
  }
  const double h = 0.5 * dt;
  uint32_t first_ev = close0 ? 1u : UINT32_MAX;
  auto step = [&](auto fast_c, int s) {
    constexpr bool FAST = decltype(fast_c)::value;
    bool bad;
    w = fma_(h, a, w);
    const bool bound = quad_drift<FAST>(Q, j, w, bad);
    const bool close = quad_accel(Q, j, d, a, h0);
    w = fma_(h, a, w);
    put_row(rows + (size_t)s * ROW, d, h0);
    if (VEL) put_velocities(vrows + (size_t)s * 3 * NP);
    if (!FAST) {
      const uint32_t key = 2u * (uint32_t)s;
      first_ev = __builtin_elementwise_min(first_ev, Q.on && !bound ? key : UINT32_MAX);
      first_ev = __builtin_elementwise_min(first_ev, close ? key + 1u : UINT32_MAX);
    }
    return FAST ? bad | (NP > 1 && close) : false;
  };
  // Once the run's first event is on record later ones cannot change it, but a
  // close pair still ends the fast form: the general one is as right.
  bool fast = true;
  int done = 0;
  while (done < nsteps) {
    const int s0 = done;
    const int nb = block_end.block(s0, nsteps - s0);
    done = s0 + nb;
    if (fast) {
      const double sj = j, sw = w, sa = a;
      bool bad = false;
      for (int t = 1; t <= nb; ++t) bad = bad | step(FormTag<true>{}, s0 + t);
      if (wave_all(!bad)) {
        if (!block_end(done)) break;
        continue;
      }
      j = sj; w = sw; a = sa;
      fast = false;
    }
    for (int t = 1; t <= nb; ++t) step(FormTag<false>{}, s0 + t);
    if (!block_end(done)) break;
  }
  if (vside && done == nsteps) put_velocities(vside + 3 * NP);
  if (writer) {
    rj[at] = j;
    vj[at] = w;
  }
  // earliest event over the wavefront: unbound -> -2, a close pair -> its step
  uint32_t ev = first_ev;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    uint32_t o = __shfl_xor(ev, off, 64);
    ev = o < ev ? o : ev;
  }
  if (lane == 0 && *flag == -1 && ev != UINT32_MAX)
    *flag = (ev & 1u) ? step0 + (int64_t)(ev >> 1) : -2;
  return done;
}

// The planet map of NP planets: one to four by matrix instructions.
template <int NP, bool ROWB, bool VEL, typename EP, typename BlockEnd = EphNoBlockEnd>
TPM_DEV int planet_map(EP E, double* rj, double* vj, double* rows, int nsteps, double dt,
                       int64_t step0, int64_t* flag, double* vside = nullptr,
                       double* vrows = nullptr, bool resumed = false,
                       BlockEnd block_end = BlockEnd()) {
  if constexpr (NP >= 1 && NP <= 4) {
    return ephemeris_quad<NP, VEL>(E, rj, vj, rows, nsteps, dt, step0, flag, vside, vrows, resumed,
                                   block_end);
  } else {
    const EphConst C = *E;
    return ephemeris_body<NP, ROWB, VEL>(C, rj, vj, rows, nsteps, dt, step0, flag, vside, vrows,
                                         resumed, block_end);
  }
}

// The row stream's blocks: what the particles of the same launch follow the
// map by.  They end where rows fill cache lines (see wait_rows), at counts one
// short of a multiple of ROW_GROUP: 15 steps, then 16 or 32, about a quarter of
// those to go.  A block's end costs the map about a microsecond (1.16 us a step at
// six planets, 1.15 with blocks of up to 64), but particles about as fast as the map
// wait once for the steps by which a block is longer than the one before: with
// blocks of up to 64, 500 steps of one planet took 446 us for 434.  After each the
// count of published steps goes up; a map that runs ahead of its launch's chunk
// stops once no other wavefront of the launch is at work.
struct EphPublish {
  const RowStream& R;
  int64_t done;                              // the count when the body started
  bool ahead;
  int first;                                 // the chunk's step the body started from
  // Steps of the block after `s` of the body's.
  TPM_DEV int block(int s, int left) const {
    const int c = first + s;
    const int want = c == 0 ? ROW_GROUP : max(ROW_GROUP, min(2 * ROW_GROUP, left >> 2));
    int nb = (c + want + 1) / ROW_GROUP * ROW_GROUP - 1 - c;
    if (nb <= 0) nb += ROW_GROUP;
    return min(left, nb);
  }
  TPM_DEV bool operator()(int t) const {
    // the release makes the rows written so far visible before the count
    __hip_atomic_store(R.done, done + t, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    if (!ahead) return true;
    const unsigned long long c = wave_uniform(
        __hip_atomic_load(R.ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    return c - R.ctr_base < R.ctr_alone;     // others still at work
  }
};

// The planet map of a particle launch (see particle_queue), run by the one
// wavefront that took the launch's first work item: publishes the rows of the
// launch's chunk block by block, then goes on into the following chunks'
// slots for as long as other wavefronts of the launch are at work, so the
// next launch finds rows to start from.  A function of its own, not inlined:
// it has the planet map's instruction choice (TPM_PLANET_KERNEL) and its own
// registers.  ka_any: the launch's argument segment (in VGPRs by the calling
// convention, wave-uniform).
template <int NP, bool VEL>
static __device__ __attribute__((noinline)) TPM_PLANET_KERNEL void planet_rows(uint64_t ka_any) {
  constexpr int ROW = 3 * NP + 3;
  const KargPtr ka = (KargPtr)wave_uniform(ka_any);
  const RowStream R = karg_stream<RowStream>(ka, 0);
  const auto E = karg_pointer<EphConst>(ka, offsetof(QueueKernelArgs<NP>, E));
  const unsigned long long t0 = __builtin_readsteadycounter();
  int64_t done = (int64_t)wave_uniform((unsigned long long)__hip_atomic_load(
      R.done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  int64_t b = R.begin;                       // first step of chunk j
  for (int j = 0; j < STREAM_CHUNKS; ++j) {
    const int len = karg_stream<int>(ka, offsetof(RowStream, len) + sizeof(int) * j);
    if (len <= 0) break;
    if (done >= b + len) {                   // an earlier launch's map ran ahead
      b += len;
      continue;
    }
    const int s0 = (int)(done - b);
    const int64_t slot = (R.slot0 + j) % R.nslots;
    const int n = planet_map<NP, false, VEL>(
        E, R.rj, R.vj, R.ring + (size_t)(slot * R.slot_rows + s0) * ROW, len - s0, R.dt,
        R.step0 + (b - R.begin) + s0, R.flag,
        R.vside ? R.vside + (size_t)slot * 6 * NP : nullptr,
        VEL ? R.vring + (size_t)(slot * R.vslot_rows + s0) * 3 * NP : nullptr, s0 > 0,
        EphPublish{R, done, j > 0, s0});
    done += n;
    if (n < len - s0) break;
    b += len;
  }
  __builtin_amdgcn_s_setprio(0);
  if ((threadIdx.x & 63) == 0) *R.ticks += __builtin_readsteadycounter() - t0;
}

template <int NP>
TPM_DEV void run_planet_rows(KargPtr ka) {
  const uint64_t p = (uint64_t)ka;
  if (karg_stream<double*>(ka, offsetof(RowStream, vring))) planet_rows<NP, true>(p);
  else planet_rows<NP, false>(p);
}

template <int NP>
__global__ void __launch_bounds__(64) TPM_PLANET_KERNEL
ephemeris_chunk(EphConst E, double* __restrict__ rj, double* __restrict__ vj,
                double* __restrict__ rows, int nsteps, double dt, int64_t step0,
                int64_t* __restrict__ flag, double* __restrict__ vside) {
  (void)E;                           // the first argument, read from the argument segment
  planet_map<NP, false, false>(
      karg_pointer<EphConst>((KargPtr)__builtin_amdgcn_kernarg_segment_ptr(), 0), rj, vj, rows,
      nsteps, dt, step0, flag, vside);
}

// Many systems at once: workgroup b runs system b (its constants, Jacobi
// state, table rows and flag are found through the per-system arrays).
__global__ void __launch_bounds__(64) TPM_PLANET_KERNEL
ephemeris_batch(const EphConst* __restrict__ E, double* __restrict__ rj, double* __restrict__ vj,
                double* __restrict__ ring, const int64_t* __restrict__ ring_off, int slot,
                int64_t slot_stride_rows, int nsteps, const double* __restrict__ dt,
                int64_t step0, int64_t* __restrict__ flag) {
  const int b = blockIdx.x;
  const EphConst& e = E[b];
  double* rows = ring + ring_off[b] + (int64_t)slot * slot_stride_rows * (3 * e.np + 3);
  double* r = rj + 3 * MAX_NP * b;
  double* v = vj + 3 * MAX_NP * b;
  switch (e.np) {
    case 1: planet_map<1, true, false>(&e, r, v, rows, nsteps, dt[b], step0, flag + b); break;
    case 2: planet_map<2, true, false>(&e, r, v, rows, nsteps, dt[b], step0, flag + b); break;
    case 3: planet_map<3, true, false>(&e, r, v, rows, nsteps, dt[b], step0, flag + b); break;
    case 4: planet_map<4, true, false>(&e, r, v, rows, nsteps, dt[b], step0, flag + b); break;
    case 5: planet_map<5, true, false>(&e, r, v, rows, nsteps, dt[b], step0, flag + b); break;
    case 6: planet_map<6, true, false>(&e, r, v, rows, nsteps, dt[b], step0, flag + b); break;
    case 7: planet_map<7, true, false>(&e, r, v, rows, nsteps, dt[b], step0, flag + b); break;
    case 8: planet_map<8, true, false>(&e, r, v, rows, nsteps, dt[b], step0, flag + b); break;
    default: planet_map<0, true, false>(&e, r, v, rows, nsteps, dt[b], step0, flag + b); break;
  }
}

// The planet map's event keys count the steps of one launch in 32 bits.
constexpr int MAX_EPH_STEPS = 1 << 30;

hipError_t launch_ephemeris_batch(const EphConst* E, double* rj, double* vj, double* ring,
                                  const int64_t* ring_off, int slot, int64_t slot_stride_rows,
                                  int nsys, int nsteps, const double* dt, int64_t step0,
                                  int64_t* flag, hipStream_t st) {
  if (nsteps < 0 || nsteps > MAX_EPH_STEPS) return hipErrorInvalidValue;
  if (nsys <= 0) return hipSuccess;
  hipLaunchKernelGGL(ephemeris_batch, dim3(nsys), dim3(64), 0, st, E, rj, vj, ring, ring_off, slot,
                     slot_stride_rows, nsteps, dt, step0, flag);
  return hipGetLastError();
}

template <int NP>
static hipError_t eph_np(const EphConst& E, double* rj, double* vj, double* rows, int nsteps,
                         double dt, int64_t step0, int64_t* flag, double* vside, hipStream_t st) {
  hipLaunchKernelGGL((ephemeris_chunk<NP>), dim3(1), dim3(64), 0, st, E, rj, vj, rows, nsteps, dt,
                     step0, flag, vside);
  return hipGetLastError();
}

hipError_t launch_ephemeris_chunk(const EphConst& E, double* rj, double* vj, double* rows,
                                  int nsteps, double dt, int64_t step0, int64_t* flag,
                                  hipStream_t st, double* vside) {
  if (nsteps < 0 || nsteps > MAX_EPH_STEPS) return hipErrorInvalidValue;
  switch (E.np) {
#define TPM_EPH(N) \
    case N: return eph_np<N>(E, rj, vj, rows, nsteps, dt, step0, flag, vside, st);
    TPM_EPH(0) TPM_EPH(1) TPM_EPH(2) TPM_EPH(3) TPM_EPH(4) TPM_EPH(5) TPM_EPH(6) TPM_EPH(7)
    TPM_EPH(8)
#undef TPM_EPH
    default: return hipErrorInvalidValue;
  }
}

// Jacobi -> heliocentric positions and velocities of the planets (one wave).
template <int NP>
__global__ void __launch_bounds__(64)
jacobi_to_helio_kernel(EphConst E, const double* rj, const double* vj, double* rh, double* vh) {
  const int lane = threadIdx.x;
  const bool body = lane >= 1 && lane <= NP;
  double jx = 0, jy = 0, jz = 0, wx = 0, wy = 0, wz = 0;
  if (body) {
    jx = rj[3 * (lane - 1) + 0]; jy = rj[3 * (lane - 1) + 1]; jz = rj[3 * (lane - 1) + 2];
    wx = vj[3 * (lane - 1) + 0]; wy = vj[3 * (lane - 1) + 1]; wz = vj[3 * (lane - 1) + 2];
  }
  double hx[NP + 1], hy[NP + 1], hz[NP + 1];
  helio_all<NP>(E, jx, jy, jz, hx, hy, hz);
  double ux[NP + 1], uy[NP + 1], uz[NP + 1];
  helio_all<NP>(E, wx, wy, wz, ux, uy, uz);
  if (body) {
    rh[3 * (lane - 1) + 0] = hx[lane]; rh[3 * (lane - 1) + 1] = hy[lane]; rh[3 * (lane - 1) + 2] = hz[lane];
    vh[3 * (lane - 1) + 0] = ux[lane]; vh[3 * (lane - 1) + 1] = uy[lane]; vh[3 * (lane - 1) + 2] = uz[lane];
  }
}

template <int NP>
static hipError_t j2h_np(const EphConst& E, const double* rj, const double* vj, double* rh,
                         double* vh, hipStream_t st) {
  hipLaunchKernelGGL(jacobi_to_helio_kernel<NP>, dim3(1), dim3(64), 0, st, E, rj, vj, rh, vh);
  return hipGetLastError();
}

hipError_t launch_jacobi_to_helio(const EphConst& E, const double* rj, const double* vj,
                                  double* rh, double* vh, hipStream_t st) {
  switch (E.np) {
    case 0: return hipSuccess;
    case 1: return j2h_np<1>(E, rj, vj, rh, vh, st);
    case 2: return j2h_np<2>(E, rj, vj, rh, vh, st);
    case 3: return j2h_np<3>(E, rj, vj, rh, vh, st);
    case 4: return j2h_np<4>(E, rj, vj, rh, vh, st);
    case 5: return j2h_np<5>(E, rj, vj, rh, vh, st);
    case 6: return j2h_np<6>(E, rj, vj, rh, vh, st);
    case 7: return j2h_np<7>(E, rj, vj, rh, vh, st);
    case 8: return j2h_np<8>(E, rj, vj, rh, vh, st);
    default: return hipErrorInvalidValue;
  }
}


// Heliocentric -> Jacobi positions or velocities of the planets (one wave):
//   r'_b = r_b - (sum_{k=1}^{b-1} mu_k r_k) / eta_{b-1}.
template <int NP>
__global__ void __launch_bounds__(64)
helio_to_jacobi_kernel(EphConst E, const double* h, double* j) {
  const int lane = threadIdx.x;
  if (lane < 1 || lane > NP) return;
  double sx = 0.0, sy = 0.0, sz = 0.0;
  for (int k = 1; k < lane; ++k) {
    sx = fma_(E.mu[k], h[3 * (k - 1) + 0], sx);
    sy = fma_(E.mu[k], h[3 * (k - 1) + 1], sy);
    sz = fma_(E.mu[k], h[3 * (k - 1) + 2], sz);
  }
  const double ie = E.inv_eta[lane - 1];
  j[3 * (lane - 1) + 0] = fma_(-sx, ie, h[3 * (lane - 1) + 0]);
  j[3 * (lane - 1) + 1] = fma_(-sy, ie, h[3 * (lane - 1) + 1]);
  j[3 * (lane - 1) + 2] = fma_(-sz, ie, h[3 * (lane - 1) + 2]);
}

hipError_t launch_helio_to_jacobi(const EphConst& E, const double* h, double* j, hipStream_t st) {
  switch (E.np) {
    case 0: return hipSuccess;
#define TPM_H2J(N) case N: hipLaunchKernelGGL(helio_to_jacobi_kernel<N>, dim3(1), dim3(64), 0, st, E, h, j); break;
    TPM_H2J(1) TPM_H2J(2) TPM_H2J(3) TPM_H2J(4) TPM_H2J(5) TPM_H2J(6) TPM_H2J(7) TPM_H2J(8)
#undef TPM_H2J
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Heliocentric -> Jacobi for many systems: workgroup b converts system b's
// planets (arrays [nsys][MAX_NP][3]).
__global__ void __launch_bounds__(64)
helio_to_jacobi_batch(const EphConst* __restrict__ E, const double* __restrict__ h,
                      double* __restrict__ j) {
  const int b = blockIdx.x;
  const EphConst& e = E[b];
  const int lane = threadIdx.x;
  if (lane < 1 || lane > e.np) return;
  const double* hb = h + 3 * MAX_NP * b;
  double* jb = j + 3 * MAX_NP * b;
  double sx = 0.0, sy = 0.0, sz = 0.0;
  for (int k = 1; k < lane; ++k) {
    sx = fma_(e.mu[k], hb[3 * (k - 1) + 0], sx);
    sy = fma_(e.mu[k], hb[3 * (k - 1) + 1], sy);
    sz = fma_(e.mu[k], hb[3 * (k - 1) + 2], sz);
  }
  const double ie = e.inv_eta[lane - 1];
  jb[3 * (lane - 1) + 0] = fma_(-sx, ie, hb[3 * (lane - 1) + 0]);
  jb[3 * (lane - 1) + 1] = fma_(-sy, ie, hb[3 * (lane - 1) + 1]);
  jb[3 * (lane - 1) + 2] = fma_(-sz, ie, hb[3 * (lane - 1) + 2]);
}

hipError_t launch_helio_to_jacobi_batch(const EphConst* E, const double* h, double* j, int nsys,
                                        hipStream_t st) {
  if (nsys <= 0) return hipSuccess;
  hipLaunchKernelGGL(helio_to_jacobi_batch, dim3(nsys), dim3(64), 0, st, E, h, j);
  return hipGetLastError();
}

// Steps particle i spent active in [step_begin, step_end) (d: its removal step).
TPM_DEV int64_t active_steps(int64_t d, int64_t step_begin, int64_t step_end) {
  const int64_t lo = step_begin < step_end ? step_begin : step_end;
  const int64_t hi = step_begin < step_end ? step_end : step_begin;
  const int64_t e = (d < 0) ? hi : (d < lo ? lo : (d > hi ? hi : d));
  return e - lo;
}

// Their sum, one addition to *acc per workgroup (a few of them, each over many
// particles: the additions all go to one address).  Returns on thread 0.
TPM_DEV void add_active_steps(const int64_t* __restrict__ dstep, int n, int64_t step_begin,
                              int64_t step_end, unsigned long long* acc) {
  __shared__ long long part[4];
  long long v = 0;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
    v += active_steps(dstep[i], step_begin, step_end);
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0)
    atomicAdd(acc, (unsigned long long)(part[0] + part[1] + part[2] + part[3]));
}
static int active_grid(int n) { return std::max(1, std::min((n + 1023) / 1024, 128)); }

// The last workgroup to finish writes the report (its loads of the sum come
// after every workgroup's addition: each adds, then counts itself done).
__global__ void __launch_bounds__(256)
run_report_kernel(const int64_t* __restrict__ dstep, int n, int64_t step_begin, int64_t step_end,
                  unsigned long long* acc, uint32_t* done, const int64_t* flag,
                  const int64_t* ticks, const int32_t* qerr, const int32_t* nactive,
                  RunReport* rep) {
  add_active_steps(dstep, n, step_begin, step_end, acc);
  if (threadIdx.x != 0) return;
  const uint32_t k = __hip_atomic_fetch_add(done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
  if (k + 1 != gridDim.x) return;
  __hip_atomic_store(done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  rep->acc = __hip_atomic_load(acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  rep->flag = *flag;
  rep->ticks = *ticks;
  rep->qerr = *qerr;
  rep->nactive = *nactive;
}

hipError_t launch_run_report(const int64_t* dstep, int n, int64_t step_begin, int64_t step_end,
                             unsigned long long* acc, uint32_t* done, const int64_t* flag,
                             const int64_t* ticks, const int32_t* qerr, const int32_t* nactive,
                             RunReport* rep, hipStream_t st) {
  hipLaunchKernelGGL(run_report_kernel, dim3(active_grid(n)), dim3(256), 0, st, dstep, n,
                     step_begin, step_end, acc, done, flag, ticks, qerr, nactive, rep);
  return hipGetLastError();
}

// ---------------------------------------------------------------- new particles
__global__ void __launch_bounds__(256)
load_particles_kernel(Out out, int n, Work w, const int32_t* __restrict__ idx, int na, bool step,
                      bool reason, bool planet, uint32_t* progress, int nclear,
                      unsigned long long* qctr, int32_t* qerr, int32_t* d_nactive) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    if (step) out.step[i] = -1;
    if (reason) out.reason[i] = ST_ACTIVE;
    if (planet) out.planet[i] = -1;
  }
  if (i < na) {
    const int64_t k = idx ? idx[i] : i;
    w.x[i] = out.r[3 * k]; w.y[i] = out.r[3 * k + 1]; w.z[i] = out.r[3 * k + 2];
    w.vx[i] = out.v[3 * k]; w.vy[i] = out.v[3 * k + 1]; w.vz[i] = out.v[3 * k + 2];
    w.slot[i] = (int32_t)k;
    w.status[i] = ST_ACTIVE;
  }
  if (i < nclear) progress[i] = 0;
  if (i == 0) {
    *qctr = 0;
    *qerr = 0;
    *d_nactive = na;
  }
}

hipError_t launch_load_particles(Out out, int n, Work w, const int32_t* idx, int na, bool step,
                                 bool reason, bool planet, uint32_t* progress, int nclear,
                                 unsigned long long* qctr, int32_t* qerr, int32_t* d_nactive,
                                 hipStream_t st) {
  const int m = std::max(std::max(n, nclear), 1);
  hipLaunchKernelGGL(load_particles_kernel, dim3((m + 255) / 256), dim3(256), 0, st, out, n, w, idx,
                     na, step, reason, planet, progress, nclear, qctr, qerr, d_nactive);
  return hipGetLastError();
}

// ---------------------------------------------------------------- compaction
constexpr int CB = 256;            // threads per compaction block
constexpr int CE = 4;              // elements per thread
constexpr int CTILE = CB * CE;     // elements per block

int compact_scratch_ints(int n_upper) {
  int nb = (n_upper + CTILE - 1) / CTILE;
  return 2 * nb + 2;
}

// Lane prefix count of a 64-bit ballot: number of set bits below this lane.
TPM_DEV int lane_prefix(uint64_t m) {
  uint32_t lo = (uint32_t)m, hi = (uint32_t)(m >> 32);
  return __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0));
}

// Stable partition in one launch.  A block takes the next tile of CTILE entries
// (in the order blocks start, so the tiles before it are in hand), counts its
// active ones, publishes the count, adds up what the tiles before it have
// published (wave 0, 64 tiles at a time, back to the nearest one whose sum is
// complete), publishes its own sum and writes its entries.  A tile's word is
// 0, or 4 * count + 1 (its count alone) or 4 * sum + 2 (with all before it).
// The last block to finish clears the words and the counters for the next
// launch, so they need no host value and a captured launch can be replayed.
// Bound by launches and latency: counting, scanning and moving in launches of
// their own, and a copy of the count to the host, took 28 us for 25,000 entries
// with the gaps between them, and made a call of 64 particles and 256 steps
// 323 us instead of 299.
constexpr uint64_t COMPACT_COUNT = 1, COMPACT_SUM = 2;

__global__ void __launch_bounds__(CB)
compact_kernel(Work src, Work dst, int32_t* d_nactive, int32_t* scratch,
               int32_t* __restrict__ host_count) {
  uint32_t* ticket = reinterpret_cast<uint32_t*>(scratch);
  uint32_t* done = ticket + 1;
  uint64_t* word = reinterpret_cast<uint64_t*>(scratch + 2);
  // (s_last is a word of its own: blocks without a tile have no barrier between
  // their wavefronts' reads of s_tile and its write)
  __shared__ int s_tile, s_n, s_off, s_last;
  __shared__ int wcount[CE][CB / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (threadIdx.x == 0) {
    s_tile = (int)__hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // (the last tile's block writes the new count only after every block with a
    // tile has published, hence read the old one)
    s_n = __hip_atomic_load(d_nactive, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  const int tile = s_tile, n = s_n;
  const int tiles = (n + CTILE - 1) / CTILE;
  if (tile < tiles) {
    const int64_t base = (int64_t)tile * CTILE + threadIdx.x;
    bool keep[CE];
    int pos[CE];
#pragma unroll
    for (int e = 0; e < CE; ++e) {
      const int64_t i = base + e * CB;
      keep[e] = i < n && src.status[i] == ST_ACTIVE;
      const uint64_t m = lanes(keep[e]);
      pos[e] = lane_prefix(m);
      if (lane == 0) wcount[e][wid] = __popcll(m);
    }
    __syncthreads();
    int total = 0;
#pragma unroll
    for (int e = 0; e < CE; ++e)
#pragma unroll
      for (int k = 0; k < CB / 64; ++k) {
        pos[e] += k < wid ? wcount[e][k] : 0;
        total += wcount[e][k];
      }
    // the entries of the rounds before
    int before = 0;
#pragma unroll
    for (int e = 0; e < CE; ++e) {
      pos[e] += before;
#pragma unroll
      for (int k = 0; k < CB / 64; ++k) before += wcount[e][k];
    }
    if (threadIdx.x == 0)
      __hip_atomic_store(word + tile, ((uint64_t)total << 2) | (tile ? COMPACT_COUNT : COMPACT_SUM),
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    double v[CE][6];
    int32_t slot[CE];
#pragma unroll
    for (int e = 0; e < CE; ++e) {
      if (!keep[e]) continue;
      const int64_t i = base + e * CB;
      v[e][0] = src.x[i]; v[e][1] = src.y[i]; v[e][2] = src.z[i];
      v[e][3] = src.vx[i]; v[e][4] = src.vy[i]; v[e][5] = src.vz[i];
      slot[e] = src.slot[i];
    }
    if (wid == 0) {
      int off = 0;
      for (int j = tile - 1; j >= 0; j -= 64) {
        // lane l reads tile j - l; every word up to the nearest complete sum is
        // published by a block that is running or has ended
        const int k = j - lane;
        uint64_t u, need;
        for (;;) {
          u = k >= 0 ? __hip_atomic_load(word + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                     : COMPACT_SUM;
          const uint64_t sums = lanes((u & 3) == COMPACT_SUM);
          need = sums ? sums ^ (sums - 1) : ~0ull;   // lanes up to the first sum
          if ((need & lanes(u == 0)) == 0) break;
          __builtin_amdgcn_s_sleep(1);
        }
        int c = lane_in(need) ? (int)(u >> 2) : 0;
        for (int d = 32; d > 0; d >>= 1) c += __shfl_xor(c, d, 64);
        off += c;
        if (need != ~0ull || lanes((u & 3) == COMPACT_SUM)) break;
      }
      if (lane == 0) {
        s_off = off;
        if (tile)
          __hip_atomic_store(word + tile, ((uint64_t)(off + total) << 2) | COMPACT_SUM,
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (tile == tiles - 1) {
          __hip_atomic_store(d_nactive, off + total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (host_count) *host_count = off + total;
        }
      }
    }
    __syncthreads();
    const int off = s_off;
#pragma unroll
    for (int e = 0; e < CE; ++e) {
      if (!keep[e]) continue;
      const int d = off + pos[e];
      dst.x[d] = v[e][0]; dst.y[d] = v[e][1]; dst.z[d] = v[e][2];
      dst.vx[d] = v[e][3]; dst.vy[d] = v[e][4]; dst.vz[d] = v[e][5];
      dst.slot[d] = slot[e];
      dst.status[d] = ST_ACTIVE;
    }
  } else if (tile == 0 && threadIdx.x == 0 && host_count) {
    *host_count = 0;                           // nothing was active
  }
  // the last block: every look-back is over
  if (threadIdx.x == 0)
    s_last = __hip_atomic_fetch_add(done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) + 1 ==
             gridDim.x;
  __syncthreads();
  if (!s_last) return;
  for (unsigned k = threadIdx.x; k < gridDim.x; k += CB) word[k] = 0;
  if (threadIdx.x < 2) scratch[threadIdx.x] = 0;
}

hipError_t launch_compact(Work src, Work dst, int32_t* d_nactive, int n_upper, int32_t* scratch,
                          int32_t* host_count, hipStream_t st) {
  const int nb = (n_upper + CTILE - 1) / CTILE;
  if (nb <= 0) return hipSuccess;
  hipLaunchKernelGGL(compact_kernel, dim3(nb), dim3(CB), 0, st, src, dst, d_nactive, scratch,
                     host_count);
  return hipGetLastError();
}

// ---------------------------------------------------------------- finalize
__global__ void __launch_bounds__(256)
finalize_kernel(Work w, const int32_t* __restrict__ d_nactive, Out out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= *d_nactive) return;
  if (w.status[i] != ST_ACTIVE) return;
  const int k = w.slot[i];
  out.r[3 * k + 0] = w.x[i]; out.r[3 * k + 1] = w.y[i]; out.r[3 * k + 2] = w.z[i];
  out.v[3 * k + 0] = w.vx[i]; out.v[3 * k + 1] = w.vy[i]; out.v[3 * k + 2] = w.vz[i];
  out.step[k] = -1;
  out.reason[k] = ST_ACTIVE;
  out.planet[k] = -1;
}

hipError_t launch_finalize(Work w, const int32_t* d_nactive, int n_upper, Out out, hipStream_t st) {
  int grid = (n_upper + 255) / 256;
  if (grid <= 0) return hipSuccess;
  hipLaunchKernelGGL(finalize_kernel, dim3(grid), dim3(256), 0, st, w, d_nactive, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------- unit checks
__global__ void sincos_test_kernel(const double* x, double* s, double* c, int n) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double ss, cc;
  sincos(x[i], ss, cc);
  s[i] = ss;
  c[i] = cc;
}

hipError_t launch_sincos_test(const double* x, double* s, double* c, int n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(sincos_test_kernel, dim3((n + 255) / 256), dim3(256), 0, st, x, s, c, n);
  return hipGetLastError();
}

// Per argument: rsqrt, sqrt (sqrt_rsqrt), rcp, mul_rsqrt3(1, x), mul_rsqrt3_1(1, x).
__global__ void rsqrt_test_kernel(const double* x, double* out, int n) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double v = x[i];
  double sq, rs;
  sqrt_rsqrt(v, sq, rs);
  out[5 * (size_t)i + 0] = rsqrt(v);
  out[5 * (size_t)i + 1] = sq;
  out[5 * (size_t)i + 2] = rcp(v);
  out[5 * (size_t)i + 3] = mul_rsqrt3(1.0, v);
  out[5 * (size_t)i + 4] = mul_rsqrt3_1(1.0, v);
}

hipError_t launch_rsqrt_test(const double* x, double* out, int n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(rsqrt_test_kernel, dim3((n + 255) / 256), dim3(256), 0, st, x, out, n);
  return hipGetLastError();
}

// mode 0: the fixed-iteration drift; 1: as the particle kernel with the
// universal fallback; 2: the universal-variable drift alone.
__global__ void drift_test_kernel(KepConst K, int kiters, double ftol, const double* in,
                                  double* out, int32_t* ok, int n, double dt, int mode) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double x = in[6 * i + 0], y = in[6 * i + 1], z = in[6 * i + 2];
  double vx = in[6 * i + 3], vy = in[6 * i + 4], vz = in[6 * i + 5];
  bool g;
  double xk, sk, mk;
  const uint64_t act = lanes(true);
  if (mode == 2) {
    g = lane_in(drift_universal_quick(K, dt, act, x, y, z, vx, vy, vz));
    if (!g) {
      x = in[6 * i + 0]; y = in[6 * i + 1]; z = in[6 * i + 2];
      vx = in[6 * i + 3]; vy = in[6 * i + 4]; vz = in[6 * i + 5];
      g = drift_universal(K.mu, dt, x, y, z, vx, vy, vz);
    }
  } else {
    g = !lane_in(drift_lanes(K, dt, kiters, ftol, quick_serves(kiters, ftol), mode == 1, act, x, y,
                             z, vx, vy, vz, xk, sk, mk));
  }
  // a refused drift leaves the state as it was
  out[6 * i + 0] = g ? x : in[6 * i + 0]; out[6 * i + 1] = g ? y : in[6 * i + 1];
  out[6 * i + 2] = g ? z : in[6 * i + 2]; out[6 * i + 3] = g ? vx : in[6 * i + 3];
  out[6 * i + 4] = g ? vy : in[6 * i + 4]; out[6 * i + 5] = g ? vz : in[6 * i + 5];
  ok[i] = g ? 1 : 0;
}

hipError_t launch_drift_test(const SysConst& S, const double* rv_in, double* rv_out, int32_t* ok,
                             int n, double dt, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  KepConst K{S.mu0, S.inv_mu0, S.sqrt_mu0, S.inv_sqrt_mu0};
  hipLaunchKernelGGL(drift_test_kernel, dim3((n + 255) / 256), dim3(256), 0, st, K, S.kiters,
                     S.ftol, rv_in, rv_out, ok, n, dt, S.universal);
  return hipGetLastError();
}

}  // namespace tpm

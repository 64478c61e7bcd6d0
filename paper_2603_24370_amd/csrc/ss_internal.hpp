// Internal definitions shared by the host API and the HIP kernels of libss.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ss {

constexpr int kHalo = 2;          // Sec. 3.1: default halo width two
constexpr int kMaxWindow = 128;   // largest stall-rule window accepted by the API
// Ring of energies for the stall rule. It is longer than the largest window, so
// the entry of step s - W is never the slot that step s overwrites.
constexpr int kHistLen = 2 * kMaxWindow;
constexpr int kMaxComp = 4;
constexpr int kNumParams = 6;  // theory parameters packed for the kernels

// Device-resident state of one flow (written only by kernels, read by the host
// through a stream-ordered copy).
struct DevStatus {
  double E;          // E_h of the field at the last arrest test
  double E_prev;     // energy the next arrest test compares with
  double gmax;       // max |G| at the last arrest test
  double eval_E;     // result slots of ss_energy_grad
  double eval_gmax;
  double grad_tol;   // stop rules (used when minimise != 0)
  double rel_e_tol;
  long long max_steps;
  long long step;        // RK4 steps started since set_field
  long long n_arrests;
  int arrest;            // 1 if the last arrest test fired
  int done;              // stop reason once a stop rule held (SS_STOP_*), else 0
  int nonfinite;         // non-finite count of the last test
  int window;
  int minimise;          // 1: the arrest pass applies the stop rules
  unsigned counter;      // these two are always 0: places in the checkpoint blob, which
  unsigned counter_obs;  // holds this struct
  int fresh;             // set when a run is armed: its first test is of the field
                         // the last run ended on (or a fresh one), whose arrest is decided
  double e_target;       // minimise stops once E <= e_target (-inf: never)
  double hist[kHistLen]; // E at step s is kept at hist[s % kHistLen]
  double obs[16];        // observable sums (see ss_api)
};

// The part of the status that a reduction changes, as a kernel holds it.
struct Head {
  double E, E_prev, gmax;
  long long step, n_arrests;
  int arrest, done, nonfinite, fresh;
};

__device__ __forceinline__ Head load_head(const DevStatus* s) {
  return Head{s->E, s->E_prev, s->gmax, s->step, s->n_arrests, s->arrest, s->done, s->nonfinite, s->fresh};
}

__device__ __forceinline__ void store_head(DevStatus* s, const Head& h) {
  s->E = h.E;
  s->E_prev = h.E_prev;
  s->gmax = h.gmax;
  s->step = h.step;
  s->n_arrests = h.n_arrests;
  s->arrest = h.arrest;
  s->done = h.done;
  s->nonfinite = h.nonfinite;
  s->fresh = h.fresh;
}

// How a pass of the single lattice learns the status. A reducing pass ends with
// one partial per workgroup; the next launch that needs the status sums them
// itself, every workgroup in the same fixed order, and takes the decisions of
// that test (Head, as decide() gives it), so a test costs no launch of its own
// (a one-workgroup launch between two passes of a small lattice takes as long as
// a third of the pass: 3.6 of 13.8 us per velocity Verlet step on 128^2). Its first
// workgroup stores the result in the other of two status copies, since the rest
// still read the first. Rules and the energy history are in st alone.
struct Link {
  DevStatus* st;
  const DevStatus* in;  // head before the pending test
  DevStatus* out;       // head after it (in where none is pending)
  const double* part;   // the pending test's partials, 4 doubles per workgroup
  int n;                // their number
  int kind;             // the tested pass's finalise_kind, or -1: nothing is pending
};

// Field buffers of one context, in the device layout: component planes of
// (Ny + 4) rows of `pitch` elements; element (c, j, i) at c*plane + (j+2)*pitch + (i+2).
template <class T>
struct Bufs {
  T* phi[2];   // ping-pong field
  T* vel[2];   // ping-pong fictitious velocity
  T* a1;       // stage-1 acceleration
  T* a2;       // stage-2 acceleration
  T* q;        // a1 + 2 a2 + 2 a3
  long pitch;
  long plane;
  int Nx, Ny;
  // demagnetising potential of the stage point a pass evaluates (FP64, padded
  // plane of row length psi_pitch = Nx + 4, zero outside the interior); null
  // when the theory has no demagnetising term
  const double* psi;
  long psi_pitch;
};

// Theory constants packed for the kernels.
struct Coeffs {
  double h, dt;
  double p[kNumParams];  // AH: {lambda}; CM: {J, D, K, B, Dy, mu_d}; BS: {kappa, mu^2}
};

// Passes of one RK4 step and the single-evaluation variants.
enum Pass : int {
  kP1 = 0,     // stage 1: a1 = -G(phi), energy, arrest test and stop rules
  kP2 = 1,     // stage 2: a2 = -G(phi + dt/2 v)
  kP3 = 2,     // stage 3: q  = a1 + 2 a2 + 2 a3, a3 = -G(phi + dt/2 v + dt^2/4 a1)
  kP4 = 3,     // stage 4: a4 = -G(phi + dt v + dt^2/2 a2); phi', v'
  kEval = 4,   // G and E of a given field; flow state untouched
  kCheck = 5,  // arrest test of the current field only (after a run of steps)
  // Gradient flow, and velocity Verlet in its stored-force form, keep the force
  // a = -G of the current field in one of two force buffers (a1, a2 by step parity):
  kPrime = 6,  // arrest test of the current field, as kCheck, and its force stored
  kGF = 8,     // gradient flow: phi' = phi + dt^2/2 a, a' = -G(phi'), E_h(phi')
  kVVA = 12,   // velocity Verlet: phi' = phi + dt v + dt^2/2 a, a' = -G(phi'),
               //   v' = v + dt/2 (a + a'), E_h(phi'); then the arrest test of phi'
  // Velocity Verlet in kick-drift-kick form (large lattices and batches): within
  // a run the velocity buffer holds u = v + dt/2 a of the current field (the
  // next half-step velocity), so a step reads and writes the field and u only.
  kVV = 7,          // phi' = phi + dt u, G' = G(phi'), v' = u - dt/2 G' (tangent
                    //   to phi' for unit fields), u' = v' - dt/2 G', E_h(phi');
                    //   then the arrest test of phi'
  kVVStart = 9,     // start of a run: u = v - dt/2 G(phi), and the arrest test
                    //   of the current field as kCheck
  kVVRestart = 10,  // before a step that follows an arrest (v = 0): u = -dt/2 G(phi)
  kVVEnd = 11,      // end of a run: v = u + dt/2 G(phi), or 0 after an arrest
  // Gradient flow on the lattice theories keeps only the field: a step tests the
  // field it reads and writes the next one.
  kGD = 13,       // E_h(phi), G(phi) and the stop rules of phi (no arrest); writes
                  //   phi' = phi - tau G(phi) (tau = dt^2/2; on the unit sphere for
                  //   unit fields); the step advances unless a rule fired
  kGDCheck = 14,  // end of a run: E_h and G of the current field, tested without arrest
};

// The pass writes a new field and tests it (its finalise advances the step first).
constexpr bool advances_first(int pass) { return pass == kVV || pass == kVVA || pass == kGF; }
// The pass reduces energy, max |G| and a non-finite count.
constexpr bool reduces(int pass) {
  return pass == kP1 || pass == kEval || pass == kCheck || pass == kPrime || advances_first(pass) ||
         pass == kVVStart || pass == kGD || pass == kGDCheck;
}
// The pass's status update takes no arrest decision (gradient flow has no velocity).
constexpr bool no_arrest(int pass) { return pass == kGF || pass == kGD || pass == kGDCheck; }
// The pass evaluates G at a stage point phi + cv v + ca a (stage_coeffs) rather
// than at the current field.
constexpr bool staged(int pass) { return pass == kP2 || pass == kP3 || pass == kP4 || advances_first(pass); }
constexpr bool stage_reads_v(int pass) { return staged(pass) && pass != kGF; }
constexpr bool stage_reads_a(int pass) { return pass == kP3 || pass == kP4 || pass == kGF || pass == kVVA; }
// The pass reads the arrest flag: RK4 stages 2-4 and the stored-force velocity
// Verlet step start from rest after an arrest, and the kick-drift-kick end of
// run sets v = 0.
constexpr bool uses_arrest(int pass) {
  return pass == kP2 || pass == kP3 || pass == kP4 || pass == kVVA || pass == kVVEnd;
}
// The pass writes the velocity buffer of the current field in place (each site
// by the thread that reads it): the velocity Verlet passes around the steps.
constexpr bool vv_in_place(int pass) { return pass == kVVStart || pass == kVVRestart || pass == kVVEnd; }
// What the status update after a reducing pass does (bits): the step advances
// before the test, the test takes no arrest decision, the step advances after it.
constexpr int kAdvanceFirst = 1, kNoArrest = 2, kAdvanceAfter = 4;
constexpr int finalise_kind(int pass) {
  return (advances_first(pass) ? kAdvanceFirst : 0) | (no_arrest(pass) ? kNoArrest : 0) |
         ((pass == kP1 || pass == kGD) ? kAdvanceAfter : 0);
}
// Passes launched once per run (or after an arrest) on one tile shape, whatever
// the context's tile.
constexpr bool fixed_tile(int pass) { return vv_in_place(pass) || pass == kGDCheck; }

// Coefficients of the stage point phi + cv v + ca a of a pass. After an arrest
// the RK4 stages 2-4 and the stored-force velocity Verlet step start from rest
// (cv = 0); the kick-drift-kick u already carries the arrest (kVVRestart).
template <class T, int PASS>
__device__ __forceinline__ void stage_coeffs(T dt, bool arrest, T& cv, T& ca) {
  cv = T(0);
  ca = T(0);
  if (PASS == kP2) cv = T(0.5) * dt;
  if (PASS == kP3) { cv = T(0.5) * dt; ca = T(0.25) * dt * dt; }
  if (PASS == kP4 || PASS == kVVA) { cv = dt; ca = T(0.5) * dt * dt; }
  if (PASS == kVV) cv = dt;
  if (PASS == kGF) ca = T(0.5) * dt * dt;
  if (arrest) cv = T(0);
}

// Map a launched workgroup id to a tile so that the workgroups one XCD receives
// (ids congruent mod 8 go to the same XCD) cover a contiguous range of tiles
// and share their halos in that XCD's L2.
__device__ __forceinline__ int xcd_tile(int b, int nlaunch) {
  const int per = nlaunch >> 3;
  return (b & 7) * per + (b >> 3);
}

// The two operands that lane i of a wave combines to reduce over lanes i and i ^ O,
// given that x is the same at lanes whose numbers differ in the bits above O (as the
// reductions below, from 32 down, leave it). Every exchange stays in the vector units:
// swaps of halves and rows, rotations within rows of 16, permutations of quads. As
// shuffles, an LDS access of some 100 cycles per step and word, the reductions of a pass
// (the pending test's and its own, three values each) took 0.6-0.7 us longer: velocity
// Verlet on 128^2 FP32 8.8 us per step, now 8.2; gradient flow of baby Skyrme on
// 1021 x 517 18.0 and 16.5.
template <int O>
__device__ __forceinline__ void lane_pair(unsigned x, unsigned& a, unsigned& b) {
  if constexpr (O == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    a = r[0];
    b = r[1];
  } else if constexpr (O == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    a = r[0];
    b = r[1];
  } else {
    constexpr int kRor8 = 0x128, kRor4 = 0x124, kQuad2301 = 0x4E, kQuad1032 = 0xB1;
    constexpr int ctrl = O == 8 ? kRor8 : O == 4 ? kRor4 : O == 2 ? kQuad2301 : kQuad1032;
    a = x;
    b = (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, 0xF, 0xF, true);
  }
}

template <int O>
__device__ __forceinline__ void lane_pair(double x, double& a, double& b) {
  const unsigned long long u = __double_as_longlong(x);
  unsigned al, bl, ah, bh;
  lane_pair<O>((unsigned)u, al, bl);
  lane_pair<O>((unsigned)(u >> 32), ah, bh);
  a = __longlong_as_double((long long)(((unsigned long long)ah << 32) | al));
  b = __longlong_as_double((long long)(((unsigned long long)bh << 32) | bl));
}

// x reduced over the 64 lanes of a wave in pairs at distance 32, 16, ..., 1, for every
// lane.
template <class V, class F>
__device__ __forceinline__ V wave_reduce(V x, F&& f) {
  V a, b;
  lane_pair<32>(x, a, b);
  x = f(a, b);
  lane_pair<16>(x, a, b);
  x = f(a, b);
  lane_pair<8>(x, a, b);
  x = f(a, b);
  lane_pair<4>(x, a, b);
  x = f(a, b);
  lane_pair<2>(x, a, b);
  x = f(a, b);
  lane_pair<1>(x, a, b);
  return f(a, b);
}

__device__ __forceinline__ double wave_sum(double x) {
  return wave_reduce(x, [](double a, double b) { return a + b; });
}

__device__ __forceinline__ double wave_max(double x) {
  return wave_reduce(x, [](double a, double b) { return fmax(a, b); });
}

__device__ __forceinline__ int wave_isum(int x) {
  return (int)wave_reduce((unsigned)x, [](unsigned a, unsigned b) { return a + b; });
}

// Workgroup reduction of (sum, max, count) in a fixed order; the result is valid
// in thread 0. `red` needs 3 * (blockDim/64) doubles of LDS.
template <int NT>
__device__ __forceinline__ void block_reduce3(double& s, double& m, int& n, double* red) {
  constexpr int NW = NT / 64;
  const int lane = threadIdx.x & 63;
  const int w = (threadIdx.y * blockDim.x + threadIdx.x) >> 6;
  s = wave_sum(s);
  m = wave_max(m);
  n = wave_isum(n);
  if (lane == 0) {
    red[w] = s;
    red[NW + w] = m;
    red[2 * NW + w] = (double)n;
  }
  __syncthreads();
  if (w == 0 && lane == 0) {
    double ss = 0.0, mm = 0.0, nn = 0.0;
    for (int k = 0; k < NW; ++k) {
      ss += red[k];
      mm = fmax(mm, red[NW + k]);
      nn += red[2 * NW + k];
    }
    s = ss;
    m = mm;
    n = (int)nn;
  }
}


// x, the same in every lane, as a scalar: what is selected by it (a ping-pong buffer's
// base) then stays in scalar registers too. The status is computed in vector registers.
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// The stop rules, and the energy of `window` steps back for the stall rule.
struct Rules {
  double grad_tol, rel_e_tol, e_target, e_window;
  long long max_steps;
  int window, minimise;
};

// The rules for the test of a head (kind: finalise_kind of the tested pass).
__device__ __forceinline__ Rules load_rules(const DevStatus* st, const Head& h, int kind) {
  Rules q{st->grad_tol, st->rel_e_tol, st->e_target, 0.0, st->max_steps, st->window, st->minimise};
  const long long s0 = h.step + (kind & kAdvanceFirst ? 1 : 0);
  if (q.window > 0 && s0 >= q.window) q.e_window = st->hist[(s0 - q.window) % kHistLen];
  return q;
}

// Whether a test of energy E arrests the flow: not the first one of a run (decide()),
// nor gradient flow's, which has no velocity.
__device__ __forceinline__ bool arrests(const Head& h, int kind, double E) {
  return !(kind & kNoArrest) && h.fresh == 0 && E > h.E_prev;
}

// Status update after a reduction of one field: arrest test E > E_prev (strict,
// eq. (4)), the stop rules when minimising, and the step counter. E is already
// multiplied by h^2. The tested step is returned (its place in the history).
__device__ __forceinline__ long long decide(Head& h, const Rules& q, int kind, double E, double gmax, int nfin) {
  // a one-pass step has written the new field: it becomes the current one, and
  // the tests below are those of the new field
  if (kind & kAdvanceFirst) ++h.step;
  const long long s0 = h.step;
  // The first test of a run is of the field the last run ended on, whose arrest
  // that run decided (and applied), or of a fresh field (E_prev infinite): it
  // takes no new arrest decision and keeps the energy the next test compares
  // with, so a run split in two decides its arrests as one run does. (Its own
  // sum of the same field may differ in the last bits: another launch shape.)
  const bool retest = h.fresh != 0;
  const int arr = arrests(h, kind, E) ? 1 : 0;
  h.fresh = 0;
  if (!retest) h.arrest = arr;
  if (arr) h.n_arrests += 1;
  if (!retest || !isfinite(h.E_prev)) h.E_prev = E;
  h.E = E;
  h.gmax = gmax;
  h.nonfinite = nfin;
  int done = 0;
  if (nfin > 0) {
    done = 4;
  } else if (q.minimise) {
    if (gmax < q.grad_tol) done = 1;
    else if (q.window > 0 && s0 >= q.window && fabs(E - q.e_window) <= q.rel_e_tol * fabs(E)) done = 2;
    else if (E <= q.e_target) done = 5;
    else if (s0 >= q.max_steps) done = 3;
  }
  if (done) h.done = done;
  else if (kind & kAdvanceAfter) h.step = s0 + 1;
  return s0;
}

// The first 256 threads' sum of n partials of (energy, max |G|, non-finite count)
// in workgroup order (strided by 256, then in wave order), for every thread. The
// loads of up to four strides are in flight together. red: 12 doubles of LDS. All
// threads of the workgroup call it.
__device__ __forceinline__ void sum_partials(const double* __restrict__ part, int n, int tid, double* red, double& se,
                                             double& sg, int& sn) {
  se = 0.0;
  sg = 0.0;
  sn = 0;
  if (tid < 256) {
    constexpr int U = 4;
    for (int k0 = 0; k0 < n; k0 += 256 * U) {
      double p[U][3];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = k0 + 256 * u + tid;
        const double* q = part + 4 * (long)(k < n ? k : 0);
        p[u][0] = q[0];
        p[u][1] = q[1];
        p[u][2] = q[2];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (k0 + 256 * u + tid < n) {
          se += p[u][0];
          sg = fmax(sg, p[u][1]);
          sn += (int)p[u][2];
        }
    }
    se = wave_sum(se);
    sg = wave_max(sg);
    sn = wave_isum(sn);
    if ((tid & 63) == 0) {
      const int w = tid >> 6;
      red[w] = se;
      red[4 + w] = sg;
      red[8 + w] = (double)sn;
    }
  }
  __syncthreads();
  double ss = 0.0, mm = 0.0, nn = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    ss += red[k];
    mm = fmax(mm, red[4 + k]);
    nn += red[8 + k];
  }
  se = ss;
  sg = mm;
  sn = (int)nn;
}

// The status as of this launch (Link), for every thread of a workgroup of at
// least 256. h2 = h^2 of the lattice. red: 12 doubles of LDS that nothing else uses:
// they are read after the last barrier here, and a workgroup without work has no
// other before it sums its own values. Its loads are independent of each other, so
// the launch waits for memory once.
__device__ __forceinline__ Head resolve(const Link& L, double h2, int tid, double* red) {
  Head h = load_head(L.in);
  if (L.kind < 0) return h;
  const Rules q = load_rules(L.st, h, L.kind);
  double se, sg;
  int sn;
  sum_partials(L.part, L.n, tid, red, se, sg, sn);
  if (!h.done) {
    const long long s0 = decide(h, q, L.kind, h2 * se, sg, sn);
    if (blockIdx.x == 0 && tid == 0) L.st->hist[s0 % kHistLen] = h.E;
  }
  if (blockIdx.x == 0 && tid == 0) store_head(L.out, h);
  return h;
}

}  // namespace ss

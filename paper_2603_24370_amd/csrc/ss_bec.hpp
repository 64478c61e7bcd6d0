// Rotating trapped Bose-Einstein condensate (Sec. 4.3) on the device.
//
// Trap units (hbar = m = omega = 1), psi = u + i w, two components:
//   e = 1/2 |grad psi|^2 + 1/2 r^2 |psi|^2 + g/2 |psi|^4 - Omega Re(psi* L_z psi),
//   L_z = -i (x d_y - y d_x), Re(psi* L_z psi) = u (x w_y - y w_x) - w (x u_y - y u_x),
// with eq. (1) first derivatives in the energy and the Euler-Lagrange gradient
//   G_u = -lap u + r^2 u + 2 g |psi|^2 u - 2 Omega (x w_y - y w_x),
//   G_w = -lap w + r^2 w + 2 g |psi|^2 w + 2 Omega (x u_y - y u_x)
// (eq. (2) second derivatives). Sites are cell-centred: x_i = (i - (Nx-1)/2) h.
//
// The flow holds the atom number N = h^2 sum |psi|^2 fixed: every stage point is
// scaled to N before its force is taken, the force is -(G - mu psi) with
// mu = <psi, G> / <psi, psi> (its projection on the tangent space of that
// sphere), and after each step the field is scaled to N and the velocity
// projected on the tangent space. Each of these needs sums over the whole lattice,
// and a sum costs a launch boundary; whatever else follows a sum is of the same site,
// and is done in the launch that ends at the next sum:
//   bec_stage   the last step's constraint, the next stage point; its norm
//   bec_grad    the scale, G; the sums of psi.G and psi.psi
//   bec_apply   mu, the force and the stage's update; in RK4's stages 1-3 the next
//               stage point and its norm, else the sums of the step's constraint
// that is 9 launches per RK4 step and 3 per step of the one-pass integrators (15 and
// 6 with a launch for each of these; 256^2 sites FP32, RK4: 89 us per step then, 60
// with these alone). A small lattice's launch takes the latency of its chain (partials, their
// sum, sites, a block sum), so the loads of a thread's first site are issued before
// the sums that they wait for. All sums are FP64 per-workgroup partials added in
// workgroup order, by every workgroup of the launch that needs the total.
#pragma once

#include "ss_kernels.hpp"

namespace ss {

constexpr int kBecGroups = 512;  // workgroups of every BEC launch (grid-stride over sites)

// Work buffers: the stage point S and the gradient G (two planes each, the flow's
// layout), three sets of FP64 workgroup partials (the stage point's norm,
// kBecGroups; the gradient's sums and the update's, kBecGroups * 4 each), and the
// scale c of the stage point to N. Sums of partials are taken by every workgroup of
// the launch that uses them (in the same fixed order), workgroup 0 of bec_grad
// keeping the scale for bec_apply.
template <class T>
struct BecBufs {
  T* S;
  T* G;
  double* part;  // {phi'.phi', phi'.v'} of the update (bec_apply)
  double* sc;    // c
  double* ps;    // the stage point's norm (bec_stage, bec_apply)
  double* pg;    // the gradient's sums (bec_grad): psi.G, psi.psi, energy, non-finite count
};

// What a step leaves to be done before the next stage point: nothing; phi' scaled to N
// and v' projected (RK4); v' projected (velocity Verlet).
enum BecEnd : int { kBecNone = 0, kBecScale = 1, kBecProject = 2 };

// The block of 256 sites that a workgroup takes first, and whose place its partials
// have: workgroups of one XCD (numbers that agree mod 8) take a band of the lattice's
// first kBecGroups blocks, so that rows that neighbours share are in one L2. A
// permutation of 0 .. kBecGroups - 1, so sums over partials keep their order. us per RK4
// step in the order of the workgroups and in bands: 256^2 FP32 39 / 37, FP64 46 / 40, 512^2
// FP32 61 / 49.
__device__ __forceinline__ int bec_block(long n) {
  const int nb = (int)min((long)kBecGroups, (n + 255) / 256), per = (nb + 7) / 8;
  const int b = blockIdx.x, q = b >> 3;
  return q < per ? (b & 7) * per + q : b;
}

#define BEC_SITES(n) \
  for (long k_ = bec_block(n) * 256L + threadIdx.x; k_ < (n); k_ += (long)gridDim.x * 256L)

// Sums of N values over 256 threads in a fixed order, for every thread. red: 4 N
// doubles of LDS that nothing else uses.
template <int N>
__device__ __forceinline__ void bec_block_sums(double (&v)[N], double* red) {
#pragma unroll
  for (int m = 0; m < N; ++m) v[m] = wave_sum(v[m]);
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int m = 0; m < N; ++m) red[4 * m + (threadIdx.x >> 6)] = v[m];
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < N; ++m) v[m] = red[4 * m] + red[4 * m + 1] + red[4 * m + 2] + red[4 * m + 3];
}

// Sums over the kBecGroups partials part[k * STRIDE + m], m < N, by a workgroup of 256
// threads in a fixed order (strided per thread, then in wave order), for every thread.
template <int N, int STRIDE>
__device__ __forceinline__ void bec_partials_sums(const double* __restrict__ part, double (&v)[N], double* red) {
  double p[kBecGroups / 256][N];
#pragma unroll
  for (int k = 0; k < kBecGroups / 256; ++k)
#pragma unroll
    for (int m = 0; m < N; ++m) p[k][m] = part[(long)(k * 256 + threadIdx.x) * STRIDE + m];
#pragma unroll
  for (int m = 0; m < N; ++m) {
    v[m] = 0.0;
#pragma unroll
    for (int k = 0; k < kBecGroups / 256; ++k) v[m] += p[k][m];
  }
  bec_block_sums(v, red);
}

__device__ __forceinline__ double bec_block_max(double v, double* red) {
  v = wave_max(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
}

// A site's share of the end-of-step constraint: v' projected on the tangent space at
// phi' (RK4 with the unscaled phi', the coefficient being scale-free), phi' scaled.
template <class T>
struct BecConstraint {
  T cs, m;
};

template <class T>
__device__ __forceinline__ BecConstraint<T> bec_constraint(const double* __restrict__ part, const Coeffs& cf,
                                                           double* red) {
  double v[2];
  bec_partials_sums<2, 4>(part, v, red);
  return BecConstraint<T>{(T)sqrt(cf.p[2] / (cf.h * cf.h * v[0])), (T)(v[1] / v[0])};
}

// Stage point of a pass over the padded lattice (as the stage passes form it) and the
// partial sums of its squares over the interior: the current field (PASS kP1, for all
// passes that evaluate it, and kEval, which takes src where that is given), or the new
// field of a one-pass step. The launch takes the pending test (Link), and before that
// ends the last step (BecEnd), which a flow that this test stops has taken as well.
template <class T, int PASS>
__global__ void __launch_bounds__(256) bec_stage(Bufs<T> B, Coeffs cf, Link link, const T* __restrict__ src,
                                                 BecBufs<T> W, int end) {
  __shared__ double red[12], redc[8], reds[4];
  constexpr bool ONEPASS = advances_first(PASS);
  Head hd = {};
  bool ended = false;
  if (PASS == kEval) {
    hd.step = link.st->step;
  } else {
    ended = end != kBecNone && !link.in->done;
    hd = resolve(link, cf.h * cf.h, threadIdx.x, red);
    if (hd.done && !ended) return;
  }
  BecConstraint<T> k = {T(1), T(0)};
  if (ended) k = bec_constraint<T>(W.part, cf, redc);
  const int cur = uniform(int(hd.step & 1));
  T cv, ca;
  stage_coeffs<T, PASS>((T)cf.dt, PASS == kVVA && hd.arrest != 0, cv, ca);
  // phc is ph but for an evaluation of src: a site is read through the one and written
  // through the other, so neither is __restrict__
  T* phc = cur ? B.phi[1] : B.phi[0];
  const T* ph = (PASS == kEval && src != nullptr) ? src : phc;
  T* __restrict__ vv = cur ? B.vel[1] : B.vel[0];
  // one-pass integrators: the current field's force in the buffer of the step's parity
  const T* __restrict__ aa = cur ? B.a2 : B.a1;
  const long Wd = B.Nx + 4, H = B.Ny + 4;
  double acc[1] = {0.0};
  BEC_SITES(Wd * H) {
    const int jj = (int)(k_ / Wd), ii = (int)(k_ - (long)jj * Wd);
    const long o = (long)jj * B.pitch + ii;
    const bool inner = ii >= 2 && ii < B.Nx + 2 && jj >= 2 && jj < B.Ny + 2;
    const bool fix = ended && inner;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      T x = ph[c * B.plane + o], v = T(0);
      if (PASS == kVVA || fix) v = vv[c * B.plane + o];
      if (fix) {
        v = v - k.m * x;
        vv[c * B.plane + o] = v;
        if (end == kBecScale) {
          x = k.cs * x;
          phc[c * B.plane + o] = x;
        }
      }
      if (PASS == kVVA) x += cv * v;
      if (ONEPASS) x += ca * aa[c * B.plane + o];
      W.S[c * B.plane + o] = x;
      if (inner) acc[0] += (double)x * (double)x;
    }
  }
  bec_block_sums(acc, reds);
  if (threadIdx.x == 0) W.ps[bec_block(Wd * H)] = acc[0];
}

// The end of a run's last step, where no stage follows (no test is taken).
template <class T>
__global__ void __launch_bounds__(256) bec_end(Bufs<T> B, Coeffs cf, const DevStatus* __restrict__ st, BecBufs<T> W,
                                               int end) {
  __shared__ double red[8];
  if (st->done) return;
  const BecConstraint<T> k = bec_constraint<T>(W.part, cf, red);
  // an RK4 step has advanced the counter; velocity Verlet's pending test does
  const int nxt = int((st->step + (end == kBecProject ? 1 : 0)) & 1);
  T* __restrict__ ph = nxt ? B.phi[1] : B.phi[0];
  T* __restrict__ v = nxt ? B.vel[1] : B.vel[0];
  const long n = (long)B.Nx * B.Ny;
  BEC_SITES(n) {
    const int j = (int)(k_ / B.Nx), i = (int)(k_ - (long)j * B.Nx);
    const long o = (long)(j + 2) * B.pitch + (i + 2);
#pragma unroll
    for (int comp = 0; comp < 2; ++comp) {
      const long q = comp * B.plane + o;
      const T p = ph[q];
      v[q] = v[q] - k.m * p;
      if (end == kBecScale) ph[q] = k.cs * p;
    }
  }
}

// G at the scaled stage point; partials {psi.G, psi.psi, energy density sum,
// non-finite count}. The scale is c = sqrt(N / (h^2 sum S^2)), of the interior. The
// energy is that of the field the pass tests, in FP64: the stage point as stored
// (unscaled) for an evaluation, a check or the first stage of RK4; the scaled stage
// point, which becomes the new field, for a one-pass step. RK4's stage 2 takes the
// test of stage 1 (Link).
template <class T, int PASS>
__global__ void __launch_bounds__(256) bec_grad(Bufs<T> B, Coeffs cf, Link link, BecBufs<T> W) {
  __shared__ double red[12], redc[4], reds[16];
  constexpr bool REDUCE = reduces(PASS);
  const long n = (long)B.Nx * B.Ny;
  // stage values along x and y at distances -2 .. 2 (the centre in both)
  T sx[2][5], sy[2][5];
  int i = 0, j = 0;
  auto load = [&](long k) {
    j = (int)(k / B.Nx);
    i = (int)(k - (long)j * B.Nx);
#pragma unroll
    for (int comp = 0; comp < 2; ++comp) {
      const T* Sc = W.S + comp * B.plane + (long)(j + 2) * B.pitch + (i + 2);
#pragma unroll
      for (int d = 0; d < 5; ++d) {
        sx[comp][d] = Sc[d - 2];
        if (d != 2) sy[comp][d] = Sc[(long)(d - 2) * B.pitch];
      }
      sy[comp][2] = sx[comp][2];
    }
  };
  const long step = (long)gridDim.x * 256L;
  const int lb = bec_block(n);
  long k = lb * 256L + threadIdx.x;
  if (k < n) load(k);
  if (PASS == kP2) {
    if (resolve(link, cf.h * cf.h, threadIdx.x, red).done) return;
  } else if (PASS != kEval) {
    if (link.in->done) return;
  }
  double norm[1];
  bec_partials_sums<1, 1>(W.ps, norm, redc);
  const double cd = sqrt(cf.p[2] / (cf.h * cf.h * norm[0]));
  if (blockIdx.x == 0 && threadIdx.x == 0) W.sc[0] = cd;
  const T c = (T)cd;
  const T g = (T)cf.p[0], Om = (T)cf.p[1];
  const double h = cf.h;
  const T c1 = T(1.0 / (12.0 * h)), c2 = T(1.0 / (12.0 * h * h));
  const double d1 = 1.0 / (12.0 * h);
  double sums[4] = {0.0, 0.0, 0.0, 0.0};
  for (; k < n; k += step) {
    T f[2], dx[2], dy[2], lap[2];
    double fd[2], dxd[2], dyd[2];
#pragma unroll
    for (int comp = 0; comp < 2; ++comp) {
      // the scaled value: c S inside the interior, S on the halo
      auto ax = [&](int d) {
        const T v = sx[comp][d + 2];
        return (i + d >= 0 && i + d < B.Nx) ? c * v : v;
      };
      auto ay = [&](int d) {
        const T v = sy[comp][d + 2];
        return (j + d >= 0 && j + d < B.Ny) ? c * v : v;
      };
      const T xm2 = ax(-2), xm1 = ax(-1), x0 = ax(0), xp1 = ax(1), xp2 = ax(2);
      const T ym2 = ay(-2), ym1 = ay(-1), yp1 = ay(1), yp2 = ay(2);
      f[comp] = x0;
      dx[comp] = c1 * ((xm2 - xp2) + T(8) * (xp1 - xm1));
      dy[comp] = c1 * ((ym2 - yp2) + T(8) * (yp1 - ym1));
      lap[comp] = c2 * ((-(xm2 + xp2) + T(16) * (xm1 + xp1)) + (-(ym2 + yp2) + T(16) * (ym1 + yp1)) - T(60) * x0);
      if (REDUCE) {
        auto rx = [&](int d) { return advances_first(PASS) ? (double)ax(d) : (double)sx[comp][d + 2]; };
        auto ry = [&](int d) { return advances_first(PASS) ? (double)ay(d) : (double)sy[comp][d + 2]; };
        fd[comp] = rx(0);
        dxd[comp] = d1 * ((rx(-2) - rx(2)) + 8.0 * (rx(1) - rx(-1)));
        dyd[comp] = d1 * ((ry(-2) - ry(2)) + 8.0 * (ry(1) - ry(-1)));
      }
    }
    const double xd = (i - 0.5 * (B.Nx - 1)) * h, yd = (j - 0.5 * (B.Ny - 1)) * h;
    const T x = (T)xd, y = (T)yd, r2 = (T)(xd * xd + yd * yd);
    const T u = f[0], w = f[1], rho = u * u + w * w;
    const T G0 = -lap[0] + r2 * u + T(2) * g * rho * u - T(2) * Om * (x * dy[1] - y * dx[1]);
    const T G1 = -lap[1] + r2 * w + T(2) * g * rho * w + T(2) * Om * (x * dy[0] - y * dx[0]);
    const long o = (long)(j + 2) * B.pitch + (i + 2);
    W.G[o] = G0;
    W.G[B.plane + o] = G1;
    sums[0] += (double)u * (double)G0 + (double)w * (double)G1;
    sums[1] += (double)u * (double)u + (double)w * (double)w;
    if (!isfinite(G0) || !isfinite(G1)) sums[3] += 1.0;
    if (REDUCE) {
      const double ud = fd[0], wd = fd[1];
      const double rhod = ud * ud + wd * wd;
      const double lz = ud * (xd * dyd[1] - yd * dxd[1]) - wd * (xd * dyd[0] - yd * dxd[0]);
      const double e = 0.5 * (dxd[0] * dxd[0] + dyd[0] * dyd[0] + dxd[1] * dxd[1] + dyd[1] * dyd[1]) +
                       0.5 * (xd * xd + yd * yd) * rhod + 0.5 * cf.p[0] * rhod * rhod - cf.p[1] * lz;
      sums[2] += e;
      if (!isfinite(e)) sums[3] += 1.0;
    }
    if (k + step < n) load(k + step);
  }
  bec_block_sums(sums, reds);
  if (threadIdx.x == 0) {
    double* p = W.pg + 4 * (long)lb;
#pragma unroll
    for (int m = 0; m < 4; ++m) p[m] = sums[m];
  }
}

// The force a = -(G - mu psi) at the scaled stage point (mu = <psi, G> / <psi, psi>)
// and the pass's update. A reducing pass leaves the partials of its test (energy,
// max |G - mu psi|, non-finite count). RK4's stages 1-3 form the next stage point in
// place of their own, over the padded lattice, and the partials of its norm; stage 2
// starts from rest after an arrest, which the energy of stage 1 decides here as the
// test will. P4 writes the new field and velocity before the step's constraint
// (BecEnd) and the partial sums {phi'.phi', phi'.v'}.
template <class T, int PASS>
__global__ void __launch_bounds__(256) bec_apply(Bufs<T> B, Coeffs cf, Link link, BecBufs<T> W,
                                                 double* __restrict__ partials, T* __restrict__ out, long out_pitch,
                                                 long out_plane) {
  __shared__ double red[16], redm[4], reds[8];
  constexpr bool STAGED = (PASS == kP2 || PASS == kP3 || PASS == kP4);
  constexpr bool THEN = (PASS == kP1 || PASS == kP2 || PASS == kP3);  // forms the next stage point
  constexpr int NEXT = PASS == kP1 ? kP2 : PASS == kP2 ? kP3 : kP4;
  const Head hd = load_head(PASS == kEval ? link.st : link.in);
  if (PASS != kEval && hd.done) return;
  const int cur = uniform(STAGED ? int((hd.step - 1) & 1) : int(hd.step & 1));
  // one-pass integrators: current force (read) and new force (written) by parity
  const T* __restrict__ a_cur = cur ? B.a2 : B.a1;
  T* __restrict__ a_new = cur ? B.a1 : B.a2;
  const T dt = (T)cf.dt;
  const T* __restrict__ ph = cur ? B.phi[1] : B.phi[0];
  const T* __restrict__ vv = cur ? B.vel[1] : B.vel[0];
  T* __restrict__ phn = cur ? B.phi[0] : B.phi[1];
  T* __restrict__ vn = cur ? B.vel[0] : B.vel[1];
  const int X0 = THEN ? 0 : 2, Wd = THEN ? B.Nx + 4 : B.Nx;
  const long n = (long)Wd * (THEN ? B.Ny + 4 : B.Ny);
  constexpr bool READ_A1 = PASS == kP2 || PASS == kP3 || PASS == kP4, READ_V = THEN || PASS == kP4 || PASS == kVVA;
  T S[2], G[2], p0[2], v0[2], a1[2], a2[2], qq[2];
  long o = 0, oo = 0;
  bool inner = false;
  auto load = [&](long k) {
    const int jj = (int)(k / Wd) + X0, ii = (int)(k - (long)(jj - X0) * Wd) + X0;
    o = (long)jj * B.pitch + ii;
    oo = (long)jj * out_pitch + ii;
    inner = !THEN || (ii >= 2 && ii < B.Nx + 2 && jj >= 2 && jj < B.Ny + 2);
#pragma unroll
    for (int comp = 0; comp < 2; ++comp) {
      const long q = comp * B.plane + o;
      S[comp] = W.S[q];
      G[comp] = W.G[q];
      if (THEN || PASS == kP4) p0[comp] = ph[q];
      if (READ_V) v0[comp] = vv[q];
      if (READ_A1) a1[comp] = B.a1[q];
      if (PASS == kP3) a2[comp] = B.a2[q];
      if (PASS == kP4) qq[comp] = B.q[q];
      if (PASS == kVVA) a1[comp] = a_cur[q];
    }
  };
  const long step = (long)gridDim.x * 256L;
  const int lb = bec_block(n);
  long k = lb * 256L + threadIdx.x;
  if (k < n) load(k);
  constexpr int NS = PASS == kP1 ? 3 : 2;
  double sg[NS];  // psi.G, psi.psi, energy
  bec_partials_sums<NS, 4>(W.pg, sg, red);
  const T mu = (T)(sg[0] / sg[1]);
  const T c = (T)W.sc[0];
  bool arrest = hd.arrest != 0;
  if constexpr (PASS == kP1) arrest = arrests(hd, finalise_kind(PASS), cf.h * cf.h * sg[2]);
  T cv, ca;
  stage_coeffs<T, NEXT>(dt, arrest, cv, ca);
  double gm = 0.0, acc[1] = {0.0}, sums[2] = {0.0, 0.0};
  for (; k < n; k += step) {
#pragma unroll
    for (int comp = 0; comp < 2; ++comp) {
      const long q = comp * B.plane + o;
      T a = T(0);
      if (inner) {
        const T Gp = G[comp] - mu * (c * S[comp]);
        a = -Gp;
        gm = fmax(gm, fabs((double)Gp));
        if (PASS == kEval) {
          if (out != nullptr) out[comp * out_plane + oo] = Gp;
        } else if (PASS == kP1) {
          B.a1[q] = a;
        } else if (PASS == kPrime) {
          // the current field's force, in the buffer of the step's parity
          T* __restrict__ as = cur ? B.a2 : B.a1;
          as[q] = a;
        } else if (PASS == kVVA || PASS == kGF) {
          // the scaled stage point is the new field; velocity Verlet also forms
          // v' = v + dt/2 (a + a'), projected after the sums below (BecEnd)
          const T pn = c * S[comp];
          phn[q] = pn;
          a_new[q] = a;
          sums[0] += (double)pn * (double)pn;
          if (PASS == kVVA) {
            const T vnew = (arrest ? T(0) : v0[comp]) + (T(0.5) * dt) * (a1[comp] + a);
            vn[q] = vnew;
            sums[1] += (double)pn * (double)vnew;
          }
        } else if (PASS == kP2) {
          B.a2[q] = a;
        } else if (PASS == kP3) {
          B.q[q] = a1[comp] + T(2) * a2[comp] + T(2) * a;
        } else if (PASS == kP4) {
          const T vs = arrest ? T(0) : v0[comp];
          const T pn = p0[comp] + dt * vs + (dt * dt / T(12)) * (qq[comp] + a1[comp]);
          const T vnew = vs + (dt / T(6)) * (qq[comp] + a);
          phn[q] = pn;
          vn[q] = vnew;
          sums[0] += (double)pn * (double)pn;
          sums[1] += (double)pn * (double)vnew;
        }
      }
      if (THEN) {
        T x = p0[comp];
        x += cv * v0[comp];
        if (PASS == kP2) x += ca * a1[comp];
        if (PASS == kP3) x += ca * a2[comp];
        W.S[q] = x;
        if (inner) acc[0] += (double)x * (double)x;
      }
    }
    if (k + step < n) load(k + step);
  }
  if (THEN) {
    bec_block_sums(acc, reds);
    if (threadIdx.x == 0) W.ps[lb] = acc[0];
  }
  if (PASS == kP4 || PASS == kVVA) {
    bec_block_sums(sums, reds);
    if (threadIdx.x == 0) {
      W.part[4 * (long)lb] = sums[0];
      W.part[4 * (long)lb + 1] = sums[1];
    }
  }
  if (reduces(PASS)) {
    const double m = bec_block_max(gm, redm);
    if (threadIdx.x == 0) {
      double* p = partials + 4 * (long)lb;
      p[0] = W.pg[4 * (long)lb + 2];
      p[1] = m;
      p[2] = W.pg[4 * (long)lb + 3];
    }
  }
}

// Observables of the current field: {E density, |psi|^2, Re(psi* L_z psi)} summed.
template <class T>
__global__ void __launch_bounds__(256) bec_obs(Bufs<T> B, Coeffs cf, const DevStatus* st, double* partials) {
  const int cur = int(st->step & 1);
  const T* __restrict__ ph = cur ? B.phi[1] : B.phi[0];
  const double h = cf.h, d1 = 1.0 / (12.0 * h);
  double v[3] = {0.0, 0.0, 0.0};
  const long n = (long)B.Nx * B.Ny;
  for (long k_ = blockIdx.x * 256L + threadIdx.x; k_ < n; k_ += (long)gridDim.x * 256L) {
    const int j = (int)(k_ / B.Nx), i = (int)(k_ - (long)j * B.Nx);
    const long o = (long)(j + 2) * B.pitch + (i + 2);
    double f[2], dx[2], dy[2];
    for (int comp = 0; comp < 2; ++comp) {
      const T* p = ph + comp * B.plane + o;
      f[comp] = p[0];
      dx[comp] = d1 * (((double)p[-2] - (double)p[2]) + 8.0 * ((double)p[1] - (double)p[-1]));
      dy[comp] = d1 * (((double)p[-2 * B.pitch] - (double)p[2 * B.pitch]) +
                       8.0 * ((double)p[B.pitch] - (double)p[-B.pitch]));
    }
    const double x = (i - 0.5 * (B.Nx - 1)) * h, y = (j - 0.5 * (B.Ny - 1)) * h;
    const double rho = f[0] * f[0] + f[1] * f[1];
    const double lz = f[0] * (x * dy[1] - y * dx[1]) - f[1] * (x * dy[0] - y * dx[0]);
    v[0] += 0.5 * (dx[0] * dx[0] + dy[0] * dy[0] + dx[1] * dx[1] + dy[1] * dy[1]) + 0.5 * (x * x + y * y) * rho +
            0.5 * cf.p[0] * rho * rho - cf.p[1] * lz;
    v[1] += rho;
    v[2] += lz;
  }
  obs_partials(v, partials);
}

#undef BEC_SITES

}  // namespace ss

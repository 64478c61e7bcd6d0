// Demagnetising potential of the chiral magnet (Sec. 4.2, eq. (5)-(6)).
//
// In units where mu_0 M_s^2 is the coefficient mu_d, the potential psi of a field
// n solves Laplace_h psi = d_x n_1 + d_y n_2 on the interior, with psi = 0 outside
// it: the divergence by eq. (1), the Laplacian by eq. (2) along each axis. The
// energy density gains mu_d/2 |grad_h psi|^2 and the Euler-Lagrange gradient
// mu_d grad_h psi (eq. (1) derivatives of psi); the stage passes add both terms
// from the potential of the stage point they evaluate, solved just before.
//
// Solver: conjugate gradients on the symmetric positive definite A = -Laplace_h,
// preconditioned by one multigrid V-cycle, all in FP64. The hierarchy coarsens
// by two per axis (a coarse cell covers two fine sites, N_c = ceil(N / 2)) down
// to a level with fewer than eight sites along an axis; each level rediscretises
// eq. (2) at its spacing 2^l h with a zero halo of width two. The V-cycle is
// symmetric, as the preconditioner of conjugate gradients must be: two weighted
// Jacobi sweeps before and after the coarse correction, bilinear prolongation P
// (weights 3/4 and 1/4 per axis), restriction P^T / 4, and on the coarsest level
// an exact solve by its inverse (computed once on the host; up to kDmExactMax
// sites) or else an even number of Jacobi sweeps from zero. A solve runs a fixed number of
// iterations, warm-started from the last potential (stage points change little
// from one pass to the next), so that it can be captured in a graph. Dot
// products are summed per workgroup and then in workgroup order (deterministic).
//
// Every launch of a solve is bound by its latency (4-6 us for a fraction of a
// microsecond of memory traffic), so the solve is cut into as few as its global
// dependencies allow: two per large level and V-cycle, one for the small levels,
// two per iteration for conjugate gradients, whose update also starts the next
// V-cycle. Two iterations on 512^2: 22 launches (36 with smoothing, restriction,
// dot product, direction and operator apart).
#pragma once

#include "ss_internal.hpp"

namespace ss {

constexpr int kDmMaxLevels = 20;
constexpr int kDmMaxGroups = 2048;  // workgroups of a launch (and partials of a dot product)
constexpr double kDmOmega = 0.8;   // Jacobi weight (stable below 15/16 for this operator)
constexpr int kDmSmooth = 2;       // sweeps before and after the coarse correction
constexpr int kDmCoarse = 40;      // sweeps on the coarsest level (even) where it has no inverse
constexpr int kDmExactMax = 256;   // coarsest levels up to this many sites are solved exactly

// One level of the hierarchy: padded planes of (Ny + 4) rows of pitch = Nx + 4 doubles.
struct DmLevel {
  double* psi;  // solution (the preconditioned residual z on level 0)
  double* tmp;  // the pre-smoothed psi
  double* rhs;  // (level 0: -r, one of the two planes of DmVecs)
  int Nx, Ny;
  long pitch;
  double h;
  double lap;  // 1 / (12 h^2), the factor of eq. (2)
};

// Level-0 vectors of conjugate gradients, the reduction partials and the scalar
// r.z of the last iteration. The direction and -r are each read with a halo by the
// launch that renews them, hence two planes.
struct DmVecs {
  double* x;       // the potential psi
  double* rhs[2];  // -r
  double* d[2];
  double* Ad;
  double* part;    // partials of r.z, one per workgroup
  double* pmv;     // partials of d.Ad
  double* sc;      // {r.z of the last iteration}
};

__device__ __forceinline__ bool dm_skip(const DevStatus* st) { return st != nullptr && st->done != 0; }

__device__ __forceinline__ long dm_at(const DmLevel& L, int j, int i) { return (long)(j + 2) * L.pitch + (i + 2); }

// Laplace_h of a padded plane at interior site (j, i): eq. (2) along both axes.
__device__ __forceinline__ double dm_lap(const double* __restrict__ x, long p, int j, int i, double lap) {
  const double* c = x + (long)(j + 2) * p + (i + 2);
  const double sx = -(c[-2] + c[2]) + 16.0 * (c[-1] + c[1]);
  const double sy = -(c[-2 * p] + c[2 * p]) + 16.0 * (c[-p] + c[p]);
  return (sx + sy - 60.0 * c[0]) * lap;
}

#define DM_SITES(L)                                                                        \
  for (long k_ = blockIdx.x * 256L + threadIdx.x; k_ < (long)(L).Nx * (L).Ny;              \
       k_ += (long)gridDim.x * 256L)

// The coarsest level where it is too large for LDS: kDmCoarse Jacobi sweeps (psi ->
// tmp -> psi ...) from zero, in one workgroup, with a barrier between sweeps. Global
// memory is coherent within a workgroup across the barrier.
static __global__ void __launch_bounds__(256) dm_coarse_solve(DmLevel L, const DevStatus* st) {
  if (dm_skip(st)) return;
  const double s = kDmOmega * L.h * L.h / 5.0;
  const long n = (long)L.Nx * L.Ny;
  for (long k = threadIdx.x; k < n; k += 256) L.psi[dm_at(L, (int)(k / L.Nx), (int)(k % L.Nx))] = 0.0;
  __syncthreads();
  for (int sweep = 0; sweep < kDmCoarse; ++sweep) {
    const double* __restrict__ src = (sweep & 1) ? L.tmp : L.psi;
    double* __restrict__ dst = (sweep & 1) ? L.psi : L.tmp;
    for (long k = threadIdx.x; k < n; k += 256) {
      const int j = (int)(k / L.Nx), i = (int)(k - (long)j * L.Nx);
      const long o = dm_at(L, j, i);
      dst[o] = src[o] - s * (L.rhs[o] - dm_lap(src, L.pitch, j, i, L.lap));
    }
    __syncthreads();
  }
}

// 1-D weight of fine index f in coarse cell J (transpose of the prolongation):
// f = 2J - 1 and 2J + 2 carry 1/4, f = 2J and 2J + 1 carry 3/4.
__device__ __forceinline__ double dm_w(int f, int J) {
  const int d = f - 2 * J;
  return (d == 0 || d == 1) ? 0.75 : 0.25;
}

// (P c)(j, i): the bilinear correction at fine site (j, i) from the coarse plane
// c of level C (cell-centred positions; coarse cells outside the level count as zero).
__device__ __forceinline__ double dm_prolong_at(const DmLevel& C, const double* __restrict__ c, int j, int i) {
  const int J = j >> 1, I = i >> 1;
  const int J2 = J + ((j & 1) ? 1 : -1), I2 = I + ((i & 1) ? 1 : -1);
  auto cv = [&](int jj, int ii) -> double {
    return (ii >= 0 && ii < C.Nx && jj >= 0 && jj < C.Ny) ? c[dm_at(C, jj, ii)] : 0.0;
  };
  return 0.5625 * cv(J, I) + 0.1875 * (cv(J, I2) + cv(J2, I)) + 0.0625 * cv(J2, I2);
}

// ---- the small levels of a V-cycle in one workgroup, in LDS
// From the first level whose planes and those of every coarser level fit in
// kDmSmallLds bytes, the V-cycle down to the coarsest level and back up runs in one
// workgroup of kDmSmallThreads on LDS copies of those planes, phase by phase with a
// barrier between phases, in the arithmetic of the per-level launches. It is a chain of
// some ten phases per level, each as long as its longest thread, so a thread's sites
// come without a division (rows of lanes as wide as the level, a power of two, so that
// a narrow level fills the lanes too) and the operator's factor is a product. The
// level's rhs is read from global memory at the start and psi written back at the end
// (with the r.z partial where it is level 0). From 32^2 down 12.5 us; with whole waves
// to a row, a division in the operator and the sweep from zero as a phase of its own
// 20.7, and on narrow levels (14 x 156) several times that. From 64^2 down, which
// 160 KB would hold, 24.4 us: more than the 9 of the two launches that it saves.
constexpr int kDmSmallThreads = 1024;
constexpr int kDmSmallLds = 64 * 1024;

struct DmHierarchy {
  DmLevel lv[kDmMaxLevels];
  int nlev;
  // inverse of Laplace_h on the coarsest level (cn x cn, row-major, sites
  // numbered row-major over the interior), or cn = 0 for Jacobi sweeps there
  const double* cinv;
  int cn;
  int off[kDmMaxLevels];  // a level's three planes in LDS, from the first small level's
};

// LDS bytes of levels l .. nlev - 1 (three padded planes each)
__host__ __device__ inline long dm_small_bytes(const DmLevel* lv, int nlev, int l) {
  long n = 0;
  for (int k = l; k < nlev; ++k) n += 3L * (lv[k].Nx + 4) * (lv[k].Ny + 4);
  return 8 * n;
}

// Sum of the workgroup's values in a fixed order (wave sums in wave order); valid
// in every thread. red: blockDim / 64 doubles.
__device__ __forceinline__ double dm_block_sum(double v, double* red) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
  for (int k = 0; k < (int)(blockDim.x >> 6); ++k) s += red[k];
  return s;
}

// Sums of n[m] partials part[m] by a workgroup of 256, each in a fixed order, for every
// thread. The loads of four strides of every sum are in flight together: one after the
// other, the 1024 partials of a dot product on 512^2 cost their launch 2-3 us. red: 4 N
// doubles that nothing else uses.
template <int N>
__device__ __forceinline__ void dm_partials(const double* const (&part)[N], const int (&n)[N], double (&v)[N],
                                            double* red) {
  constexpr int U = 4;
  int top = 0;
#pragma unroll
  for (int m = 0; m < N; ++m) {
    v[m] = 0.0;
    top = n[m] > top ? n[m] : top;
  }
  for (int k0 = 0; k0 < top; k0 += 256 * U) {
    double p[N][U];
#pragma unroll
    for (int m = 0; m < N; ++m)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = k0 + 256 * u + threadIdx.x;
        p[m][u] = part[m][k < n[m] ? k : 0];
      }
#pragma unroll
    for (int m = 0; m < N; ++m)
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (k0 + 256 * u + (int)threadIdx.x < n[m]) v[m] += p[m][u];
  }
#pragma unroll
  for (int m = 0; m < N; ++m) {
    v[m] = wave_sum(v[m]);
    if ((threadIdx.x & 63) == 0) red[4 * m + (threadIdx.x >> 6)] = v[m];
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < N; ++m) {
    v[m] = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) v[m] += red[4 * m + k];
  }
}

static __global__ void __launch_bounds__(kDmSmallThreads) dm_vcycle_small(DmHierarchy H, int l0,
                                                                          double* __restrict__ part,
                                                                          const DevStatus* st) {
  if (dm_skip(st)) return;
  extern __shared__ double smem[];
  __shared__ double red[kDmSmallThreads / 64];
  const int last = H.nlev - 1;
  // the LDS copy of level l, a value built per use, so that no array of levels is
  // indexed at run time
  auto lds_level = [&](int l) {
    DmLevel L = H.lv[l];
    const int pl = (L.Nx + 4) * (L.Ny + 4);
    L.psi = smem + H.off[l];
    L.tmp = L.psi + pl;
    L.rhs = L.tmp + pl;
    return L;
  };
  // body(j, i, o) for every interior site of a level, o its offset in a plane: 2^w
  // lanes, up to a wave, along a row
  auto sites = [&](const DmLevel& L, auto&& body) {
    const int w = L.Nx > 32 ? 6 : L.Nx > 16 ? 5 : L.Nx > 8 ? 4 : 3;
    for (int j = threadIdx.x >> w; j < L.Ny; j += kDmSmallThreads >> w)
      for (int i = threadIdx.x & ((1 << w) - 1); i < L.Nx; i += 64) body(j, i, (j + 2) * (int)L.pitch + i + 2);
  };
  auto jacobi = [&](const DmLevel& L, const double* src, double* dst) {
    const double s = kDmOmega * L.h * L.h / 5.0;
    sites(L, [&](int j, int i, int o) { dst[o] = src[o] - s * (L.rhs[o] - dm_lap(src, L.pitch, j, i, L.lap)); });
    __syncthreads();
  };
  {
    // every plane zero, halos included, but the first level's rhs, whose loads are
    // issued before that
    const DmLevel G = H.lv[l0], L0 = lds_level(l0);
    const int pl = (G.Nx + 4) * (G.Ny + 4), total = (int)(dm_small_bytes(H.lv, H.nlev, l0) / 8);
    const int row = (int)G.pitch;
    auto interior = [&](int k) {
      const int j = k / row - 2, i = k - (j + 2) * row - 2;
      return i >= 0 && i < G.Nx && j >= 0 && j < G.Ny ? G.rhs[k] : 0.0;
    };
    constexpr int Q = 2;
    double v[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int k = threadIdx.x + q * kDmSmallThreads;
      v[q] = k < pl ? interior(k) : 0.0;
    }
    for (int k = threadIdx.x; k < 2 * pl; k += kDmSmallThreads) smem[k] = 0.0;
    for (int k = 3 * pl + threadIdx.x; k < total; k += kDmSmallThreads) smem[k] = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int k = threadIdx.x + q * kDmSmallThreads;
      if (k < pl) L0.rhs[k] = v[q];
    }
    for (int k = threadIdx.x + Q * kDmSmallThreads; k < pl; k += kDmSmallThreads) L0.rhs[k] = interior(k);
    __syncthreads();
  }
  for (int l = l0; l < last; ++l) {
    const DmLevel F = lds_level(l);
    const DmLevel C = lds_level(l + 1);
    // two sweeps from zero, the first of which is x = -s rhs; rhs is read as it is
    // needed for it (its halo is zero)
    const double s = kDmOmega * F.h * F.h / 5.0;
    sites(F, [&](int, int, int o) {
      const int p = (int)F.pitch;
      auto x = [&](int k) { return -(s * F.rhs[o + k]); };
      const double sx = -(x(-2) + x(2)) + 16.0 * (x(-1) + x(1));
      const double sy = -(x(-2 * p) + x(2 * p)) + 16.0 * (x(-p) + x(p));
      F.psi[o] = x(0) - s * (F.rhs[o] - (sx + sy - 60.0 * x(0)) * F.lap);
    });
    __syncthreads();
    sites(F, [&](int j, int i, int o) { F.tmp[o] = F.rhs[o] - dm_lap(F.psi, F.pitch, j, i, F.lap); });
    __syncthreads();
    sites(C, [&](int J, int I, int o) {
      // rows and columns outside the level carry the zeros of the halo
      double acc = 0.0;
#pragma unroll
      for (int a = -1; a <= 2; ++a) {
        const double* p = F.tmp + (2 * J + a + 2) * (int)F.pitch + 2 * I + 2;
        acc += dm_w(a, 0) * (((0.25 * p[-1] + 0.75 * p[0]) + 0.75 * p[1]) + 0.25 * p[2]);
      }
      C.rhs[o] = 0.25 * acc;
    });
    __syncthreads();
  }
  const DmLevel B = lds_level(last);
  if (H.cn > 0) {
    // the coarsest level solved exactly: psi = (Laplace_h)^-1 rhs, each row summed in site order
    for (int k = threadIdx.x; k < H.cn; k += kDmSmallThreads) {
      double acc = 0.0;
      int m = 0;
      for (int jm = 0; jm < B.Ny; ++jm)
        for (int im = 0; im < B.Nx; ++im, ++m) acc += H.cinv[(long)k * H.cn + m] * B.rhs[dm_at(B, jm, im)];
      const int jk = k / B.Nx, ik = k - jk * B.Nx;
      B.psi[dm_at(B, jk, ik)] = acc;
    }
    __syncthreads();
  } else {
    for (int k = 0; k < kDmCoarse; k += 2) {
      jacobi(B, B.psi, B.tmp);
      jacobi(B, B.tmp, B.psi);
    }
  }
  for (int l = last - 1; l >= l0; --l) {
    const DmLevel F = lds_level(l);
    const DmLevel C = lds_level(l + 1);
    sites(F, [&](int j, int i, int o) { F.psi[o] += dm_prolong_at(C, C.psi, j, i); });
    __syncthreads();
    jacobi(F, F.psi, F.tmp);
    jacobi(F, F.tmp, F.psi);
  }
  const DmLevel G = H.lv[l0], L0 = lds_level(l0);
  double rz = 0.0;
  sites(G, [&](int, int, int o) {
    const double z = L0.psi[o];
    G.psi[o] = z;
    rz -= L0.rhs[o] * z;
  });
  if (l0 == 0) {
    rz = dm_block_sum(rz, red);
    if (threadIdx.x == 0) part[0] = rz;
  }
}

// ---- the large levels: two launches per level and V-cycle
// Down: pre-smoothing (two sweeps from zero) and the restricted residual. Up: the
// prolonged correction and post-smoothing (two sweeps). Weighted Jacobi:
// x' = x - omega h^2/5 (rhs - Laplace_h x) (the operator's diagonal is -5/h^2), on
// interior sites only; halos stay zero. Both work on 16 x 16 fine sites per
// workgroup through LDS, with the halo that the sweeps need computed again.
constexpr int kDmTile = 16;                // fine sites per side of a tile
constexpr int kDmCT = kDmTile / 2;         // coarse sites per side
constexpr int kDmRF = kDmTile + 2;         // down: fine residuals per side
constexpr int kDmSF = kDmRF + 4;           //       smoothed psi
constexpr int kDmBF = kDmSF + 4;           //       rhs (and the first sweep)
constexpr int kDmTA = kDmTile + 8;         // up: the input
constexpr int kDmTB = kDmTile + 4;         //     after one sweep, and rhs
constexpr int kDmTC = kDmTA / 2 + 2;       //     coarse correction

// tiles of a level: each covers kDmTile sites (an odd last site starts a tile of its own)
__host__ __device__ inline int dm_tiles(const DmLevel& L) {
  return ((L.Nx + kDmTile - 1) / kDmTile) * ((L.Ny + kDmTile - 1) / kDmTile);
}

// A launch's item as a tile: workgroups whose numbers agree mod 8 share an XCD and its
// L2, and take tiles of one band of the level, so that neighbours' halos meet there (a
// 16 x 16 tile's launch reads 2.6 times its sites): a step on 512^2 FP32 147 -> 136 us, on
// 64^2 as before.
// The grid is a multiple of 8; items past the last tile (dm_items is the next multiple
// of 8) have none.
__host__ __device__ inline int dm_items(int nt) { return (nt + 7) / 8 * 8; }
__device__ __forceinline__ int dm_tile_of(int item, int nt) { return (item & 7) * ((nt + 7) / 8) + (item >> 3); }

// Coarse rhs = P^T (rhs - Laplace_h x) / 4 with x the two sweeps from zero, which is
// kept in F.tmp. A tile is kDmTile fine sites (2 Y0, 2 X0) .., i.e. kDmCT coarse sites.
// UPDATE (level 0): rhs is first renewed as the end of a conjugate-gradient iteration,
// x += alpha d and rhs' = rhs + alpha Ad (-r' of r' = r - alpha Ad) into the other
// plane, alpha = r.z / d.Ad summed from the partials by every workgroup (0 once d.Ad is
// 0: the residual has vanished); workgroup 0 keeps r.z for the next iteration's beta.
template <bool UPDATE>
__global__ void __launch_bounds__(256) dm_down(DmLevel F, DmLevel C, DmVecs D, int cur, int nrz, int nmv,
                                               const DevStatus* st) {
  if (dm_skip(st)) return;
  constexpr int NB = kDmBF * kDmBF, NS = kDmSF * kDmSF, NR = kDmRF * kDmRF, NC = kDmCT * kDmCT;
  __shared__ double b[NB];
  __shared__ double x1[NB];
  __shared__ double x2[NS];
  __shared__ double res[NR];
  __shared__ double red[8];
  const double s = kDmOmega * F.h * F.h / 5.0;
  const int ntx = (F.Nx + kDmTile - 1) / kDmTile;
  const int nt = dm_tiles(F);
  auto inside = [&](int j, int i) { return j >= 0 && j < F.Ny && i >= 0 && i < F.Nx; };
  double alpha = 0.0;
  bool first = true;
  for (int item = blockIdx.x; item < dm_items(nt); item += gridDim.x) {
    const int t = dm_tile_of(item, nt);
    if (t >= nt) continue;
    const int y0 = (t / ntx) * kDmTile, x0 = (t % ntx) * kDmTile;
    const double* __restrict__ rhs = UPDATE ? D.rhs[cur] : F.rhs;
    constexpr int QB = (NB + 255) / 256;
    double vb[QB], va[QB];
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int k = threadIdx.x + 256 * q;
      const int ly = k / kDmBF, lx = k - ly * kDmBF;
      const int j = y0 - 5 + ly, i = x0 - 5 + lx;
      const bool in = k < NB && inside(j, i);
      vb[q] = in ? rhs[dm_at(F, j, i)] : 0.0;
      va[q] = (UPDATE && in) ? D.Ad[dm_at(F, j, i)] : 0.0;
    }
    double vx = 0.0, vd = 0.0;  // the thread's own site of the tile
    const int oy = threadIdx.x / kDmTile, ox = threadIdx.x - oy * kDmTile;
    const bool own = inside(y0 + oy, x0 + ox);
    const long oo = dm_at(F, y0 + oy, x0 + ox);
    if (UPDATE && own) {
      vx = D.x[oo];
      vd = D.d[cur][oo];
    }
    if (UPDATE && first) {
      double v[2];  // r.z, d.Ad
      dm_partials({D.part, D.pmv}, {nrz, nmv}, v, red);
      alpha = v[1] > 0.0 ? v[0] / v[1] : 0.0;
      if (blockIdx.x == 0 && threadIdx.x == 0) D.sc[0] = v[0];
      first = false;
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int k = threadIdx.x + 256 * q;
      if (k < NB) {
        const double v = UPDATE ? vb[q] + alpha * va[q] : vb[q];
        b[k] = v;
        x1[k] = -(s * v);
      }
    }
    __syncthreads();
    if (UPDATE && own) {
      D.x[oo] = vx + alpha * vd;
      D.rhs[cur ^ 1][oo] = b[(oy + 5) * kDmBF + ox + 5];
    }
#pragma unroll
    for (int q = 0; q < (NS + 255) / 256; ++q) {
      const int k = threadIdx.x + 256 * q;
      if (k < NS) {
        const int ly = k / kDmSF, lx = k - ly * kDmSF;
        const int o = (ly + 2) * kDmBF + lx + 2;
        x2[k] = inside(y0 - 3 + ly, x0 - 3 + lx) ? x1[o] - s * (b[o] - dm_lap(x1, kDmBF, ly, lx, F.lap)) : 0.0;
      }
    }
    __syncthreads();
    if (own) F.tmp[oo] = x2[(oy + 3) * kDmSF + ox + 3];
#pragma unroll
    for (int q = 0; q < (NR + 255) / 256; ++q) {
      const int k = threadIdx.x + 256 * q;
      if (k < NR) {
        const int ly = k / kDmRF, lx = k - ly * kDmRF;
        res[k] = inside(y0 - 1 + ly, x0 - 1 + lx)
                     ? b[(ly + 4) * kDmBF + lx + 4] - dm_lap(x2, kDmSF, ly, lx, F.lap) : 0.0;
      }
    }
    __syncthreads();
    if (threadIdx.x < NC) {
      const int cy = threadIdx.x / kDmCT, cx = threadIdx.x - cy * kDmCT;
      const int J = y0 / 2 + cy, I = x0 / 2 + cx;
      if (J < C.Ny && I < C.Nx) {
        double acc = 0.0;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const double* p = res + (2 * cy + a) * kDmRF + 2 * cx;
          acc += dm_w(a - 1, 0) * (((0.25 * p[0] + 0.75 * p[1]) + 0.75 * p[2]) + 0.25 * p[3]);
        }
        C.rhs[dm_at(C, J, I)] = 0.25 * acc;
      }
    }
    __syncthreads();
  }
}

// psi = two sweeps of F.tmp + P (C.psi) against rhs. DOT (level 0): also the
// workgroup's partial of r.z (r = -rhs, z = psi).
template <bool DOT>
__global__ void __launch_bounds__(256) dm_up(DmLevel F, DmLevel C, const double* __restrict__ rhs,
                                             double* __restrict__ part, const DevStatus* st) {
  if (dm_skip(st)) return;
  constexpr int NA = kDmTA * kDmTA, NB = kDmTB * kDmTB, NCC = kDmTC * kDmTC;
  __shared__ double a[NA];
  __shared__ double b[NB];
  __shared__ double r[NB];
  __shared__ double cc[NCC];
  __shared__ double red[4];
  const double s = kDmOmega * F.h * F.h / 5.0;
  const int ntx = (F.Nx + kDmTile - 1) / kDmTile;
  const int nt = dm_tiles(F);
  auto inside = [&](int j, int i) { return j >= 0 && j < F.Ny && i >= 0 && i < F.Nx; };
  double rz = 0.0;
  for (int item = blockIdx.x; item < dm_items(nt); item += gridDim.x) {
    const int t = dm_tile_of(item, nt);
    if (t >= nt) continue;
    const int y0 = (t / ntx) * kDmTile, x0 = (t % ntx) * kDmTile;
    const int cy0 = y0 / 2 - 3, cx0 = x0 / 2 - 3;  // first coarse row and column of cc
    constexpr int QA = (NA + 255) / 256, QB = (NB + 255) / 256;
    double va[QA], vr[QB], vc = 0.0;
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int k = threadIdx.x + 256 * q;
      const int ly = k / kDmTA, lx = k - ly * kDmTA;
      const int j = y0 - 4 + ly, i = x0 - 4 + lx;
      va[q] = (k < NA && inside(j, i)) ? F.tmp[dm_at(F, j, i)] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int k = threadIdx.x + 256 * q;
      const int ly = k / kDmTB, lx = k - ly * kDmTB;
      const int j = y0 - 2 + ly, i = x0 - 2 + lx;
      vr[q] = (k < NB && inside(j, i)) ? rhs[dm_at(F, j, i)] : 0.0;
    }
    static_assert(NCC <= 256, "one coarse value per thread");
    if (threadIdx.x < NCC) {
      const int ly = threadIdx.x / kDmTC, lx = threadIdx.x - ly * kDmTC;
      const int J = cy0 + ly, I = cx0 + lx;
      if (J >= 0 && J < C.Ny && I >= 0 && I < C.Nx) vc = C.psi[dm_at(C, J, I)];
      cc[threadIdx.x] = vc;
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int k = threadIdx.x + 256 * q;
      if (k < NB) r[k] = vr[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < QA; ++q) {
      const int k = threadIdx.x + 256 * q;
      if (k < NA) {
        const int ly = k / kDmTA, lx = k - ly * kDmTA;
        const int j = y0 - 4 + ly, i = x0 - 4 + lx;
        // (P c)(j, i), as dm_prolong_at
        const double* c0 = cc + ((j >> 1) - cy0) * kDmTC + ((i >> 1) - cx0);
        const int dj = (j & 1) ? kDmTC : -kDmTC, di = (i & 1) ? 1 : -1;
        a[k] = inside(j, i)
                   ? va[q] + (0.5625 * c0[0] + 0.1875 * (c0[di] + c0[dj]) + 0.0625 * c0[dj + di]) : 0.0;
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int k = threadIdx.x + 256 * q;
      if (k < NB) {
        const int ly = k / kDmTB, lx = k - ly * kDmTB;
        b[k] = inside(y0 - 2 + ly, x0 - 2 + lx)
                   ? a[(ly + 2) * kDmTA + (lx + 2)] - s * (r[k] - dm_lap(a, kDmTA, ly, lx, F.lap)) : 0.0;
      }
    }
    __syncthreads();
    const int ly = threadIdx.x / kDmTile, lx = threadIdx.x - ly * kDmTile;
    if (inside(y0 + ly, x0 + lx)) {
      const int o = (ly + 2) * kDmTB + (lx + 2);
      const double z = b[o] - s * (r[o] - dm_lap(b, kDmTB, ly, lx, F.lap));
      F.psi[dm_at(F, y0 + ly, x0 + lx)] = z;
      if (DOT) rz -= r[o] * z;
    }
    __syncthreads();
  }
  if (DOT) {
    rz = dm_block_sum(rz, red);
    if (threadIdx.x == 0) part[blockIdx.x] = rz;
  }
}

// Direction and operator in one launch: d' = z + beta d on the tile and a halo of two
// (into the other plane), Ad = -Laplace_h d' and the workgroup's partial of d'.Ad.
// beta = r.z / (r.z of the last iteration) (0 on the first iteration or once that is
// 0), r.z summed from the partials by every workgroup.
static __global__ void __launch_bounds__(256) dm_direction(DmLevel L0, DmVecs D, int cur, int first, int nrz,
                                                           const DevStatus* st) {
  if (dm_skip(st)) return;
  constexpr int NB = kDmTB * kDmTB, QB = (NB + 255) / 256;
  __shared__ double b[NB];
  __shared__ double red[4], redp[4];
  const int ntx = (L0.Nx + kDmTile - 1) / kDmTile;
  const int nt = dm_tiles(L0);
  auto inside = [&](int j, int i) { return j >= 0 && j < L0.Ny && i >= 0 && i < L0.Nx; };
  double beta = 0.0, acc = 0.0;
  bool head = first == 0;
  for (int item = blockIdx.x; item < dm_items(nt); item += gridDim.x) {
    const int t = dm_tile_of(item, nt);
    if (t >= nt) continue;
    const int y0 = (t / ntx) * kDmTile, x0 = (t % ntx) * kDmTile;
    double vz[QB], vd[QB];
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int k = threadIdx.x + 256 * q;
      const int ly = k / kDmTB, lx = k - ly * kDmTB;
      const int j = y0 - 2 + ly, i = x0 - 2 + lx;
      const bool in = k < NB && inside(j, i);
      vz[q] = in ? L0.psi[dm_at(L0, j, i)] : 0.0;
      vd[q] = (!first && in) ? D.d[cur ^ 1][dm_at(L0, j, i)] : 0.0;
    }
    if (head) {
      double v[1];
      const double last = D.sc[0];
      dm_partials({D.part}, {nrz}, v, redp);
      beta = last == 0.0 ? 0.0 : v[0] / last;
      head = false;
    }
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int k = threadIdx.x + 256 * q;
      if (k < NB) b[k] = first ? vz[q] : vz[q] + beta * vd[q];
    }
    __syncthreads();
    const int ly = threadIdx.x / kDmTile, lx = threadIdx.x - ly * kDmTile;
    if (inside(y0 + ly, x0 + lx)) {
      const double d = b[(ly + 2) * kDmTB + lx + 2];
      const double ad = -dm_lap(b, kDmTB, ly, lx, L0.lap);
      const long o = dm_at(L0, y0 + ly, x0 + lx);
      D.d[cur][o] = d;
      D.Ad[o] = ad;
      acc += d * ad;
    }
    __syncthreads();
  }
  acc = dm_block_sum(acc, red);
  if (threadIdx.x == 0) D.pmv[blockIdx.x] = acc;
}

// The end of an iteration where no dm_down<true> follows: x += alpha d, and (more != 0)
// rhs += alpha Ad into the other plane. alpha as there.
static __global__ void __launch_bounds__(256) dm_update(DmLevel L0, DmVecs D, int cur, int more, int nrz, int nmv,
                                                        const DevStatus* st) {
  if (dm_skip(st)) return;
  __shared__ double red[8];
  double v[2];  // r.z, d.Ad
  dm_partials({D.part, D.pmv}, {nrz, nmv}, v, red);
  const double alpha = v[1] > 0.0 ? v[0] / v[1] : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) D.sc[0] = v[0];
  DM_SITES(L0) {
    const int j = (int)(k_ / L0.Nx), i = (int)(k_ - (long)j * L0.Nx);
    const long o = dm_at(L0, j, i);
    D.x[o] += alpha * D.d[cur][o];
    if (more) D.rhs[cur ^ 1][o] = D.rhs[cur][o] + alpha * D.Ad[o];
  }
}

// Start of a solve for the stage point a pass evaluates: rhs = -r of r = b - A x with
// b = -(d_x S_1 + d_y S_2) and A = -Laplace_h (the V-cycle solves Laplace_h z = -r),
// x the last potential. The stage point is formed as the pass forms it
// (phi + cv v + ca a, put on the unit sphere at interior sites when the pass moves the
// field) on the tile and its halo of two, in LDS. For an evaluation the field is `src`
// or, when that is null, the current field. The launch takes the flow's pending test
// (Link) and is skipped once a flow has stopped, as the pass itself is.
template <class T, int PASS>
__global__ void __launch_bounds__(256) dm_begin(Bufs<T> B, Coeffs cf, Link link, const T* __restrict__ src,
                                                DmLevel L0, DmVecs D) {
  __shared__ double red[12];
  constexpr int NB = kDmTB * kDmTB, QB = (NB + 255) / 256;
  __shared__ T s1[NB];
  __shared__ T s2[NB];
  __shared__ double xs[NB];
  const int ntx = (L0.Nx + kDmTile - 1) / kDmTile;
  const int nt = dm_tiles(L0);
  // a tile's potential; the first tile's while the test is taken
  double xv[QB];
  auto load_x = [&](int t) {
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int k = threadIdx.x + 256 * q;
      const int ly = k / kDmTB, lx = k - ly * kDmTB;
      const int j = (t / ntx) * kDmTile - 2 + ly, i = (t % ntx) * kDmTile - 2 + lx;
      xv[q] = k < NB && j >= 0 && j < L0.Ny && i >= 0 && i < L0.Nx ? D.x[dm_at(L0, j, i)] : 0.0;
    }
  };
  load_x(dm_tile_of(blockIdx.x, nt));
  Head hd = {};
  if (PASS == kEval) hd.step = link.st->step;
  else hd = resolve(link, cf.h * cf.h, threadIdx.x, red);
  if (PASS != kEval && hd.done) return;
  constexpr bool ONEPASS = advances_first(PASS);
  constexpr bool STAGED = staged(PASS);
  constexpr bool WITH_V = stage_reads_v(PASS);
  constexpr bool WITH_A = stage_reads_a(PASS);
  constexpr bool AFTER_P1 = (PASS == kP2 || PASS == kP3 || PASS == kP4);
  const int cur = uniform(AFTER_P1 ? int((hd.step - 1) & 1) : int(hd.step & 1));
  const bool arrest = uses_arrest(PASS) ? (uniform(hd.arrest) != 0) : false;
  const T dt = (T)cf.dt;
  T cv, ca;
  stage_coeffs<T, PASS>(dt, arrest, cv, ca);
  const T* __restrict__ ph = (PASS == kEval && src != nullptr) ? src : (cur ? B.phi[1] : B.phi[0]);
  const T* __restrict__ vv = cur ? B.vel[1] : B.vel[0];
  const T* __restrict__ aa = ONEPASS ? (cur ? B.a2 : B.a1) : (PASS == kP3) ? B.a1 : B.a2;
  const double c1 = 1.0 / (12.0 * L0.h);
  for (int item = blockIdx.x; item < dm_items(nt); item += gridDim.x) {
    const int t = dm_tile_of(item, nt);
    if (t >= nt) continue;
    if (item != (int)blockIdx.x) load_x(t);
    const int y0 = (t / ntx) * kDmTile, x0 = (t % ntx) * kDmTile;
#pragma unroll
    for (int q = 0; q < QB; ++q) {
      const int k = threadIdx.x + 256 * q;
      if (k >= NB) break;
      const int ly = k / kDmTB, lx = k - ly * kDmTB;
      const int j = y0 - 2 + ly, i = x0 - 2 + lx;  // the padded lattice ends at N + 1
      T S[3] = {T(0), T(0), T(0)};
      if (j <= L0.Ny + 1 && i <= L0.Nx + 1) {
        const long o = (long)(j + 2) * B.pitch + (i + 2);
        const bool in = j >= 0 && j < L0.Ny && i >= 0 && i < L0.Nx;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          if (!STAGED && c == 2) continue;
          T x = ph[c * B.plane + o];
          if (STAGED) {
            if (WITH_V) x += cv * vv[c * B.plane + o];
            if (WITH_A) x += ca * aa[c * B.plane + o];
          }
          S[c] = x;
        }
        if (STAGED && in) {
          const T inv = T(1) / sqrt(S[0] * S[0] + S[1] * S[1] + S[2] * S[2]);
          S[0] *= inv;
          S[1] *= inv;
        }
      }
      s1[k] = S[0];
      s2[k] = S[1];
      xs[k] = xv[q];
    }
    __syncthreads();
    const int ly = threadIdx.x / kDmTile, lx = threadIdx.x - ly * kDmTile;
    const int j = y0 + ly, i = x0 + lx;
    if (j < L0.Ny && i < L0.Nx) {
      const T* p1 = s1 + (ly + 2) * kDmTB + lx + 2;
      const T* p2 = s2 + (ly + 2) * kDmTB + lx + 2;
      const double dx = c1 * (((double)p1[-2] - (double)p1[2]) + 8.0 * ((double)p1[1] - (double)p1[-1]));
      const double dy = c1 * (((double)p2[-2 * kDmTB] - (double)p2[2 * kDmTB]) +
                              8.0 * ((double)p2[kDmTB] - (double)p2[-kDmTB]));
      const double r = -(dx + dy) + dm_lap(xs, kDmTB, ly, lx, L0.lap);
      D.rhs[0][dm_at(L0, j, i)] = -r;
    }
    __syncthreads();
  }
}

#undef DM_SITES

}  // namespace ss

// Definitions and instances of ss_launch.hpp for one element type and theory.
#pragma once

#include <algorithm>

#include "ss_launch.hpp"

namespace ss {

// Workgroups of one kernel resident on the whole GPU at once: the runtime's occupancy
// for one CU times the CUs.
inline long resident_of(const void* kernel, int threads) {
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess || per_cu < 1) {
    (void)hipGetLastError();  // a failed query must not surface as a launch error
    return kMaxGroups;
  }
  return std::min(kMaxGroups, kNumCUs * per_cu);
}

// Of one stage-pass instantiation, queried once, on the first device that launches it.
template <class T, int TH, int PASS, int TX, int TY, int RY>
long resident_groups() {
  static const long n = resident_of(reinterpret_cast<const void*>(&stage_pass<T, TH, PASS, TX, TY, RY>), TX * (TY / RY));
  return n;
}

// Launches a pass and returns its workgroup count. P1 runs with at most its
// resident workgroups, each walking longer column segments (on 4096^2 with
// 64 x 16 tiles: 512 groups, 0.184 -> 0.177 ms against 2048).
template <class T, int TH, int PASS, int CFG>
int launch_cfg(const PassArgs<T>& a, int nlaunch, hipStream_t s) {
  constexpr TileCfg tc = kTiles[CFG];
  PassArgs<T> b = a;
  if constexpr (PASS == kP1 || PASS == kPrime || advances_first(PASS) || fixed_tile(PASS) || PASS == kGD) {
    const long r = resident_groups<T, TH, PASS, tc.TX, tc.TY, tc.RY>();
    if (nlaunch > r) {
      nlaunch = (int)r;
      b.seg = choose_seg(a.ntx, a.nty, nlaunch);
    }
  }
  hipLaunchKernelGGL((stage_pass<T, TH, PASS, tc.TX, tc.TY, tc.RY>), dim3(nlaunch), dim3(tc.TX, tc.TY / tc.RY), 0,
                     s, b);
  return nlaunch;
}

template <class T, int TH, int PASS>
int launch_tiled(int tile, const PassArgs<T>& a, int nlaunch, hipStream_t s) {
  if constexpr (!fixed_tile(PASS)) {
    if (tile == 1) return launch_cfg<T, TH, PASS, 1>(a, nlaunch, s);
    if (tile == 2) return launch_cfg<T, TH, PASS, 2>(a, nlaunch, s);
    if (tile == 3) return launch_cfg<T, TH, PASS, 3>(a, nlaunch, s);
  }
  if constexpr (sizeof(T) == 8)
    if (tile == kSmallShape) return launch_cfg<T, TH, PASS, kSmallShape>(a, nlaunch, s);
  return launch_cfg<T, TH, PASS, 0>(a, nlaunch, s);
}

// With at most its resident workgroups, since each sums the pending test's partials, also
// where the flow has stopped and the pass returns: with one per tile, up to kMaxGroups, a
// relaxation of two steps on 1746 x 898 FP64 Abelian Higgs by gradient flow (62 passes
// after it has stopped) took 979 us, now 448; a step of velocity Verlet in FP32 73.4, now
// 68.2. An evaluation takes no test and keeps its grid.
template <class T, int TH, int PASS>
int launch_exact(const PassArgs<T>& a, int nlaunch, hipStream_t s) {
  PassArgs<T> b = a;
  if constexpr (PASS != kEval) {
    static const long resident = resident_of(reinterpret_cast<const void*>(&stage_pass_exact<T, TH, PASS>), 256);
    if (nlaunch > resident) {
      nlaunch = (int)resident;
      b.seg = choose_seg(a.ntx, a.nty, nlaunch);
    }
  }
  hipLaunchKernelGGL((stage_pass_exact<T, TH, PASS>), dim3(nlaunch), dim3(kExTX, kExTY / kExRY), 0, s, b);
  return nlaunch;
}

// The fused pass with at most its resident workgroups, each walking longer column
// segments, so that none waits for a free CU.
template <class T, int TH, int TY>
void launch_fused_cfg(const PassArgs<T>& a, int nlaunch, hipStream_t s) {
  static const long resident = resident_of(reinterpret_cast<const void*>(&stage_pass_fused<T, TH, 64, TY, 2>), 32 * TY);
  PassArgs<T> b = a;
  if (nlaunch > resident) {
    nlaunch = (int)resident;
    b.seg = choose_seg(a.ntx, a.nty, nlaunch);
  }
  hipLaunchKernelGGL((stage_pass_fused<T, TH, 64, TY, 2>), dim3(nlaunch), dim3(64, TY / 2), 0, s, b);
}

template <class T, int TH>
void launch_fused_t(int layout_tile, const PassArgs<T>& a, int nlaunch, hipStream_t s) {
  if constexpr (sizeof(T) == 4) {
    if (layout_tile == 0) return launch_fused_cfg<T, TH, 16>(a, nlaunch, s);
  }
  launch_fused_cfg<T, TH, 8>(a, nlaunch, s);
}

template <class T, int TH, int PASS, int CFG>
void batch_launch_cfg(const BatchArgs<T>& a, int nlaunch, hipStream_t s) {
  constexpr TileCfg tc = kTiles[CFG];
  hipLaunchKernelGGL((batch_pass<T, TH, PASS, tc.TX, tc.TY, tc.RY>), dim3(nlaunch), dim3(tc.TX, tc.TY / tc.RY), 0,
                     s, a);
}

template <class T, int TH, int PASS>
void batch_launch_t(int tile, const BatchArgs<T>& a, int nlaunch, hipStream_t s) {
  switch (tile) {
    case 0: batch_launch_cfg<T, TH, PASS, 0>(a, nlaunch, s); break;
    case 1: batch_launch_cfg<T, TH, PASS, 1>(a, nlaunch, s); break;
    case 2: batch_launch_cfg<T, TH, PASS, 2>(a, nlaunch, s); break;
    default: batch_launch_cfg<T, TH, PASS, 3>(a, nlaunch, s); break;
  }
}

template <class T, int TH>
void batch_launch_fused_t(int tile, const BatchArgs<T>& a, int nlaunch, hipStream_t s) {
  if constexpr (sizeof(T) == 4) {
    if (tile == 0) {
      hipLaunchKernelGGL((batch_pass_fused<T, TH, 64, 16, 2>), dim3(nlaunch), dim3(64, 8), 0, s, a);
      return;
    }
  }
  hipLaunchKernelGGL((batch_pass_fused<T, TH, 64, 8, 2>), dim3(nlaunch), dim3(64, 4), 0, s, a);
}

#define SS_LATTICE_PASS(T, TH, P)                                                       \
  template int launch_tiled<T, TH, P>(int, const PassArgs<T>&, int, hipStream_t);       \
  template int launch_exact<T, TH, P>(const PassArgs<T>&, int, hipStream_t);

// every pass of the lattice theories
#define SS_LATTICE_PASSES(T, TH)                                                        \
  SS_LATTICE_PASS(T, TH, kP1) SS_LATTICE_PASS(T, TH, kP2) SS_LATTICE_PASS(T, TH, kP3)   \
  SS_LATTICE_PASS(T, TH, kP4) SS_LATTICE_PASS(T, TH, kEval)                             \
  SS_LATTICE_PASS(T, TH, kCheck) SS_LATTICE_PASS(T, TH, kPrime)                         \
  SS_LATTICE_PASS(T, TH, kVVA) SS_LATTICE_PASS(T, TH, kVV)                              \
  SS_LATTICE_PASS(T, TH, kVVStart) SS_LATTICE_PASS(T, TH, kVVRestart)                   \
  SS_LATTICE_PASS(T, TH, kVVEnd) SS_LATTICE_PASS(T, TH, kGD)                            \
  SS_LATTICE_PASS(T, TH, kGDCheck)                                                      \
  template void launch_fused_t<T, TH>(int, const PassArgs<T>&, int, hipStream_t);

#define SS_BATCH_PASS(T, TH, P) \
  template void batch_launch_t<T, TH, P>(int, const BatchArgs<T>&, int, hipStream_t);

// every pass of a batch
#define SS_BATCH_PASSES(T, TH)                                                          \
  SS_BATCH_PASS(T, TH, kP1) SS_BATCH_PASS(T, TH, kP2) SS_BATCH_PASS(T, TH, kP3)         \
  SS_BATCH_PASS(T, TH, kP4) SS_BATCH_PASS(T, TH, kCheck) SS_BATCH_PASS(T, TH, kVV)      \
  SS_BATCH_PASS(T, TH, kVVStart) SS_BATCH_PASS(T, TH, kVVRestart)                       \
  SS_BATCH_PASS(T, TH, kVVEnd) SS_BATCH_PASS(T, TH, kGD) SS_BATCH_PASS(T, TH, kGDCheck) \
  template void batch_launch_fused_t<T, TH>(int, const BatchArgs<T>&, int, hipStream_t);

}  // namespace ss

// Launches of the lattice passes. The kernels of one element type and theory are
// compiled in a source file of their own (ss_pass_*.hip, from ss_pass.hpp), so
// that the library builds in parallel; the host code sees these declarations.
#pragma once

#include "ss_kernels.hpp"

namespace ss {

// Tile shapes compiled into the library: a workgroup covers TX x TY sites,
// each thread RY rows of one column. ss_autotune times them on the caller's
// lattice; SS_TILE (environment) or ss_set_tile force one.
struct TileCfg {
  int TX, TY, RY;
};
constexpr TileCfg kTiles[] = {{64, 16, 2}, {64, 8, 2}, {64, 16, 4}, {64, 32, 4}};
constexpr long kMaxGroups = 2048;  // persistent launch: at most 8 workgroups per CU
constexpr long kNumCUs = 256;

// A pass of the Euler-Lagrange form on tile shape `tile` with at most nlaunch
// workgroups (passes of fixed_tile: tile 0); returns its workgroup count.
template <class T, int TH, int PASS>
int launch_tiled(int tile, const PassArgs<T>& a, int nlaunch, hipStream_t s);

// A pass of the exact-gradient form.
template <class T, int TH, int PASS>
void launch_exact(const PassArgs<T>& a, int groups, hipStream_t s);

// Fused stages 2-4 on the layout of tile 0 (FP32 only) or 1.
template <class T, int TH>
void launch_fused_t(int layout_tile, const PassArgs<T>& a, int nlaunch, hipStream_t s);

// A pass, and fused stages 2-4, of a batch.
template <class T, int TH, int PASS>
void batch_launch_t(int tile, const BatchArgs<T>& a, int nlaunch, hipStream_t s);
template <class T, int TH>
void batch_launch_fused_t(int tile, const BatchArgs<T>& a, int nlaunch, hipStream_t s);

}  // namespace ss

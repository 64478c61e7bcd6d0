// Launches of the lattice passes. The kernels of one element type and theory are
// compiled in a source file of their own (ss_pass_*.hip, from ss_pass.hpp), so
// that the library builds in parallel; the host code sees these declarations.
#pragma once

#include <algorithm>

#include "ss_kernels.hpp"

namespace ss {

// Tile shapes compiled into the library: a workgroup covers TX x TY sites,
// each thread RY rows of one column. ss_autotune times them on the caller's
// lattice; SS_TILE (environment) or ss_set_tile force one.
struct TileCfg {
  int TX, TY, RY;
};
// The first kNumTiles are the caller's; kSmallShape (FP64 only) stands in for tile 0 on
// small lattices.
constexpr TileCfg kTiles[] = {{64, 16, 2}, {64, 8, 2}, {64, 16, 4}, {64, 32, 4}, {64, 4, 1}};
constexpr int kNumTiles = 4;
constexpr int kSmallShape = 4;
constexpr long kMaxGroups = 2048;  // persistent launch: at most 8 workgroups per CU
constexpr long kNumCUs = 256;

// Tiles per work unit (for_each_tile) for `groups` workgroups on ntx x nty tiles: the
// segments per tile column of the least estimated time. A round of units takes a
// unit's tiles and a quarter of one for the halo that its first tile reads itself,
// times one more than the workgroups that share a CU in it (two take less than twice
// the time of one). Cut by the mean number of tiles per group, rounded down, an odd
// lattice's units did not fit the groups: on 1000^2 (16 x 63 tiles) 336 units of 3 for
// 256 groups, two rounds, take 1.3 times as long per RK4 step as 256 units of 4 (72.7 and
// 55.7 us with the fused pass of then). The other way round, 528 tiles for 512 groups are
// best left single: gradient flow of baby Skyrme on 1021 x 517 takes 1.24 times as long
// in 272 units of 2.
inline int choose_seg(int ntx, int nty, int groups) {
  int best = nty;
  double best_cost = 1e300;
  for (int r = 1; r <= 8; ++r) {
    const long nseg0 = std::max<long>(1, std::min<long>(nty, (long)r * groups / ntx));
    const int seg = (int)((nty + nseg0 - 1) / nseg0);
    double cost = 0.0;
    for (long left = (long)ntx * ((nty + seg - 1) / seg); left > 0; left -= groups)
      cost += (seg + 0.25) * (1 + (std::min<long>(left, groups) + kNumCUs - 1) / kNumCUs);
    if (cost < best_cost) {
      best_cost = cost;
      best = seg;
    }
  }
  return best;
}

// A pass of the Euler-Lagrange form on tile shape `tile` with at most nlaunch
// workgroups (passes of fixed_tile: tile 0); returns its workgroup count.
template <class T, int TH, int PASS>
int launch_tiled(int tile, const PassArgs<T>& a, int nlaunch, hipStream_t s);

// A pass of the exact-gradient form, likewise.
template <class T, int TH, int PASS>
int launch_exact(const PassArgs<T>& a, int nlaunch, hipStream_t s);

// Fused stages 2-4 on the layout of tile 0 (FP32 only) or 1.
template <class T, int TH>
void launch_fused_t(int layout_tile, const PassArgs<T>& a, int nlaunch, hipStream_t s);

// A pass, and fused stages 2-4, of a batch.
template <class T, int TH, int PASS>
void batch_launch_t(int tile, const BatchArgs<T>& a, int nlaunch, hipStream_t s);
template <class T, int TH>
void batch_launch_fused_t(int tile, const BatchArgs<T>& a, int nlaunch, hipStream_t s);

}  // namespace ss

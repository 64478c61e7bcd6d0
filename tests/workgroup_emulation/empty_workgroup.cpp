// A workgroup without a tile (grids are rounded up to a multiple of 8 and dealt to the
// XCDs in bands): it takes the pending test like every other and adds nothing to its own
// pass, whatever the order its waves run in. Prints "ok", or the first order that went
// wrong.
#include "ss_kernels.hpp"

#include <algorithm>
#include <limits>

using namespace ss;

namespace {

// The pass `kernel` (TX x TY/RY threads) on a lattice of ntiles tiles, as workgroup 15 of
// 16, with a pending test whose largest |G|, in the partials that wave `top` sums, alone
// keeps the flow from its gradient tolerance.
template <class T, int PASS, class K>
bool check(const char* name, int threads_y, int ntiles, K kernel) {
  constexpr int kGroups = 16, kPending = 1024;
  std::vector<double> part(4 * kPending), out(4 * kGroups);
  DevStatus st, alt;
  std::vector<int> order(threads_y);
  for (int top = 0; top < 4; ++top) {
    for (int k = 0; k < threads_y; ++k) order[k] = k;
    do {
      memset(&st, 0, sizeof(st));
      memset(&alt, 0, sizeof(alt));
      st.E_prev = std::numeric_limits<double>::infinity();
      st.e_target = -std::numeric_limits<double>::infinity();
      st.grad_tol = 0.5;
      st.minimise = 1;
      st.max_steps = 1000;
      for (int k = 0; k < kPending; ++k) {
        part[4 * k] = 1.0;
        part[4 * k + 1] = k % 256 / 64 == top ? 1.0 : 0.25;
        part[4 * k + 2] = 0.0;
      }
      for (double& x : out) x = 7.0;  // a partial of an earlier pass
      PassArgs<T> a;
      memset(&a, 0, sizeof(a));
      a.B.Nx = 64;
      a.B.Ny = 16 * ntiles;
      a.cf.h = 0.5;
      a.cf.dt = 0.1;
      a.link = Link{&st, &st, &alt, part.data(), kPending, finalise_kind(PASS)};
      a.partials = out.data();
      a.ntx = 1;
      a.nty = ntiles;
      a.seg = 1;
      const bool ended = emu::run(dim3{64, (unsigned)threads_y, 1}, dim3{kGroups, 1, 1}, kGroups - 1, order, [&] { kernel(a); });
      const double* p = &out[4 * (kGroups - 1)];
      if (!ended || p[0] != 0.0 || p[1] != 0.0 || p[2] != 0.0) {
        printf("%s: %s, partial (%g, %g, %g), largest |G| with wave %d, waves in the order", name,
               ended ? "ended" : "hung", p[0], p[1], p[2], top);
        for (int k : order) printf(" %d", k);
        printf("\n");
        return false;
      }
    } while (std::next_permutation(order.begin(), order.begin() + 4));
  }
  return true;
}

}  // namespace

int main() {
  const bool ok =
      check<double, kVV>("velocity Verlet, 64 x 4, FP64", 4, 9, stage_pass<double, kAH, kVV, 64, 4, 1>) &&
      check<float, kGD>("gradient flow, 64 x 8, FP32", 4, 9, stage_pass<float, kCM, kGD, 64, 8, 2>) &&
      check<float, kP1>("stage 1, 64 x 16, FP32", 8, 9, stage_pass<float, kBS, kP1, 64, 16, 2>) &&
      check<double, kVVA>("exact gradient, FP64", 4, 9, stage_pass_exact<double, kAH, kVVA>);
  if (ok) printf("ok\n");
  return ok ? 0 : 1;
}

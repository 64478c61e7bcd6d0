// Lattice passes of the chiral magnet in FP64.
#include "ss_pass.hpp"

namespace ss {
SS_LATTICE_PASSES(double, kCM)
SS_BATCH_PASSES(double, kCM)
}  // namespace ss

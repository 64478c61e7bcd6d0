// Lattice passes of the chiral magnet in FP32.
#include "ss_pass.hpp"

namespace ss {
SS_LATTICE_PASSES(float, kCM)
SS_BATCH_PASSES(float, kCM)
}  // namespace ss

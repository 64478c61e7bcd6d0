// Lattice passes of the Baby Skyrme model in FP32.
#include "ss_pass.hpp"

namespace ss {
SS_LATTICE_PASSES(float, kBS)
}  // namespace ss

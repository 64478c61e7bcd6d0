// Lattice passes of the Baby Skyrme model in FP64.
#include "ss_pass.hpp"

namespace ss {
SS_LATTICE_PASSES(double, kBS)
}  // namespace ss

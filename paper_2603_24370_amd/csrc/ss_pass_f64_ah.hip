// Lattice passes of the Abelian Higgs model in FP64.
#include "ss_pass.hpp"

namespace ss {
SS_LATTICE_PASSES(double, kAH)
SS_BATCH_PASSES(double, kAH)
}  // namespace ss

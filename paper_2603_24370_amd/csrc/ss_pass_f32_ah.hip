// Lattice passes of the Abelian Higgs model in FP32.
#include "ss_pass.hpp"

namespace ss {
SS_LATTICE_PASSES(float, kAH)
SS_BATCH_PASSES(float, kAH)
}  // namespace ss

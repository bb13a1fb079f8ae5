// The substep by one workgroup per leaf, for small batches, in binary64
// storage: all three variants (plain, node copies, CFL minimum).
#include "octohydro_kernels.h"

namespace octohydro {

hipError_t launch_leaf_f64(const StepArgs& a, int mode, int blocks, hipStream_t st) {
  switch (mode) {
    case STEP_PLAIN: return launch_leaf_t<double, STEP_PLAIN>(a, blocks, st);
    case STEP_RESTRICT: return launch_leaf_t<double, STEP_RESTRICT>(a, blocks, st);
    case STEP_CFL: return launch_leaf_t<double, STEP_CFL>(a, blocks, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace octohydro

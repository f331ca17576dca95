// Collide-and-stream launches of the D3Q27 lattice in float: single steps and
// passes of two.
#include "step_kernel.h"
#include "step2_kernel.h"

namespace mclbm {

hipError_t launch_step_d3q27_f32(StepKind kind, const StepLaunch& L, hipStream_t s) {
  return launch_step_k<27, float>(kind, L, s);
}

hipError_t launch_step2_d3q27_f32(const Step2Launch& L, hipStream_t s) {
  return launch_step2_t<27, float>(L, s);
}

}  // namespace mclbm

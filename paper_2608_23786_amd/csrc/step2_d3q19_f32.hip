// Two-step passes of the D3Q19 lattice in float.
#include "step2_kernel.h"

namespace mclbm {

hipError_t launch_step2_d3q19_f32(const Step2Launch& L, hipStream_t s) {
  return launch_step2_t<19, float>(L, s);
}

}  // namespace mclbm

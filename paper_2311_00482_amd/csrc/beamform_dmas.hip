// Single-frame DMAS kernels (beamform_kernels.h).
#include <hip/hip_runtime.h>

#include "beamform_kernels.h"

namespace pwbf {

hipError_t launch_dmas(const FramePlan &P, hipStream_t stream) {
  return launch_mode<kDmas>(P, stream);
}

}  // namespace pwbf

// Single-frame pDAS kernels (beamform_kernels.h).
#include <hip/hip_runtime.h>

#include "beamform_kernels.h"

namespace pwbf {

hipError_t launch_pdas(const FramePlan &P, hipStream_t stream) {
  return launch_mode<kPdas>(P, stream);
}

}  // namespace pwbf

// Single-frame IQ-DAS kernels (beamform_kernels.h).
#include <hip/hip_runtime.h>

#include "beamform_kernels.h"

namespace pwbf {

hipError_t launch_iqdas(const FramePlan &P, hipStream_t stream) {
  return launch_mode<kIqdas>(P, stream);
}

}  // namespace pwbf

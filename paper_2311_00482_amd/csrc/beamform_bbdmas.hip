// Single-frame BB-DMAS kernels (beamform_kernels.h).
#include <hip/hip_runtime.h>

#include "beamform_kernels.h"

namespace pwbf {

hipError_t launch_bbdmas(const FramePlan &P, hipStream_t stream) {
  return launch_mode<kBbdmas>(P, stream);
}

}  // namespace pwbf

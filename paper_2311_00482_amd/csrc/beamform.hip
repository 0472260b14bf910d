// Single-frame launch of the beamformer, and the DAS kernels (beamform_kernels.h).
#include <hip/hip_runtime.h>

#include "beamform_kernels.h"

namespace pwbf {

hipError_t launch_dmas(const FramePlan &P, hipStream_t stream);
hipError_t launch_pdas(const FramePlan &P, hipStream_t stream);
hipError_t launch_iqdas(const FramePlan &P, hipStream_t stream);
hipError_t launch_bbdmas(const FramePlan &P, hipStream_t stream);

namespace {

__global__ void k_clear_max(uint32_t *slots) { dev::frame_max_clear(slots, threadIdx.x); }

}  // namespace

hipError_t launch_beamform(const FramePlan &P, hipStream_t stream) {
  if (is_iq_mode(P.mode) && P.ws_max) {
    hipLaunchKernelGGL(k_clear_max, dim3(1), dim3(kMaxSlots), 0, stream, P.ws_max);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  switch (P.mode) {
    case kDas: return launch_mode<kDas>(P, stream);
    case kDmas: return launch_dmas(P, stream);
    case kPdas: return launch_pdas(P, stream);
    case kIqdas: return launch_iqdas(P, stream);
    case kBbdmas: return launch_bbdmas(P, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace pwbf

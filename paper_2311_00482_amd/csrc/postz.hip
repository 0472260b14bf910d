// Depth-wise post-processing of a beamformed image, column by column.
//
// A column (nz samples, a power of two) is transformed (fft_reg.h), multiplied
// by the one-sided weights of the analytic signal (1 at DC and Nyquist, 2 for
// positive bins, 0 for negative ones) and, for the band-pass, by the brick-wall
// mask keeping the round-trip band [f0, 3 f0] (signed bins k_lo..k_hi), then
// transformed back. The real part of the result is the band-passed column; its
// magnitude is the envelope. The log image needs the frame maximum of the
// envelope: each wavefront folds its columns' maximum into the frame's maximum
// slots, and a second kernel maps every pixel to max(20 log10(env / max), floor).
//
// What bounds k_postz on one frame is latency: a launch, a read of the column,
// two transforms and a write, all blocks at once (a wavefront alone on its SIMD
// issues one instruction in about five cycles). Eight samples a thread in
// registers and no barrier up to 512 samples, instead of a 256-thread block per
// column with two barriers a pass: 512 columns of 512 samples 7.2 -> 4.6 us,
// 128 of 256 5.9 -> 4.6 us, 1024 of 1024 9.7 -> 8.2 us; in a batch of 16 frames
// 26 -> 14 us per branch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "postz_device.h"

namespace pwbf {

namespace {

template <int L>
__global__ void __launch_bounds__(post_block(L)) __attribute__((amdgpu_waves_per_eu(4)))
    k_postz(const PostPlan Q) {
  extern __shared__ __align__(16) float2 sm[];
  dev::postz_columns<L>(Q, (int)blockIdx.x * post_columns(L, post_block(L)), sm);
}

template <int L>
hipError_t launch_columns(const PostPlan &Q, hipStream_t stream) {
  const int per = post_columns(L, post_block(L));
  hipLaunchKernelGGL(k_postz<L>, dim3((Q.nx + per - 1) / per), dim3(post_block(L)),
                     dev::post_lds_bytes<L>(post_block(L)), stream, Q);
  return hipGetLastError();
}

__global__ void k_logc(const float *__restrict__ env, float *__restrict__ out,
                       const uint32_t *__restrict__ ws_max, size_t n, float floor_db) {
  const float m = dev::frame_max_read(ws_max);
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    out[i] = dev::log_db(env[i], m, floor_db);
}

// four pixels per thread through 16-byte loads and stores (n4 = n / 4)
__global__ void k_logc4(const float4 *__restrict__ env, float4 *__restrict__ out,
                        const uint32_t *__restrict__ ws_max, size_t n4, float floor_db) {
  const float m = dev::frame_max_read(ws_max);
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4;
       i += (size_t)gridDim.x * blockDim.x) {
    const float4 e = env[i];
    out[i] = make_float4(dev::log_db(e.x, m, floor_db), dev::log_db(e.y, m, floor_db),
                         dev::log_db(e.z, m, floor_db), dev::log_db(e.w, m, floor_db));
  }
}

}  // namespace

hipError_t launch_logc(const float *env, float *logimg, const uint32_t *ws_max, size_t n,
                       float floor_db, hipStream_t stream) {
  const int threads = 256;
  if (n % 4 == 0 && (uintptr_t)env % 16 == 0 && (uintptr_t)logimg % 16 == 0) {
    const size_t n4 = n / 4;
    const int blocks = (int)std::min<size_t>((n4 + threads - 1) / threads, 1024);
    hipLaunchKernelGGL(k_logc4, dim3(blocks), dim3(threads), 0, stream, (const float4 *)env,
                       (float4 *)logimg, ws_max, n4, floor_db);
  } else {
    const int blocks = (int)std::min<size_t>((n + threads - 1) / threads, 4096);
    hipLaunchKernelGGL(k_logc, dim3(blocks), dim3(threads), 0, stream, env, logimg, ws_max, n,
                       floor_db);
  }
  return hipGetLastError();
}

hipError_t launch_post(const PostPlan &Q, hipStream_t stream) {
  hipError_t e = hipErrorInvalidValue;
  switch (Q.log2nz) {
#define PWBF_POST(L) \
  case L: e = launch_columns<L>(Q, stream); break;
    PWBF_POST(1) PWBF_POST(2) PWBF_POST(3) PWBF_POST(4) PWBF_POST(5) PWBF_POST(6)
    PWBF_POST(7) PWBF_POST(8) PWBF_POST(9) PWBF_POST(10) PWBF_POST(11) PWBF_POST(12)
#undef PWBF_POST
    default: break;
  }
  if (e != hipSuccess || !Q.logimg) return e;
  return launch_logc(Q.env, Q.logimg, Q.ws_max, (size_t)Q.nx * Q.nz, Q.floor_db, stream);
}

}  // namespace pwbf

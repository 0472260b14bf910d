#pragma once
// The single-frame beamform kernel and its launch for one beamformer: one block
// per pixel tile. The tile body (staging, delays, gather, reductions) lives in
// beamform_device.h; each beamformer's kernels are compiled in a source of their
// own (beamform.hip, beamform_dmas.hip, ...).
//
// Tiles run deepest row first: a tile's cost grows with the receive aperture,
// which widens with depth, so the costliest tiles start first and the cheap
// shallow ones fill the end of the launch. Consecutive block ids go
// round-robin to the 8 XCDs, so every XCD takes every 8th tile of each tile
// row: an equal share of every depth.
#include <hip/hip_runtime.h>

#include "beamform_device.h"

namespace pwbf {

namespace {

// Wavefronts per SIMD the register allocation leaves room for: six (80 registers), so
// that three 8-wavefront blocks fit a CU as the default LDS budget lets them, where the
// unrolled angles fit without being read one after another; else four (128).
//   DAS: six up to 11 angles, 8 in several lane groups (512 x 512 pixels of 128
//   channels, 16 x 32 tiles, 16 angles: 66 us at 95 registers, 89 at 80; 11 angles in
//   four groups 81 and 91), and for 13 to 16 angles of wavefronts that share pixels
//   where the launch fills those three blocks twice (16 angles of 128 channels, 1000 x
//   1000: 178 us at 80 registers, 194 at 128; 384 x 384: 43 and 34).
//   DMAS, pDAS: six up to 12 (14-angle DMAS 85 us at 115 registers, 92 at 80), in
//   several lane groups up to 16 (106 and 90), except that blocks of four wavefronts
//   or fewer cannot fill the registers so (133 and 142).
//   IQ: six up to 11, two sums and a transmit delay each (1024 x 1024 IQ-DAS 222 us at
//   108 registers, 185 at 80 with the entries read four at a time; BB-DMAS 311 and
//   277), with up to 40 bytes a lane spilled outside the gather loop. In several lane
//   groups, whose addresses differ by lane, the loop itself would spill from five
//   angles on: four (11 angles, 512 x 512, two groups: 82 us, 111 at 80 registers, 98
//   without a bound). The predicated kernels hold 64 sums and 32 transmit delays and
//   get 256 registers (17 angles, 384 x 384, 173 us at 165 registers, 1006 at 128 with
//   696 bytes spilled).
constexpr int min_waves(int am, bool pred, int mode, int group) {
  const bool groups = dev::lane_groups(group);
  if (is_iq_mode(mode)) return pred ? 2 : (am <= (groups ? 4 : 11) ? 6 : 4);
  if (mode == kDas) return am <= (groups ? 8 : 11) ? 6 : 4;
  return am <= (groups ? 16 : 12) ? 6 : 4;
}

template <int AM, bool PRED, int MODE, int GROUP, int WAVES = min_waves(AM, PRED, MODE, GROUP)>
__global__ void __launch_bounds__(kWave * kMaxWavesPerBlock)
    __attribute__((amdgpu_waves_per_eu(WAVES))) k_beamform(const FramePlan P) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int b = blockIdx.x;
  // RF modes: clear the frame maximum the post-processing folds into (the IQ
  // modes fold it here, so their launch clears it beforehand)
  if (!is_iq_mode(MODE) && P.ws_max && b == 0) dev::frame_max_clear(P.ws_max, threadIdx.x);
  const int q = b / P.tiles_x;
  const int tz = P.tiles_z - 1 - q, tx = b - q * P.tiles_x;
  dev::process_tile<AM, PRED, MODE, GROUP>(P, tz, tx, smem);
}

template <int AM, bool PRED, int MODE>
hipError_t launch_angles(const FramePlan &P, hipStream_t stream) {
  const dim3 block(kWave * P.wz * P.wx * P.wc);
  const dim3 grid(P.n_tiles);
  const size_t lds = plan_lds_bytes(P);
  if constexpr (wave_ref_mode(MODE) && AM > 11 && AM <= 16) {
    if (P.cpw > 1 && P.wc == 1 && P.wz * P.wx <= 4) {  // four wavefronts: see min_waves
      hipLaunchKernelGGL((k_beamform<AM, PRED, MODE, dev::kGroups, 4>), grid, block, lds, stream,
                         P);
      return hipGetLastError();
    }
  }
  if constexpr (MODE == kDas && AM > 12 && AM <= 16) {
    if (P.cpw == 1 && P.wc > 1 && P.n_tiles >= 2 * 3 * 256) {  // see min_waves
      hipLaunchKernelGGL((k_beamform<AM, PRED, MODE, dev::kShared, 6>), grid, block, lds, stream,
                         P);
      return hipGetLastError();
    }
  }
  if (P.cpw > 1 && P.wc > 1)
    hipLaunchKernelGGL((k_beamform<AM, PRED, MODE, dev::kGroupsShared>), grid, block, lds, stream,
                       P);
  else if (P.cpw > 1)
    hipLaunchKernelGGL((k_beamform<AM, PRED, MODE, dev::kGroups>), grid, block, lds, stream, P);
  else if (P.wc > 1)
    hipLaunchKernelGGL((k_beamform<AM, PRED, MODE, dev::kShared>), grid, block, lds, stream, P);
  else
    hipLaunchKernelGGL((k_beamform<AM, PRED, MODE, dev::kOneGroup>), grid, block, lds, stream, P);
  return hipGetLastError();
}

// An exactly unrolled kernel for every angle count, except 17..32 angles of the
// IQ modes (two sums and a transmit delay per angle stay in registers: 96 of
// them at 32 angles), which share a predicated one. A kernel that tests each
// angle against the count takes the angles of a channel one LDS round trip
// after another instead of all at once: a 21-angle DAS frame of 96 channels and
// 301 x 777 pixels takes 238 us with it and 101 us unrolled, a 7-angle BB-DMAS
// frame of 64 channels and 384 x 500 pixels 102 and 67 us (demodulation and log
// image included).
template <int MODE>
hipError_t launch_mode(const FramePlan &P, hipStream_t stream) {
  switch (P.n_angles) {
#define PWBF_CASE(n) \
  case n: return launch_angles<n, false, MODE>(P, stream);
    PWBF_CASE(1) PWBF_CASE(2) PWBF_CASE(3) PWBF_CASE(4) PWBF_CASE(5) PWBF_CASE(6) PWBF_CASE(7)
    PWBF_CASE(8) PWBF_CASE(9) PWBF_CASE(10) PWBF_CASE(11) PWBF_CASE(12) PWBF_CASE(13)
    PWBF_CASE(14) PWBF_CASE(15) PWBF_CASE(16)
    default: break;
  }
  if constexpr (is_iq_mode(MODE)) {
    if (P.n_angles > 16 && P.n_angles <= kMaxAngles)
      return launch_angles<kMaxAngles, true, MODE>(P, stream);
  } else {
    switch (P.n_angles) {
      PWBF_CASE(17) PWBF_CASE(18) PWBF_CASE(19) PWBF_CASE(20) PWBF_CASE(21) PWBF_CASE(22)
      PWBF_CASE(23) PWBF_CASE(24) PWBF_CASE(25) PWBF_CASE(26) PWBF_CASE(27) PWBF_CASE(28)
      PWBF_CASE(29) PWBF_CASE(30) PWBF_CASE(31) PWBF_CASE(32)
      default: break;
    }
  }
#undef PWBF_CASE
  return hipErrorInvalidValue;
}

}  // namespace

}  // namespace pwbf

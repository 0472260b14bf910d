#pragma once
// Device code of the depth-wise post-processing (band-pass, envelope, column
// maximum), shared by the single-frame and the batched launches.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fft_reg.h"
#include "frame_max.h"
#include "plan.h"
#include "post_layout.h"

namespace pwbf {
namespace dev {

// LDS of a block of that many threads
template <int L>
__host__ __device__ constexpr size_t post_lds_bytes(int block_threads) {
  return (size_t)fftr::padded<L>() * post_columns(L, block_threads) * 8;
}
// LDS of a batched block, whatever the length of its columns
constexpr size_t kPostBatchLdsBytes = post_lds_bytes<12>(kPostThreads);
static_assert(post_lds_bytes<3>(kPostThreads) == kPostBatchLdsBytes &&
                  post_lds_bytes<2>(kPostThreads) <= kPostBatchLdsBytes &&
                  post_lds_bytes<1>(kPostThreads) <= kPostBatchLdsBytes,
              "");

// One-sided weight of the analytic signal at bin k of n: 1 at DC and Nyquist,
// 2 on positive bins, 0 on negative ones.
__device__ __forceinline__ float analytic_weight(int k, int n) {
  const int half_n = n >> 1;
  return (k == 0 || k == half_n) ? 1.f : (k < half_n ? 2.f : 0.f);
}

// Largest m >= 0 of the wavefront, in lane 63. Lanes combine within rows of 16
// by data-parallel moves, then rows 0 and 2 into 1 and 3, then 1 into 3 (a
// shuffle is an LDS round trip, six of them in a row at the end of every
// column).
__device__ __forceinline__ float wave_max63(float m) {
  auto step = [](float v, auto ctrl, auto rows) {
    const int o = __builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value,
                                              decltype(rows)::value, 0xf, false);
    return fmaxf(v, __int_as_float(o));
  };
  using all = std::integral_constant<int, 0xf>;
  m = step(m, std::integral_constant<int, 0x111>{}, all{});  // row_shr:1
  m = step(m, std::integral_constant<int, 0x112>{}, all{});  // row_shr:2
  m = step(m, std::integral_constant<int, 0x114>{}, all{});  // row_shr:4
  m = step(m, std::integral_constant<int, 0x118>{}, all{});  // row_shr:8
  m = step(m, std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});
  m = step(m, std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});
  return m;
}

// Post-process columns ix0, ix0 + 1, ... of the frame described by Q, of 2^L
// samples each, one per thread group of the block (post_columns of them; those
// past the last column of the frame do nothing), with LDS at sm.
template <int L>
__device__ __forceinline__ void postz_columns(const PostPlan &Q, int ix0, float2 *sm) {
  using namespace fftr;
  constexpr int n = 1 << L, T = threads(L), E = points(L);
  const int row = (int)threadIdx.x / T, t = (int)threadIdx.x & (T - 1);
  float2 *x = sm + row * padded<L>();
  const int ix = ix0 + row;
  const bool mine = ix < Q.nx;
  const size_t base = (size_t)min(ix, Q.nx - 1) * n;

  float2 v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) v[e] = make_float2(Q.src[base + index_of<L, false>(e, t)], 0.f);
  // analytic-signal weights, band mask, and the 1/nz of the inverse
  const bool band = Q.bandpass;
  const int k_lo = Q.k_lo, k_hi = Q.k_hi;
  filter<L>(v, x, t, [&](int k) __attribute__((always_inline)) {
    const float h = analytic_weight(k, n) * (1.0f / n);
    const int ak = k <= n / 2 ? k : n - k;
    return band && (ak < k_lo || ak > k_hi) ? 0.f : h;
  });

  float m = 0.f;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const size_t o = base + index_of<L, false>(e, t);
    const float a = sqrtf(v[e].x * v[e].x + v[e].y * v[e].y);
    if (mine) {
      if (Q.filtered) Q.filtered[o] = v[e].x;
      if (Q.env) Q.env[o] = a;
      m = fmaxf(m, a);
    }
  }
  if (Q.ws_max) {
    m = wave_max63(m);
    if (((int)threadIdx.x & 63) == 63) frame_max_fold(Q.ws_max, m);
  }
}

// the same for a column length known only at run time (uniform over the block)
__device__ __forceinline__ void postz_columns_any(const PostPlan &Q, int ix0, float2 *sm) {
  switch (Q.log2nz) {
    case 1: postz_columns<1>(Q, ix0, sm); break;
    case 2: postz_columns<2>(Q, ix0, sm); break;
    case 3: postz_columns<3>(Q, ix0, sm); break;
    case 4: postz_columns<4>(Q, ix0, sm); break;
    case 5: postz_columns<5>(Q, ix0, sm); break;
    case 6: postz_columns<6>(Q, ix0, sm); break;
    case 7: postz_columns<7>(Q, ix0, sm); break;
    case 8: postz_columns<8>(Q, ix0, sm); break;
    case 9: postz_columns<9>(Q, ix0, sm); break;
    case 10: postz_columns<10>(Q, ix0, sm); break;
    case 11: postz_columns<11>(Q, ix0, sm); break;
    default: postz_columns<12>(Q, ix0, sm); break;
  }
}

// 20 log10(env / max), clipped at the floor (the floor everywhere when max is 0);
// a true division, so the maximum itself maps to exactly 0 dB
__device__ __forceinline__ float log_db(float env, float max, float floor_db) {
  return max > 0.f ? fmaxf(20.0f * log10f(env / max), floor_db) : floor_db;
}

}  // namespace dev
}  // namespace pwbf

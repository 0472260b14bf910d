// Baseband (IQ) demodulation of channel records, two records per transform, and
// the decimating form, one record per transform (fft_reg.h).
//
// The analytic signal of a record x of n = 2^L samples is the inverse DFT of
// its spectrum times the one-sided weights w(k) (1 at DC and Nyquist, 2 on
// positive bins, 0 on negative ones); since w(k) + w(n - k) = 2, its real part
// is x itself and its imaginary part is the discrete Hilbert transform H(x).
// Two records x1, x2 go through one transform pair: the inverse DFT of w(k)
// times the DFT of x1 + i x2 is (x1 + i H(x1)) + i (x2 + i H(x2)), so
// H(x1) = Im - x2 and H(x2) = x1 - Re, with x1 and x2 the samples read
// again. Each analytic record is then multiplied by exp(-2 pi i r k) with
// r = f0 / fs, k the sample index. The carrier phase is formed in revolutions
// from r as a float-float pair: k * r_hi splits exactly into a rounded product
// and its error (one FMA), so frac(k r) is accurate to ~1e-7 revolutions for
// every k, where a plain float product would drift by ~k ulp.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "postz_device.h"

namespace pwbf {

namespace {

using fft::cmul;

template <int DT>
__device__ __forceinline__ float rf_sample(const void *rf, size_t i) {
  if constexpr (DT == kI16) return (float)((const int16_t *)rf)[i];
  if constexpr (DT == kF16) return __half2float(((const __half *)rf)[i]);
  return ((const float *)rf)[i];
}

// exp(-2 pi i r k): the carrier phase at sample k in revolutions, from r as a
// float-float pair (the FMA gives the exact error of the rounded product); the
// hardware sine and cosine take their argument in revolutions, as the IQ
// beamformer's phase rotation does
__device__ __forceinline__ float2 carrier(int k, float r_hi, float r_lo) {
  const float fk = (float)k;
  const float p = fk * r_hi;
  const float e = fmaf(fk, r_hi, -p);  // exact error of the product
  const float rho = (p - floorf(p)) + fmaf(fk, r_lo, e);
  return make_float2(__builtin_amdgcn_cosf(rho), -__builtin_amdgcn_sinf(rho));
}

// What bounds it at 4096 samples is the two transforms' VALU work and LDS
// exchanges (69 MB read and written would take 13 us): 1408 records in 20.0 us,
// 22.1 us with the transforms in LDS.
template <int DT, int L>
__global__ void __launch_bounds__(post_block(L)) __attribute__((amdgpu_waves_per_eu(4)))
    k_iq_demod(const void *__restrict__ rf, float2 *__restrict__ iq, int rows, float r_hi,
               float r_lo) {
  using namespace fftr;
  extern __shared__ __align__(16) float2 sm[];
  constexpr int n = 1 << L, T = threads(L), E = points(L);
  const int row = (int)threadIdx.x / T, t = (int)threadIdx.x & (T - 1);
  // records past the last one are read again from it and not written; a missing
  // second record is zero
  const int r0 = 2 * ((int)blockIdx.x * post_columns(L, post_block(L)) + row);
  const bool one = r0 < rows, two = r0 + 1 < rows;
  const size_t base0 = (size_t)min(r0, rows - 1) * n, base1 = two ? base0 + n : base0;
  auto samples = [&](const void *p, int e) __attribute__((always_inline)) {  // (x1, x2)
    const int k = index_of<L, false>(e, t);
    const float v1 = rf_sample<DT>(p, base1 + k);
    return make_float2(rf_sample<DT>(p, base0 + k), two ? v1 : 0.f);
  };
  float2 v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) v[e] = samples(rf, e);
  filter<L>(v, sm + row * padded<L>(), t, [](int k) __attribute__((always_inline)) {
    return dev::analytic_weight(k, n) * (1.0f / n);
  });
  // the samples again, from the cache (kept in registers, they spill at four
  // wavefronts per SIMD): an address the compiler cannot tell is the same
  const void *again = rf;
  asm("" : "+s"(again));
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int k = index_of<L, false>(e, t);
    const float2 ph = carrier(k, r_hi, r_lo);
    const float2 x12 = samples(again, e);
    if (one) iq[base0 + k] = cmul(make_float2(x12.x, v[e].y - x12.y), ph);
    if (two) iq[base1 + k] = cmul(make_float2(x12.y, x12.x - v[e].x), ph);
  }
}

// Decimation by D = 2^LD, one record per transform: of the analytic spectrum only
// the bins k_lo..k_hi are kept (those within fs / (2 D) of f0, decided on the
// host), then mixed down, and every D-th sample is kept. The band limit takes the
// real part off the record itself, so the two-records-per-transform form above
// does not apply here. Bin k of the record is bin k mod n / D of the kept samples,
// so the inverse transform has n / D points (448 records of 2048 samples at D = 2:
// 10.5 -> 8.5 us). The kept band is n / D bins wide without its edges, but where
// both edges fall on bins the host's rounded comparison may keep them both
// (fs = 62.5 MHz / 3, f0 = 5 fs / 16, D = 4: n / D + 1 bins): the upper one,
// n / D past the lower, is added to the same bin once that is stored. The inverse's row
// needs only a part of the threads of the record's (T / T2 copies of them compute
// the same, each on LDS of its own).
template <int DT, int L, int LD>
__global__ void __launch_bounds__(post_block(L))
    k_iq_demod_decim(const void *__restrict__ rf, float2 *__restrict__ iq, int rows, int k_lo,
                     int k_hi, float r_hi, float r_lo) {
  using namespace fftr;
  extern __shared__ __align__(16) float2 sm[];
  constexpr int n = 1 << L, T = threads(L), E = points(L);
  constexpr int L2 = L - LD, n2 = 1 << L2, T2 = threads(L2), E2 = points(L2);
  static_assert((T / T2) * padded<L2>() <= padded<L>(), "the copies fit the record's LDS");
  const int row = (int)threadIdx.x / T, t = (int)threadIdx.x & (T - 1);
  float2 *x = sm + row * padded<L>();
  const int rec = (int)blockIdx.x * post_columns(L, post_block(L)) + row;
  const size_t base = (size_t)min(rec, rows - 1) * n;
  float2 v[E];
#pragma unroll
  for (int e = 0; e < E; ++e)
    v[e] = make_float2(rf_sample<DT>(rf, base + index_of<L, false>(e, t)), 0.f);
  TwiddlesOf<L, false> fwd;
  fwd.load(t);
  transform<L, false>(v, fwd, x, t);
  TwiddlesOf<L2, true> inv;
  inv.load(t & (T2 - 1));
  // the kept bins, weighted and folded; the others are zero
  row_sync<L>();
  for (int k = t; k < n2; k += T) x[k] = make_float2(0.f, 0.f);
  row_sync<L>();
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int k = index_of<L, true>(e, t);
    const float h = dev::analytic_weight(k, n) * (1.0f / n);
    v[e] = make_float2(v[e].x * h, v[e].y * h);
    if (k >= k_lo && k <= k_hi && k - k_lo < n2) x[k & (n2 - 1)] = v[e];
  }
  row_sync<L>();
  if (k_hi - k_lo >= n2) {  // the band's upper edge as well as its lower (uniform)
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int k = index_of<L, true>(e, t);
      if (k <= k_hi && k - k_lo >= n2) x[k & (n2 - 1)] = fft::cadd(x[k & (n2 - 1)], v[e]);
    }
    row_sync<L>();
  }
  const int t2 = t & (T2 - 1);
  float2 y[E2];
#pragma unroll
  for (int e = 0; e < E2; ++e) y[e] = x[index_of<L2, true>(e, t2)];
  row_sync<L>();
  transform<L2, true>(y, inv, x + (t / T2) * padded<L2>(), t2);
  if (t >= T2 || rec >= rows) return;
  const size_t out = (size_t)rec * n2;
#pragma unroll
  for (int e = 0; e < E2; ++e) {
    const int m = index_of<L2, false>(e, t2);
    iq[out + m] = cmul(y[e], carrier(m << LD, r_hi, r_lo));
  }
}

template <int DT, int L>
hipError_t launch_full(const void *rf, float2 *iq, int rows, float r_hi, float r_lo,
                       hipStream_t stream) {
  const int per = 2 * post_columns(L, post_block(L));
  hipLaunchKernelGGL((k_iq_demod<DT, L>), dim3((rows + per - 1) / per), dim3(post_block(L)),
                     dev::post_lds_bytes<L>(post_block(L)), stream, rf, iq, rows, r_hi, r_lo);
  return hipGetLastError();
}

template <int DT, int L, int LD>
hipError_t launch_decim(const void *rf, float2 *iq, int rows, int k_lo, int k_hi, float r_hi,
                        float r_lo, hipStream_t stream) {
  if constexpr (L > LD) {  // (a decimated record holds at least two samples)
    const int per = post_columns(L, post_block(L));
    hipLaunchKernelGGL((k_iq_demod_decim<DT, L, LD>), dim3((rows + per - 1) / per),
                       dim3(post_block(L)), dev::post_lds_bytes<L>(post_block(L)), stream, rf, iq,
                       rows, k_lo, k_hi, r_hi, r_lo);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

template <int DT, int L>
hipError_t launch_length(const void *rf, float2 *iq, int rows, float r_hi, float r_lo, int log2d,
                         int k_lo, int k_hi, hipStream_t stream) {
  switch (log2d) {
    case 0: return launch_full<DT, L>(rf, iq, rows, r_hi, r_lo, stream);
    case 1: return launch_decim<DT, L, 1>(rf, iq, rows, k_lo, k_hi, r_hi, r_lo, stream);
    case 2: return launch_decim<DT, L, 2>(rf, iq, rows, k_lo, k_hi, r_hi, r_lo, stream);
    case 3: return launch_decim<DT, L, 3>(rf, iq, rows, k_lo, k_hi, r_hi, r_lo, stream);
    default: return hipErrorInvalidValue;
  }
}

template <int DT>
hipError_t launch_type(const void *rf, float2 *iq, int rows, int log2ns, float r_hi, float r_lo,
                       int log2d, int k_lo, int k_hi, hipStream_t stream) {
  switch (log2ns) {
#define PWBF_LEN(L) \
  case L: return launch_length<DT, L>(rf, iq, rows, r_hi, r_lo, log2d, k_lo, k_hi, stream);
    PWBF_LEN(1) PWBF_LEN(2) PWBF_LEN(3) PWBF_LEN(4) PWBF_LEN(5) PWBF_LEN(6) PWBF_LEN(7)
    PWBF_LEN(8) PWBF_LEN(9) PWBF_LEN(10) PWBF_LEN(11) PWBF_LEN(12)
#undef PWBF_LEN
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_iq_demod(const void *rf, int dtype, void *iq, int rows, int log2ns, float r_hi,
                           float r_lo, int log2d, int k_lo, int k_hi, hipStream_t stream) {
  float2 *out = (float2 *)iq;
  if (dtype == kI16)
    return launch_type<kI16>(rf, out, rows, log2ns, r_hi, r_lo, log2d, k_lo, k_hi, stream);
  if (dtype == kF16)
    return launch_type<kF16>(rf, out, rows, log2ns, r_hi, r_lo, log2d, k_lo, k_hi, stream);
  return launch_type<kF32>(rf, out, rows, log2ns, r_hi, r_lo, log2d, k_lo, k_hi, stream);
}

}  // namespace pwbf

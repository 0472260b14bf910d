// f-k migrations (Stolt's and Lu's) for steered plane waves. Every stage runs
// over all angles of the call in one launch (blockIdx.y selects the angle), so
// even a single frame gives the chip thousands of blocks. The two methods share
// every stage but the remap. Transforms keep their points in registers between
// passes, and the two transposes between channel-major and bin-major data happen
// inside blocks that hold several rows, so every global access is a contiguous run.
// Bound by instruction issue (transforms, float-float positions) and by the planes
// between the stages (230 MB for 11 angles of 128 channels and 4096 samples, which
// the 256 MB cache holds in part). That compound, 1024 x 1024 pixels: time 15.4 us,
// space 16.2, remap 22.6, itime 17.7, image 24 (with every transform
// in LDS by 256 threads: 16.6, 21.8, 26.2, 21.0); one 64-channel record of
// 2048 samples on 500 x 512: 5.2, 4.6, 11.6, 4.0, 4.1 (6.8, 7.5, 12.1, 5.9, 4.2).
//
//  k_fk_time      row per (channel pair, angle): one complex FFT of two traces
//                 (Nt samples each, as real and imaginary parts), split into the
//                 two spectra; the positive bins times exp(2 pi i k c_e) (the trace
//                 advanced by its element's firing delay and shifted to t = 0) go
//                 to T, blocked by the ROWS bins of one kx-transform block
//  k_fk_space     block per (ROWS bins, angle): reads the bins k0..k0+ROWS of every
//                 channel (one contiguous block of T), FFTs along the array
//                 zero-padded to Nx, writes P[k][m]
//                 (Lu) or P[m][k] (Stolt, whose remap reads along frequency)
//  k_fk_remap     block per (ROWS image rows kz_j, angle): each cell (j, m) takes
//                 the data spectrum from P -
//                   Stolt: at bin u = sqrt((alpha m')^2 + j^2) (m' the signed
//                   index), linearly (zeros past the last bin), times j / u;
//                   Lu: at frequency bin u = (beta^2 m'^2 + j^2) /
//                   (beta m' sin + j cos) and spatial bin m' - u sin / (2 beta),
//                   bilinearly (periodic in the spatial bin), times
//                   (j - u cos / 2) / (beta m' sin + j cos), zero where the
//                   receive wavenumber j - u cos / 2 is negative -
//                 then inverse FFTs along kx, and writes the window's columns
//                 transposed, U[e][j0..j0+ROWS)
//  k_fk_itime     row per window column x1 (and angle): inverse FFT along kz of
//                 U[e][.], zero-filled to Nt, scaled by 1/(Nx Nt); stores the
//                 window's rows of M
//  k_fk_image     thread per two pixels (adjacent columns, one depth): for every
//                 angle the migrated image at (x1, z1), affine in the pixel
//                 indices, by bilinear interpolation; the complex sum over angles
//                 gives the real, imaginary and magnitude planes and the frame
//                 maximum
//
// Interpolation positions are float-float: neighbouring spectral bins of an echo
// differ by up to a half turn of phase, so a weight off by 1e-4 (a float32
// position near bin 2000) would show in the image; products of a float-float
// constant and an integer index are exact up to the final rounding.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "beamform_device.h"
#include "fft_reg.h"
#include "fk.h"
#include "postz_device.h"

namespace pwbf {

namespace {

using dev::ff;
using fft::cmul;

constexpr int kFkThreads = fft::kThreads;  // of the blocks along the array

template <int DT>
__device__ __forceinline__ float trace_sample(const void *rf, size_t i) {
  if constexpr (DT == kI16) return (float)((const int16_t *)rf)[i];
  if constexpr (DT == kF16) return __half2float(((const __half *)rf)[i]);
  return ((const float *)rf)[i];
}

__device__ __forceinline__ ff ffi(int i) { return {(float)i, 0.f}; }

// frac(k c) in revolutions for an integer k and c = hi + lo
__device__ __forceinline__ float frac_revs(int k, ff c) {
#pragma clang fp contract(off)
  const float fk = (float)k;
  const float p = fk * c.hi;
  return (p - floorf(p)) + fmaf(fk, c.lo, fmaf(fk, c.hi, -p));
}

// integer part and fraction of a float-float value (fraction in [0, 1)),
// |u| < 2^24
__device__ __forceinline__ int split_index(ff u, float *frac) {
  const float fl = floorf(u.hi);
  const float f = (u.hi - fl) + u.lo;
  const float c = floorf(f);  // -1, 0 or 1: the low part crossed an integer
  *frac = f - c;
  return (int)fl + (int)c;
}

__device__ __forceinline__ int kbins_of(const FkPlan &F) { return (1 << F.log2nt) / 2 + 1; }

// The transforms along time run in registers, eight points a thread (fft_reg.h): a
// block holds kTimeRows<L> rows of 2^L points, one from 512 points on.
template <int L>
constexpr int kTimeThreads = fftr::threads(L) < kWave ? kWave : fftr::threads(L);
template <int L>
constexpr int kTimeRows = kTimeThreads<L> / fftr::threads(L);
template <int L>
constexpr size_t kTimeLds = (size_t)fftr::padded<L>() * kTimeRows<L> * 8;

// Two traces per row: channels e0 and e0 + 1 go in as the real and imaginary parts
// of one complex sequence z (a missing second trace is zero). With Z its DFT and
// Z(Nt) = Z(0), the traces' spectra are X0(k) = (Z(k) + conj Z(Nt - k)) / 2 and
// X1(k) = (Z(k) - conj Z(Nt - k)) / (2i).
template <int L, int DT>
__global__ void __launch_bounds__(kTimeThreads<L>) k_fk_time(FkPlan F) {
  extern __shared__ __align__(16) float2 sm[];
  constexpr int nt = 1 << L, kbins = nt / 2 + 1, T = fftr::threads(L), E = fftr::points(L);
  const int row = threadIdx.x / T, t = threadIdx.x % T, a = blockIdx.y;
  const int e0 = 2 * (blockIdx.x * kTimeRows<L> + row);
  const bool one = e0 < F.n_ch, two = e0 + 1 < F.n_ch;
  // the frame maximum that the image kernel, last of the call, folds into
  if (F.ws_max && blockIdx.x == 0 && blockIdx.y == 0) dev::frame_max_clear(F.ws_max, threadIdx.x);
  float2 *x = sm + row * fftr::padded<L>();
  // every read inside the record array
  const size_t base = ((size_t)a * F.n_ch + (one ? e0 : 0)) * nt;
  const size_t base1 = two ? base + nt : base;
  float2 v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int k = fftr::index_of<L, false>(e, t);
    const float v1 = trace_sample<DT>(F.rf, base1 + k);
    v[e] = make_float2(trace_sample<DT>(F.rf, base + k), two ? v1 : 0.f);
  }
  fftr::TwiddlesOf<L, false> tw;
  tw.load(t);
  fftr::transform<L, false>(v, tw, x, t);
  fftr::row_sync<L>();  // the last exchange's reads are done
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int k = fftr::index_of<L, true>(e, t);
    if (k == 0 || k >= nt / 2) x[fftr::pad<L>(k)] = v[e];
  }
  fftr::row_sync<L>();
  const FkAngleConst &A = F.ang[a];
  const ff c0 = dev::ff_add({A.c0_hi, A.c0_lo}, dev::ff_mul(ffi(e0), {A.c1_hi, A.c1_lo}));
  const ff c1 = dev::ff_add({A.c0_hi, A.c0_lo}, dev::ff_mul(ffi(e0 + 1), {A.c1_hi, A.c1_lo}));
  // T[a][k / R][e][k mod R]: the pair's rows of a block are adjacent, 2 R bins
  const int LR = 12 - F.log2nx, R = 1 << LR;
  float2 *T0 = F.T + (size_t)a * F.n_ch * fk_kbins_padded(L, F.log2nx) + e0 * R;
  // exp(2 pi i k c) at the thread's first bin, then by the step of T bins: a thread's
  // bins t + m T are at most five products from an accurate phase
  float sn, cs;
  sincospif(2.0f * frac_revs(t, c0), &sn, &cs);
  float2 ph0 = make_float2(cs, sn);
  sincospif(2.0f * frac_revs(T, c0), &sn, &cs);
  const float2 step0 = make_float2(cs, sn);
  sincospif(2.0f * frac_revs(t, c1), &sn, &cs);
  float2 ph1 = make_float2(cs, sn);
  sincospif(2.0f * frac_revs(T, c1), &sn, &cs);
  const float2 step1 = make_float2(cs, sn);
  constexpr int RL = 1 << fftr::radix_bits(L, fftr::passes(L) - 1), Q = E / RL;
#pragma unroll
  for (int m = 0; m <= E / 2; ++m) {
    const int k = t + m * T, e = m % Q * RL + m / Q;  // v[e] is bin k
    if (k < kbins && one) {
      const float2 z = v[e], w = x[fftr::pad<L>((nt - k) & (nt - 1))];  // Z(k), Z(Nt - k)
      const float2 x0 = make_float2(0.5f * (z.x + w.x), 0.5f * (z.y - w.y));
      const float2 x1 = make_float2(0.5f * (z.y + w.y), 0.5f * (w.x - z.x));
      float2 *q = T0 + (size_t)(k >> LR) * F.n_ch * R + (k & (R - 1));
      q[0] = cmul(x0, ph0);
      if (two) q[R] = cmul(x1, ph1);
    }
    ph0 = cmul(ph0, step0);
    ph1 = cmul(ph1, step1);
  }
}

template <int L, int METHOD>
__global__ void __launch_bounds__(kFkThreads) k_fk_space(FkPlan F) {
  constexpr int nx = 1 << L, ROWS = kFkRowPoints >> L;
  extern __shared__ __align__(16) float2 sm[];
  const int kbins = kbins_of(F), k0 = blockIdx.x * ROWS, a = blockIdx.y;
  // the block's bins of every channel are one contiguous run of T (bins past
  // the last are never written and read as zero)
  const float2 *T = F.T + ((size_t)a * fk_kbins_padded(F.log2nt, L) + k0) * F.n_ch;
  float2 *P = F.P + (size_t)a * kbins * nx;
  auto load = [&](int r, int e) {
    return e < F.n_ch && k0 + r < kbins ? T[e * ROWS + r] : make_float2(0.f, 0.f);
  };
  // Stolt's remap reads along frequency at fixed kx: store P[m][k], consecutive
  // threads on consecutive bins
  auto store = [&](int r, int m, float2 v) {
    const unsigned k = k0 + r;
    if ((int)k < kbins) P[METHOD == kFkStolt ? m * kbins + k : k * nx + m] = v;
  };
  fft::transform_io<L, false, ROWS, true, METHOD == kFkStolt>(sm, load, store);
}

// Float-float helpers with hardware reciprocal and square root in the leading
// term: the error-free residual of the correction step absorbs their ulp-level
// error, so the results match the correctly rounded versions to ~1e-14.
__device__ __forceinline__ ff quick_two_sum(float a, float b) {  // |a| >= |b|
#pragma clang fp contract(off)
  const float s = a + b;
  return {s, b - (s - a)};
}

__device__ __forceinline__ ff ff_sqrt_hw(ff a) {  // a.hi > 0
#pragma clang fp contract(off)
  const float s = __builtin_amdgcn_sqrtf(a.hi);
  const float r = fmaf(-s, s, a.hi) + a.lo;
  return quick_two_sum(s, r * (0.5f * __builtin_amdgcn_rcpf(s)));
}

__device__ __forceinline__ ff ff_div_hw(ff a, ff b) {  // b.hi != 0
#pragma clang fp contract(off)
  const float rb = __builtin_amdgcn_rcpf(b.hi);
  const float q1 = a.hi * rb;
  const float p = q1 * b.hi, e = fmaf(q1, b.hi, -p);
  const float r = ((a.hi - p) - e) + (a.lo - q1 * b.lo);
  return quick_two_sum(q1, r * rb);
}

// v - u c for float-float v, u, c (c's product split exactly)
__device__ __forceinline__ ff ff_sub_mul(ff v, ff u, float c_hi, float c_lo) {
#pragma clang fp contract(off)
  const float p = u.hi * c_hi, e = fmaf(u.hi, c_hi, -p) + (u.hi * c_lo + u.lo * c_hi);
  const ff d = dev::two_sum(v.hi, -p);
  return dev::two_sum(d.hi, d.lo + (v.lo - e));
}

// The remap bodies below leave floating-point contraction on (their weights
// and sums may fuse into FMAs); every error-free step sits in a helper that
// turns it off.

// The cells of a remap block: per thread a fixed set of kx columns m (one when
// Nx <= 256) and, for each, every row of the block that falls to the thread.
template <int L>
struct RemapCells {
  static constexpr int nx = 1 << L, ROWS = kFkRowPoints >> L;
  static constexpr int MPT = nx >= kFkThreads ? nx / kFkThreads : 1;  // columns per thread
  static constexpr int RSTEP = nx >= kFkThreads ? 1 : kFkThreads / nx;  // rows apart
  __device__ static int m(int mi) {
    return nx >= kFkThreads ? (int)threadIdx.x + kFkThreads * mi : (int)threadIdx.x & (nx - 1);
  }
  __device__ static int r0() { return nx >= kFkThreads ? 0 : (int)threadIdx.x >> L; }
};

// Stolt's remap: the cell (j, m) takes the data spectrum at bin
// u = sqrt((alpha m')^2 + j^2), linearly (zeros past the last bin), times j / u.
// P is stored [m][k]; consecutive threads take consecutive rows j of one column, so
// their bins u are close and the gathers contiguous.
template <int L>
__device__ __forceinline__ float2 stolt_cell(const FkAngleConst &A, const float2 *__restrict__ P,
                                             int j0, int r, int m, int kbins) {
  constexpr int nx = 1 << L;
  const int ms = m < nx / 2 ? m : m - nx;
  const int j = min(j0 + r, kbins - 1);  // rows past the last bin are zero below
  const float fj = (float)j;
  const ff am = dev::ff_mul(ffi(ms), {A.m0_hi, A.m0_lo});
  const ff am2 = dev::ff_mul(am, am);  // (alpha m')^2
  const ff u2 = dev::two_sum(am2.hi, fj * fj);  // j^2 < 2^24 is exact
  const ff u2n = dev::two_sum(u2.hi, u2.lo + am2.lo);
  const bool in_band = u2n.hi > 0.f && u2n.hi < (float)(kbins + 1) * (float)(kbins + 1);
  const ff u = ff_sqrt_hw(in_band ? u2n : ff{1.f, 0.f});
  float w;
  const int i0 = split_index(u, &w);
  // clamped loads, always issued; taps outside the spectrum weigh zero
  const bool ok = in_band && i0 >= 0 && i0 <= kbins - 1 && j0 + r < kbins;
  const int ia = ok ? i0 : 0, ib = min(ia + 1, kbins - 1);
  const unsigned cb = (unsigned)(m * kbins);  // < 2^21 cells per angle
  const float2 lo = P[cb + ia], hi = P[cb + ib];
  const float jac = ok ? fj * __builtin_amdgcn_rcpf(u.hi) : 0.f;
  const float wl = (1.f - w) * jac, wh = (ok && i0 + 1 <= kbins - 1) ? w * jac : 0.f;
  return make_float2(wl * lo.x + wh * hi.x, wl * lo.y + wh * hi.y);
}

// Lu's remap of the block's rows: the cell (j, m) takes the data spectrum at
// frequency bin u = (beta^2 m'^2 + j^2) / (beta m' sin + j cos) and spatial bin
// m' - u sin / (2 beta), bilinearly (periodic in the spatial bin, zeros past the
// last frequency bin), times (j - u cos / 2) / (beta m' sin + j cos); zero where
// the receive wavenumber j - u cos / 2 is negative or the denominator is not
// positive.
template <int L>
__device__ __forceinline__ void lu_rows(const FkAngleConst &A, const float2 *__restrict__ P,
                                        int j0, int kbins, float2 *x) {
  using C = RemapCells<L>;
  constexpr int stride = fft::row_stride(C::nx, C::ROWS);
  const float ch = 0.5f * A.m2_hi, cl = 0.5f * A.m2_lo;  // cos / 2
  for (int mi = 0; mi < C::MPT; ++mi) {
    const int m = C::m(mi), ms = m < C::nx / 2 ? m : m - C::nx;
    const ff bm = dev::ff_mul(ffi(ms), {A.m0_hi, A.m0_lo});
    const ff bm2 = dev::ff_mul(bm, bm);                     // beta^2 m'^2
    const ff bms = dev::ff_mul(bm, {A.m1_hi, A.m1_lo});     // beta m' sin
#pragma unroll 2
    for (int r = C::r0(); r < C::ROWS; r += C::RSTEP) {
      const int j = min(j0 + r, kbins - 1);
      const float fj = (float)j;
      // den = beta m' sin + j cos
      const float pc = fj * A.m2_hi, ec = fmaf(fj, A.m2_hi, -pc) + fj * A.m2_lo;
      const ff d0 = dev::two_sum(bms.hi, pc);
      const ff den = dev::two_sum(d0.hi, d0.lo + (bms.lo + ec));
      const bool pos = den.hi > 0.f;
      // num = beta^2 m'^2 + j^2
      const ff n0 = dev::two_sum(bm2.hi, fj * fj);
      const ff num = dev::two_sum(n0.hi, n0.lo + bm2.lo);
      const ff u = ff_div_hw(num, pos ? den : ff{1.f, 0.f});  // source frequency bin
      // the receive wavenumber j - u cos / 2 only weighs the cell: float suffices
      const float kzr = fmaf(-u.lo, ch, fmaf(-u.hi, ch, fj)) - u.hi * cl;
      const bool branch = pos && kzr >= 0.f && u.hi < (float)kbins && j0 + r < kbins;
      const ff mf = ff_sub_mul(ffi(ms), u, A.m3_hi, A.m3_lo);  // spatial bin
      float wu, wm;
      const int i0 = split_index(branch ? u : ff{0.f, 0.f}, &wu);
      const int m0 = split_index(branch ? mf : ff{0.f, 0.f}, &wm);
      const bool ok = branch && i0 >= 0 && i0 <= kbins - 1;
      const int ia = ok ? i0 : 0, ib = min(ia + 1, kbins - 1);
      const int ma = m0 & (C::nx - 1), mb = (m0 + 1) & (C::nx - 1);  // periodic in kx
      const unsigned ra = (unsigned)(ia * C::nx), rb = (unsigned)(ib * C::nx);  // < 2^21
      const float2 p00 = P[ra + ma], p01 = P[ra + mb], p10 = P[rb + ma], p11 = P[rb + mb];
      const float jac = ok ? kzr * __builtin_amdgcn_rcpf(den.hi) : 0.f;
      const float hw = (ok && i0 + 1 <= kbins - 1) ? wu : 0.f;  // zeros past the last bin
      const float w00 = (1.f - wm) * (1.f - wu) * jac, w01 = wm * (1.f - wu) * jac;
      const float w10 = (1.f - wm) * hw * jac, w11 = wm * hw * jac;
      x[r * stride + fft::pad(m)] =
          make_float2(w00 * p00.x + w01 * p01.x + w10 * p10.x + w11 * p11.x,
                      w00 * p00.y + w01 * p01.y + w10 * p10.y + w11 * p11.y);
    }
  }
}

template <int L, int METHOD>
__global__ void __launch_bounds__(kFkThreads) k_fk_remap(FkPlan F) {
  constexpr int nx = 1 << L, ROWS = kFkRowPoints >> L;
  extern __shared__ __align__(16) float2 sm[];
  const int kbins = kbins_of(F), j0 = blockIdx.x * ROWS, a = blockIdx.y;
  const FkAngleConst &A = F.ang[a];
  const float2 *P = F.P + (size_t)a * kbins * nx;
  // the window's columns, transposed: consecutive threads take consecutive rows
  float2 *U = F.U + (size_t)a * nx * kbins;
  auto store = [&](int r, int e, float2 v) {
    if ((unsigned)(e - A.col0) < (unsigned)A.ncol && j0 + r < kbins)
      U[(unsigned)(e * kbins + j0 + r)] = v;
  };
  if constexpr (METHOD == kFkLu) {
    lu_rows<L>(A, P, j0, kbins, sm);
    __syncthreads();
    fft::transform_io<L, true, ROWS, false, true>(sm, fft::FromLds(), store);
  } else {
    auto load = [&](int r, int m) { return stolt_cell<L>(A, P, j0, r, m, kbins); };
    fft::transform_io<L, true, ROWS, true, true>(sm, load, store);
  }
}

template <int L>
__global__ void __launch_bounds__(kTimeThreads<L>) k_fk_itime(FkPlan F) {
  extern __shared__ __align__(16) float2 sm[];
  constexpr int nt = 1 << L, kbins = nt / 2 + 1, T = fftr::threads(L), E = fftr::points(L);
  const int row = threadIdx.x / T, t = threadIdx.x % T, a = blockIdx.y, nx = 1 << F.log2nx;
  const FkAngleConst &A = F.ang[a];
  const int c = blockIdx.x * kTimeRows<L> + row;
  if ((int)blockIdx.x * kTimeRows<L> >= A.ncol) return;  // the whole block: outside the window
  const bool mine = c < A.ncol;
  const int col = A.col0 + (mine ? c : 0);
  const float2 *I = F.U + ((size_t)a * nx + col) * kbins;
  float2 v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int j = fftr::index_of<L, false>(e, t);
    v[e] = j < kbins ? I[j] : make_float2(0.f, 0.f);
  }
  fftr::TwiddlesOf<L, false> tw;  // a forward transform with the parts swapped
  tw.load(t);
#pragma unroll
  for (int e = 0; e < E; ++e) v[e] = fft::swap(v[e]);
  fftr::transform<L, false>(v, tw, sm + row * fftr::padded<L>(), t);
  const float scale = 1.0f / ((float)nx * (float)nt);
  float2 *out = F.M + ((size_t)a * nx + col) * nt;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int l = fftr::index_of<L, true>(e, t);
    if (mine && (unsigned)(l - A.row0) < (unsigned)A.nrow)
      out[l] = make_float2(v[e].y * scale, v[e].x * scale);
  }
}

// Integer part and fraction of v0 + k c for float-float v0, c and an integer
// 0 <= k < 2^24: the product split exactly (one FMA), the large terms summed
// with an error-free addition, the small ones added once; the fraction is
// accurate to ~1e-7 of an index step. Returns false when the value is outside
// (lo, hi), before any conversion to an integer.
__device__ __forceinline__ bool map_index(float v0h, float v0l, float k, float ch, float cl,
                                          float lo, float hi, int *idx, float *frac) {
#pragma clang fp contract(off)
  const float p = k * ch, e = fmaf(k, ch, -p);
  const ff t = dev::two_sum(v0h, p);
  if (!(t.hi > lo && t.hi < hi)) return false;
  const float small = (t.lo + (v0l + e)) + k * cl;
  const float fl = floorf(t.hi);
  const float f = (t.hi - fl) + small;
  const float c = floorf(f);  // -1, 0 or 1: the small terms crossed an integer
  *idx = (int)fl + (int)c;
  *frac = f - c;
  return true;
}

// Adds the bilinear value of one angle's migrated image M at column i0 + fx,
// row j0 + fz to (re, im); taps outside the angle's window are outside
// [0, Nx) x [0, Nt) too (the window holds every tap inside, with a margin), so
// they read as zero.
__device__ __forceinline__ void add_taps(const float2 *M, int nt, const FkAngleConst &A, int i0,
                                         float fx, int j0, float fz, float &re, float &im) {
  const int c1 = A.col0 + A.ncol, r1 = A.row0 + A.nrow;
  if (i0 >= A.col0 && i0 + 1 < c1 && j0 >= A.row0 && j0 + 1 < r1) {
    const float2 *q = M + (unsigned)(i0 * nt + j0);
    const float2 v00 = q[0], v01 = q[1], v10 = q[nt], v11 = q[nt + 1];
    const float w00 = (1.f - fx) * (1.f - fz), w01 = (1.f - fx) * fz;
    const float w10 = fx * (1.f - fz), w11 = fx * fz;
    re += w00 * v00.x + w01 * v01.x + w10 * v10.x + w11 * v11.x;
    im += w00 * v00.y + w01 * v01.y + w10 * v10.y + w11 * v11.y;
  } else {
#pragma unroll
    for (int di = 0; di < 2; ++di) {
#pragma unroll
      for (int dj = 0; dj < 2; ++dj) {
        const int i = i0 + di, j = j0 + dj;
        if (i >= A.col0 && i < c1 && j >= A.row0 && j < r1) {
          const float w = (di ? fx : 1.f - fx) * (dj ? fz : 1.f - fz);
          const float2 v = M[(unsigned)(i * nt + j)];
          re = fmaf(w, v.x, re);
          im = fmaf(w, v.y, im);
        }
      }
    }
  }
}

// Pixel (ix, iz) reads column ux0 + ix uxi + iz uxk and row uz0 + iz uzk of the
// migrated image of each angle. A block is a depth run of two image columns:
// each column's lateral base ux0 + ix uxi (float-float) is formed once per
// angle and shared through LDS, and a thread's two pixels share the row map.
__global__ void __launch_bounds__(256) k_fk_image(FkPlan F, int zchunks) {
  const int nt = 1 << F.log2nt, nx1 = 1 << F.log2nx;
  const int px = blockIdx.x / zchunks, iz = (blockIdx.x - px * zchunks) * 256 + threadIdx.x;
  const int ix0 = 2 * px;
  const bool two = ix0 + 1 < F.nx_img, mine = iz < F.nz_img;
  const float fiz = (float)iz;
  __shared__ float2 s_xb[2][kMaxAngles];
  {
    const int c = threadIdx.x >> 5, a = threadIdx.x & 31;  // column c of the pair, angle a
    if (c < 2 && a < F.n_ang) {
#pragma clang fp contract(off)
      const FkAngleConst &A = F.ang[a];
      const float fix = (float)(ix0 + c);
      const float p = fix * A.uxi_hi, e = fmaf(fix, A.uxi_hi, -p);
      const ff t = dev::two_sum(A.ux0_hi, p);
      const ff b = dev::two_sum(t.hi, (t.lo + (A.ux0_lo + e)) + fix * A.uxi_lo);
      s_xb[c][a] = make_float2(b.hi, b.lo);
    }
  }
  __syncthreads();
  float re0 = 0.f, im0 = 0.f, re1 = 0.f, im1 = 0.f;
  for (int a = 0; a < F.n_ang; ++a) {
    const FkAngleConst &A = F.ang[a];
    if (A.ncol == 0) continue;
    // far outside the migrated image: nothing to read (and no integer overflow)
    int j0;
    float fz;
    if (!map_index(A.uz0_hi, A.uz0_lo, fiz, A.uzk_hi, A.uzk_lo, -2.f, (float)(nt + 1), &j0, &fz))
      continue;
    const float2 *M = F.M + (size_t)a * nx1 * nt;
    int i0;
    float fx;
    const float2 xb0 = s_xb[0][a], xb1 = s_xb[1][a];
    if (map_index(xb0.x, xb0.y, fiz, A.uxk_hi, A.uxk_lo, -2.f, (float)(nx1 + 1), &i0, &fx))
      add_taps(M, nt, A, i0, fx, j0, fz, re0, im0);
    if (two && map_index(xb1.x, xb1.y, fiz, A.uxk_hi, A.uxk_lo, -2.f, (float)(nx1 + 1), &i0, &fx))
      add_taps(M, nt, A, i0, fx, j0, fz, re1, im1);
  }
  const float e0 = sqrtf(re0 * re0 + im0 * im0), e1 = sqrtf(re1 * re1 + im1 * im1);
  if (mine) {
    const size_t t = (size_t)ix0 * F.nz_img + iz;
    F.out_rf[t] = re0;
    if (F.out_imag) F.out_imag[t] = im0;
    if (F.out_env) F.out_env[t] = e0;
    if (two) {
      const size_t t1 = t + F.nz_img;
      F.out_rf[t1] = re1;
      if (F.out_imag) F.out_imag[t1] = im1;
      if (F.out_env) F.out_env[t1] = e1;
    }
  }
  if (F.ws_max) {
    __shared__ float wm[4];
    float m = mine ? fmaxf(e0, two ? e1 : 0.f) : 0.f;
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0) wm[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0)
      dev::frame_max_fold(F.ws_max, fmaxf(fmaxf(wm[0], wm[1]), fmaxf(wm[2], wm[3])));
  }
}

template <int L>
hipError_t launch_rows(const FkPlan &F, hipStream_t s) {
  constexpr int ROWS = kFkRowPoints >> L;
  const int kbins = (1 << F.log2nt) / 2 + 1;
  const dim3 grid((kbins + ROWS - 1) / ROWS, F.n_ang), blk(kFkThreads);
  const size_t lds = fft::lds_bytes(1 << L, ROWS);
  if (F.method == kFkLu) {
    hipLaunchKernelGGL((k_fk_space<L, kFkLu>), grid, blk, lds, s, F);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_fk_remap<L, kFkLu>), grid, blk, lds, s, F);
  } else {
    hipLaunchKernelGGL((k_fk_space<L, kFkStolt>), grid, blk, lds, s, F);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_fk_remap<L, kFkStolt>), grid, blk, lds, s, F);
  }
  return hipGetLastError();
}

// the transform along time of the records (ncol < 0) or of ncol window columns
template <int L>
hipError_t launch_time_rows(const FkPlan &F, int ncol, hipStream_t s) {
  const int rows = ncol < 0 ? (F.n_ch + 1) / 2 : ncol;  // two traces to a row
  const dim3 grid((rows + kTimeRows<L> - 1) / kTimeRows<L>, F.n_ang), blk(kTimeThreads<L>);
  if (ncol >= 0)
    hipLaunchKernelGGL(k_fk_itime<L>, grid, blk, kTimeLds<L>, s, F);
  else if (F.dtype == kI16)
    hipLaunchKernelGGL((k_fk_time<L, kI16>), grid, blk, kTimeLds<L>, s, F);
  else if (F.dtype == kF16)
    hipLaunchKernelGGL((k_fk_time<L, kF16>), grid, blk, kTimeLds<L>, s, F);
  else
    hipLaunchKernelGGL((k_fk_time<L, kF32>), grid, blk, kTimeLds<L>, s, F);
  return hipGetLastError();
}

hipError_t launch_time(const FkPlan &F, int ncol, hipStream_t s) {
  switch (F.log2nt) {
    case 1: return launch_time_rows<1>(F, ncol, s);
    case 2: return launch_time_rows<2>(F, ncol, s);
    case 3: return launch_time_rows<3>(F, ncol, s);
    case 4: return launch_time_rows<4>(F, ncol, s);
    case 5: return launch_time_rows<5>(F, ncol, s);
    case 6: return launch_time_rows<6>(F, ncol, s);
    case 7: return launch_time_rows<7>(F, ncol, s);
    case 8: return launch_time_rows<8>(F, ncol, s);
    case 9: return launch_time_rows<9>(F, ncol, s);
    case 10: return launch_time_rows<10>(F, ncol, s);
    case 11: return launch_time_rows<11>(F, ncol, s);
    case 12: return launch_time_rows<12>(F, ncol, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_fk(const FkPlan &F, int ncol_max, hipStream_t s) {
  hipError_t e = launch_time(F, -1, s);
  if (e != hipSuccess) return e;
  switch (F.log2nx) {
    case 2: e = launch_rows<2>(F, s); break;
    case 3: e = launch_rows<3>(F, s); break;
    case 4: e = launch_rows<4>(F, s); break;
    case 5: e = launch_rows<5>(F, s); break;
    case 6: e = launch_rows<6>(F, s); break;
    case 7: e = launch_rows<7>(F, s); break;
    case 8: e = launch_rows<8>(F, s); break;
    case 9: e = launch_rows<9>(F, s); break;
    case 10: e = launch_rows<10>(F, s); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  if (ncol_max > 0) {
    if ((e = launch_time(F, ncol_max, s)) != hipSuccess) return e;
  }
  const int zchunks = (F.nz_img + 255) / 256;
  hipLaunchKernelGGL(k_fk_image, dim3((F.nx_img + 1) / 2 * zchunks), dim3(256), 0, s, F,
                     zchunks);
  return hipGetLastError();
}

}  // namespace pwbf

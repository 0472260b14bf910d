#pragma once
// FFTs whose points stay in registers between passes, for rows that are loaded,
// transformed, weighted, transformed back and stored by the same threads: the
// depth post-processing, the IQ demodulation and the f-k migrations' transforms along
// time.
//
// A row of n = 2^L points belongs to T = n / 8 threads with E = 8 points each: a
// row of up to 512 points is one wavefront or a part of one, so its passes need
// no barrier, and every thread has a butterfly in every pass. (With one 256-thread
// block to a row in LDS, radix-16 passes over 512 points kept 32 of the threads
// busy. Sixteen points a thread from 1024 points on were slower: 128 registers and,
// at 4096, spills.) Passes are Stockham's as in fft_lds.h: radix E, the last pass
// (the first of the inverse) takes the remaining factor. Point (q, r) of thread t,
// butterfly q of E / R, is x[t + q T + r n / R]: the first pass loads it from
// memory and the last leaves it at the same index, so a row crosses LDS only
// between passes (twice per 512-point transform), and a spectrum is weighted in
// registers between the forward and the inverse transform.
//
// The twiddles of a direction are asked for before its first pass, the forward
// ones together with the row's samples.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fft_lds.h"
#include "post_layout.h"

namespace pwbf {
namespace fftr {

using fft::cmul;

__host__ __device__ constexpr int log2_points(int L) { return fft_log2_points(L); }
__host__ __device__ constexpr int points(int L) { return 1 << log2_points(L); }
__host__ __device__ constexpr int threads(int L) { return fft_threads(L); }
__host__ __device__ constexpr int passes(int L) {
  return (L + log2_points(L) - 1) / log2_points(L);
}
// log2 of the radix of forward pass i; the inverse runs them backwards
__host__ __device__ constexpr int radix_bits(int L, int i) {
  const int e = log2_points(L);
  return i + 1 < passes(L) ? e : L - e * (passes(L) - 1);
}
__host__ __device__ constexpr int radix_bits(int L, int i, bool inv) {
  return radix_bits(L, inv ? passes(L) - 1 - i : i);
}
// log2 of the product of the radices before pass i
__host__ __device__ constexpr int done_bits(int L, int i, bool inv) {
  int b = 0;
  for (int k = 0; k < i; ++k) b += radix_bits(L, k, inv);
  return b;
}

// LDS positions: one pad element per E, so that the first pass's writes with a
// stride of E spread over the banks
template <int L>
__host__ __device__ constexpr int pad(int i) {
  return i + (i >> log2_points(L));
}
template <int L>
__host__ __device__ constexpr int padded() {
  return pad<L>(1 << L);
}

// Orders a row's LDS writes before its reads: nothing but the compiler's order
// within a wavefront (its LDS instructions execute in order), else a barrier.
template <int L>
__device__ __forceinline__ void row_sync() {
  if constexpr (threads(L) <= 64) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

struct NoTwiddles {
  __device__ __forceinline__ void load(int) {}
};
// both directions have the same radices in the same order, and so the same
// twiddles
__host__ __device__ constexpr bool palindromic(int L) {
  return radix_bits(L, 0) == radix_bits(L, passes(L) - 1);
}

// Twiddle bases of the passes after the first of one direction: w, w^2, w^4 of
// W_{NS R}^k, per butterfly whose k differs.
template <int L, bool INV, int I = 1>
struct Twiddles {
  static constexpr int RB = radix_bits(L, I, INV), R = 1 << RB, NSB = done_bits(L, I, INV);
  static constexpr int Q = points(L) / R, T = threads(L);
  static constexpr int QK = (1 << NSB) <= T ? 1 : Q;  // k = t mod NS for every butterfly, or not
  float2 w[QK][RB];
  std::conditional_t<I + 1 < passes(L), Twiddles<L, INV, I + 1>, NoTwiddles> next;
  __device__ __forceinline__ void load(int t) {
#pragma unroll
    for (int q = 0; q < QK; ++q) {
      const int k = (t + q * T) & ((1 << NSB) - 1);
#pragma unroll
      for (int b = 0; b < RB; ++b) w[q][b] = fft::w4096((k << b) << (12 - NSB - RB));
    }
    next.load(t);
  }
};

// the butterflies of pass I on v[q R + r]
template <int L, bool INV, int I, class TW>
__device__ __forceinline__ void butterflies(float2 (&v)[points(L)], const TW *tw) {
  constexpr int R = 1 << radix_bits(L, I, INV), Q = points(L) / R;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    float2 x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = v[q * R + r];
    if constexpr (I > 0) {
      const auto &w = tw->w[TW::QK == 1 ? 0 : q];
      float2 p[R];
      p[1] = w[0];
      if constexpr (R >= 4) {
        p[2] = w[1];
        p[3] = cmul(p[2], p[1]);
      }
      if constexpr (R >= 8) {
        p[4] = w[2];
#pragma unroll
        for (int r = 5; r < 8; ++r) p[r] = cmul(p[4], p[r - 4]);
      }
#pragma unroll
      for (int r = 1; r < R; ++r) x[r] = cmul(x[r], p[r]);
    }
    fft::dft<R>(x);
#pragma unroll
    for (int r = 0; r < R; ++r) v[q * R + r] = x[r];
  }
}

// from the outputs of pass I to the inputs of pass I + 1, through LDS row x
template <int L, bool INV, int I>
__device__ __forceinline__ void exchange(float2 (&v)[points(L)], float2 *x, int t) {
  constexpr int T = threads(L), n = 1 << L;
  constexpr int R = 1 << radix_bits(L, I, INV), Q = points(L) / R;
  constexpr int NS = 1 << done_bits(L, I, INV);
  constexpr int R2 = 1 << radix_bits(L, I + 1, INV), Q2 = points(L) / R2;
  row_sync<L>();  // the row's reads of the exchange before are done
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int j = t + q * T, k = j & (NS - 1), o = (j - k) * R + k;
#pragma unroll
    for (int r = 0; r < R; ++r) x[pad<L>(o + r * NS)] = v[q * R + r];
  }
  row_sync<L>();
#pragma unroll
  for (int q = 0; q < Q2; ++q)
#pragma unroll
    for (int r = 0; r < R2; ++r) v[q * R2 + r] = x[pad<L>(t + q * T + r * (n / R2))];
}

template <int L, bool INV, int I, class TW>
__device__ __forceinline__ void later_passes(float2 (&v)[points(L)], const TW *tw, float2 *x,
                                             int t) {
  if constexpr (I < passes(L)) {
    exchange<L, INV, I - 1>(v, x, t);
    butterflies<L, INV, I>(v, tw);
    later_passes<L, INV, I + 1>(v, &tw->next, x, t);
  }
}

// Index of v[e] of thread t: before the forward and after the inverse transform
// (both with the forward's first radix), and of the spectrum between them (with
// its last radix).
template <int L, bool SPECTRUM>
__device__ __forceinline__ int index_of(int e, int t) {
  constexpr int R = 1 << radix_bits(L, SPECTRUM ? passes(L) - 1 : 0);
  return t + (e / R) * threads(L) + (e % R) * ((1 << L) / R);
}

// Forward transform of the row in v (thread t of its T), or the inverse without
// the 1/n; x: the row's LDS, padded<L>() elements. The inverse swaps real and
// imaginary parts around the forward passes.
template <int L, bool INV, class TW>
__device__ __forceinline__ void transform(float2 (&v)[points(L)], const TW &tw, float2 *x, int t) {
  if constexpr (INV) {
#pragma unroll
    for (int e = 0; e < points(L); ++e) v[e] = fft::swap(v[e]);
  }
  butterflies<L, INV, 0>(v, &tw);
  later_passes<L, INV, 1>(v, &tw, x, t);
  if constexpr (INV) {
#pragma unroll
    for (int e = 0; e < points(L); ++e) v[e] = fft::swap(v[e]);
  }
}

// the twiddles of a direction (one pass: none)
template <int L, bool INV>
using TwiddlesOf = std::conditional_t<(passes(L) > 1), Twiddles<L, INV && !palindromic(L)>,
                                      NoTwiddles>;

// Forward transform, weight(k) on every bin k, inverse transform (without 1/n).
template <int L, class W>
__device__ __forceinline__ void filter(float2 (&v)[points(L)], float2 *x, int t, W weight) {
  TwiddlesOf<L, false> fwd;
  fwd.load(t);
  transform<L, false>(v, fwd, x, t);
  TwiddlesOf<L, true> inv;
  if constexpr (!palindromic(L)) inv.load(t);
#pragma unroll
  for (int e = 0; e < points(L); ++e) {
    const float h = weight(index_of<L, true>(e, t));
    v[e] = make_float2(v[e].x * h, v[e].y * h);
  }
  if constexpr (palindromic(L))
    transform<L, true>(v, fwd, x, t);
  else
    transform<L, true>(v, inv, x, t);
}

}  // namespace fftr
}  // namespace pwbf

// Image metrics of the evaluation (Section II-D) on an envelope image
// [nx][nz]: contrast of cysts, Eq. (5) CR and Eq. (6) CNR, and the lateral and
// axial full width at half maximum of point targets.
//
// Regions are discs in pixel units. A pixel is inside when
// ((ix - cx) sx)^2 + ((iz - cz) sz)^2 <= 1, evaluated with separately rounded
// float32 operations (no fused multiply-add), so that the decision is
// reproducible bit for bit on the host. One block per cyst or target; sums are
// taken per thread in a fixed stride order and combined in a fixed order, so
// results do not depend on scheduling.
#include <hip/hip_runtime.h>

#include "frame_max.h"
#include "metrics.h"

namespace pwbf {

namespace {

constexpr int kThreads = 256, kWave = 64;

// ((i - c) s)^2, every operation rounded on its own: a fused u*u + v*v would
// decide pixels on the circle differently from the host. A pixel is in the disc
// where the squares of both axes sum to at most 1.
__device__ __forceinline__ float square_off(int i, float c, float s) {
#pragma clang fp contract(off)
  const float u = ((float)i - c) * s;
  return u * u;
}

__device__ __forceinline__ bool inside(const DiscPix &d, int ix, int iz) {
#pragma clang fp contract(off)
  return square_off(ix, d.cx, d.sx) + square_off(iz, d.cz, d.sz) <= 1.0f;
}

// Sum over the block in a fixed order: LDS tree over the 256 partials.
__device__ float block_sum(float v, float *sh) {
  __syncthreads();
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int s = kThreads / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  return sh[0];
}

// The pixels t, t + T, t + 2T, ... of a disc's box (columns ix0.., h pixels each,
// depth fastest) as (ix, iz), without a division per pixel.
struct BoxWalk {
  int ix, iz, dx, dz, h;
  __device__ __forceinline__ BoxWalk(int t, int T, int height) : h(height) {
    ix = t / h;
    iz = t - ix * h;
    dx = T / h;
    dz = T - dx * h;
  }
  __device__ __forceinline__ void step() {
    ix += dx;
    iz += dz;
    if (iz >= h) {
      iz -= h;
      ++ix;
    }
  }
};

// A cyst's block: half of its wavefronts take the inside disc, half the
// background, over the columns of 64 depths of the disc's box: the depth part of
// the test is formed once per 64 depths and the rest is the same in every lane.
// Bound by instruction issue on the cyst's one compute unit. Three cysts of 2-4 mm
// on a 1024 x 1024 image (boxes of up to 30 000 pixels): 14.3 us; 256 threads a
// cyst that divided for every pixel's column took 101 us.
constexpr int kCystThreads = 1024, kHalf = kCystThreads / 2, kAhead = 8;

// sum over the half block of each of N values, in a fixed order: wavefronts by a
// butterfly, then their sums in order; every thread of the half gets them
template <int N>
__device__ __forceinline__ void half_sum(float (&v)[N], float (*sh)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i)
    for (int off = 1; off < kWave; off <<= 1) v[i] += __shfl_xor(v[i], off);
  const int wave = (int)threadIdx.x / kWave, first = wave & ~(kHalf / kWave - 1);
  __syncthreads();
  if ((threadIdx.x & (kWave - 1)) == 0)
#pragma unroll
    for (int i = 0; i < N; ++i) sh[wave][i] = v[i];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) {
    v[i] = 0.f;
    for (int w = 0; w < kHalf / kWave; ++w) v[i] += sh[first + w][i];
  }
}

// CR (Eq. (5)) and CNR (Eq. (6)) of env between the two discs of cyst k
__global__ void __launch_bounds__(kCystThreads)
    k_contrast(const float *__restrict__ env, int nz, CystSet cs, pwbf_contrast *__restrict__ out) {
  __shared__ float sh2[kCystThreads / kWave][2], sh1[kCystThreads / kWave][1];
  __shared__ float stat[2][3];
  const int k = blockIdx.x, t = (int)threadIdx.x % kHalf;
  // the same in every lane of a wavefront, and known to be: the disc stays in
  // scalar registers
  const int side = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kHalf);
  const DiscPix d = side ? cs.out[k] : cs.in[k];
  const int lane = t & (kWave - 1), first = d.ix0 + __builtin_amdgcn_readfirstlane(t / kWave);
  constexpr int step = kHalf / kWave;  // columns between two of a wavefront
  // Calls visit(in the disc, value) for this lane's depth of every column of its
  // wavefront, kAhead loads in flight. Lanes past the box read its last depth.
  auto walk = [&](auto visit) __attribute__((always_inline)) {
    for (int z0 = d.iz0; z0 <= d.iz1; z0 += kWave) {
      const int iz = min(z0 + lane, d.iz1);
      const float vv = z0 + lane <= d.iz1 ? square_off(iz, d.cz, d.sz) : 2.f;
      for (int ix = first; ix <= d.ix1; ix += kAhead * step) {
        float v[kAhead];
        bool in[kAhead];
#pragma unroll
        for (int e = 0; e < kAhead; ++e) {
          const int x = min(ix + e * step, d.ix1);
          v[e] = env[(size_t)x * nz + iz];
          in[e] = ix + e * step <= d.ix1 && square_off(x, d.cx, d.sx) + vv <= 1.0f;
        }
#pragma unroll
        for (int e = 0; e < kAhead; ++e) visit(in[e], v[e]);
      }
    }
  };
  float cs2[2] = {0.f, 0.f};
  walk([&](bool in, float v) {
    cs2[0] += in ? 1.f : 0.f;
    cs2[1] += in ? v : 0.f;
  });
  half_sum(cs2, sh2);
  const float n = cs2[0], mu = cs2[1] / n;
  float q[1] = {0.f};
  walk([&](bool in, float v) {
    const float c = in ? v - mu : 0.f;
    q[0] = fmaf(c, c, q[0]);
  });
  half_sum(q, sh1);
  if (t == 0) {
    stat[side][0] = n;
    stat[side][1] = n > 0.f ? mu : __builtin_nanf("");
    stat[side][2] = n > 0.f ? sqrtf(q[0] / n) : __builtin_nanf("");
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  const float mu_in = stat[0][1], mu_bg = stat[1][1], sd_in = stat[0][2], sd_bg = stat[1][2];
  pwbf_contrast r;
  r.mu_in = mu_in;
  r.mu_out = mu_bg;
  r.sigma_in = sd_in;
  r.sigma_out = sd_bg;
  r.cr_db = (mu_in > 0.f && mu_bg > 0.f) ? 20.0f * log10f(mu_in / mu_bg) : __builtin_nanf("");
  const float den = sqrtf(0.5f * (sd_in * sd_in + sd_bg * sd_bg));
  r.cnr = den > 0.f ? (mu_in - mu_bg) / den : __builtin_nanf("");
  r.n_in = (int)stat[0][0];
  r.n_out = (int)stat[1][0];
  out[k] = r;
}

// the block's item: the k with block0[k] <= b < block0[k + 1]
__device__ __forceinline__ int quality_item(const QualityList &ql, int b) {
  int lo = 0, hi = ql.n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (ql.block0[mid] <= b)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// (count, sum, sum of squares) of env over the disc's pixels in columns
// [c0, c1] of its box
__device__ float4 disc_partial(const float *env, int nz, const DiscPix &d, int c0, int c1,
                               float *sh) {
  const int h = d.iz1 - d.iz0 + 1, w = c1 - c0 + 1;
  const int total = w > 0 && h > 0 ? w * h : 0;
  float c = 0.f, s = 0.f, q = 0.f;
  BoxWalk p(threadIdx.x, kThreads, max(h, 1));
#pragma unroll 4
  for (int k = threadIdx.x; k < total; k += kThreads, p.step()) {
    const int ix = c0 + p.ix, iz = d.iz0 + p.iz;
    if (inside(d, ix, iz)) {
      const float e = env[(size_t)ix * nz + iz];
      c += 1.f;
      s += e;
      q = fmaf(e, e, q);
    }
  }
  const float n = block_sum(c, sh), sum = block_sum(s, sh), sq = block_sum(q, sh);
  return make_float4(n, sum, sq, 0.f);
}

// mean and population deviation from combined partials
__device__ __forceinline__ void stats_of(float n, float s, float q, float *mu, float *sd) {
  if (!(n > 0.f)) {
    *mu = __builtin_nanf("");
    *sd = __builtin_nanf("");
    return;
  }
  const float m = s / n;
  *mu = m;
  *sd = sqrtf(fmaxf(q / n - m * m, 0.f));
}

// one block per column chunk of a disc of a checked slot
__global__ void __launch_bounds__(kThreads)
    k_quality(const QualityPlan *__restrict__ plans, QualityList ql, QualityOut *__restrict__ out,
              float4 *__restrict__ partials, int *__restrict__ counters) {
  __shared__ float sh[kThreads];
  __shared__ bool s_last;
  const int k = quality_item(ql, blockIdx.x);
  const QualityPlan &Q = plans[ql.plan[k]];
  const int b = blockIdx.x - ql.block0[k];
  const bool in = b < Q.chunks_in;
  const DiscPix &d = in ? Q.in : Q.out;
  const int chunk = in ? b : b - Q.chunks_in, cols = in ? Q.cols_in : Q.cols_out;
  const int c0 = d.ix0 + chunk * cols, c1 = min(d.ix1, c0 + cols - 1);
  const float4 p = disc_partial(Q.env, Q.nz, d, c0, c1, sh);
  if (threadIdx.x == 0) {
    partials[blockIdx.x] = p;
    __threadfence();  // the partial is visible before the count says so
    const int nb = ql.block0[k + 1] - ql.block0[k];
    s_last = atomicAdd(&counters[k], 1) == nb - 1;
  }
  __syncthreads();
  if (!s_last) return;  // uniform over the block
  __threadfence();
  const float m = dev::frame_max_read(Q.ws_max);
  if (threadIdx.x == 0) {
    // the slot's partials in chunk order: inside disc, then background
    float ni = 0.f, si = 0.f, qi = 0.f, no = 0.f, so = 0.f, qo = 0.f;
    const int first = ql.block0[k];
    for (int j = 0; j < Q.chunks_in; ++j) {
      const float4 v = partials[first + j];
      ni += v.x;
      si += v.y;
      qi += v.z;
    }
    for (int j = 0; j < Q.chunks_out; ++j) {
      const float4 v = partials[first + Q.chunks_in + j];
      no += v.x;
      so += v.y;
      qo += v.z;
    }
    float mu_in, sd_in, mu_bg, sd_bg;
    stats_of(ni, si, qi, &mu_in, &sd_in);
    stats_of(no, so, qo, &mu_bg, &sd_bg);
    QualityOut r;
    r.frame_max = m;
    r.cr_db = (mu_in > 0.f && mu_bg > 0.f) ? 20.0f * log10f(mu_in / mu_bg) : __builtin_nanf("");
    const float den = sqrtf(0.5f * (sd_in * sd_in + sd_bg * sd_bg));
    r.cnr = den > 0.f ? (mu_in - mu_bg) / den : __builtin_nanf("");
    r.ok = (m > 0.f && r.cr_db <= Q.max_cr_db) ? 1 : 0;  // a NaN CR fails
    out[k] = r;
    counters[k] = 0;  // ready for the next batch that uses this buffer
  }
}

// where the line through (0, a) and (1, b) crosses the half level, as a
// fraction of the pixel step from a
__device__ __forceinline__ float cross(float a, float b, float half) {
  return (half - a) / (b - a);
}

__global__ void __launch_bounds__(kThreads)
    k_resolution(const float *__restrict__ env, int nx, int nz, float dx, float dz, TargetSet ts,
                 pwbf_resolution *__restrict__ out) {
  __shared__ float sv[kThreads];
  __shared__ int si[kThreads];
  const DiscPix d = ts.t[blockIdx.x];
  const int w = d.ix1 - d.ix0 + 1, h = d.iz1 - d.iz0 + 1;
  const int total = w > 0 && h > 0 ? w * h : 0;
  // argmax; among equal values the smallest flat index ix * nz + iz
  float best = -__builtin_inff();
  int bi = -1;
  BoxWalk p(threadIdx.x, kThreads, max(h, 1));
#pragma unroll 4
  for (int k = threadIdx.x; k < total; k += kThreads, p.step()) {
    const int ix = d.ix0 + p.ix, iz = d.iz0 + p.iz;
    if (!inside(d, ix, iz)) continue;
    const int flat = ix * nz + iz;
    const float v = env[flat];
    if (v > best || (v == best && (bi < 0 || flat < bi))) {
      best = v;
      bi = flat;
    }
  }
  sv[threadIdx.x] = best;
  si[threadIdx.x] = bi;
  __syncthreads();
  for (int s = kThreads / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      const float v = sv[threadIdx.x + s];
      const int i = si[threadIdx.x + s];
      if (i >= 0 && (si[threadIdx.x] < 0 || v > sv[threadIdx.x] ||
                     (v == sv[threadIdx.x] && i < si[threadIdx.x]))) {
        sv[threadIdx.x] = v;
        si[threadIdx.x] = i;
      }
    }
    __syncthreads();
  }
  // The half-level walks along the row and the column through the peak, one
  // wavefront each way, 64 pixels a step (one thread walking pixel by pixel paid a
  // memory latency per pixel): the distance to the first pixel below half, or to
  // the image's edge.
  __shared__ int reach[4];  // left, right, up, down
  static_assert(kThreads == 4 * kWave, "a wavefront for each way");
  const int flat = si[0], way = (int)threadIdx.x / kWave, lane = (int)threadIdx.x & (kWave - 1);
  const float peak = sv[0], half = peak * 0.5f;
  const int ix = flat >= 0 ? flat / nz : -1, iz = flat >= 0 ? flat - ix * nz : -1;
  if (flat >= 0) {
    const int room = way == 0 ? ix + 1 : (way == 1 ? nx - ix : (way == 2 ? iz + 1 : nz - iz));
    const long long step = way == 0 ? -(long long)nz : (way == 1 ? nz : (way == 2 ? -1 : 1));
    int k = 0;
    for (; k < room; k += kWave) {
      const int j = k + lane;
      const bool below = j < room && !(env[flat + step * j] >= half);
      const unsigned long long m = __ballot(below);
      if (m) {
        k += (int)__builtin_ctzll(m);
        break;
      }
    }
    if (lane == 0) reach[way] = min(k, room);
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  pwbf_resolution r;
  const float nanv = __builtin_nanf("");
  r.peak = nanv;
  r.fwhm_x = nanv;
  r.fwhm_z = nanv;
  r.ix = -1;
  r.iz = -1;
  if (flat >= 0) {
    r.peak = peak;
    r.ix = ix;
    r.iz = iz;
    // Lateral profile: row iz, stride nz; i and j the first pixels below half. A
    // negative peak lies below its own half, so both are then the peak itself: at
    // the image's edge a pixel that the crossing needs is missing, and the width is
    // NaN as where a side never falls below half.
    int i = ix - reach[0], j = ix + reach[1];
    if (i >= 0 && i + 1 < nx && j > 0 && j < nx) {
      const float left =
          (float)i + cross(env[(size_t)i * nz + iz], env[(size_t)(i + 1) * nz + iz], half);
      const float right =
          (float)(j - 1) + cross(env[(size_t)(j - 1) * nz + iz], env[(size_t)j * nz + iz], half);
      r.fwhm_x = (right - left) * dx;
    }
    // axial profile: column ix, contiguous
    const float *col = env + (size_t)ix * nz;
    i = iz - reach[2];
    j = iz + reach[3];
    if (i >= 0 && i + 1 < nz && j > 0 && j < nz) {
      const float left = (float)i + cross(col[i], col[i + 1], half);
      const float right = (float)(j - 1) + cross(col[j - 1], col[j], half);
      r.fwhm_z = (right - left) * dz;
    }
  }
  out[blockIdx.x] = r;
}

}  // namespace

hipError_t launch_quality(const QualityPlan *plans, const QualityList &ql, QualityOut *out,
                          float4 *partials, int *counters, hipStream_t stream) {
  if (ql.n < 1) return hipSuccess;
  hipLaunchKernelGGL(k_quality, dim3(ql.block0[ql.n]), dim3(kThreads), 0, stream, plans, ql, out,
                     partials, counters);
  return hipGetLastError();
}

hipError_t launch_contrast(const float *env, int nz, const CystSet &cs, int n, pwbf_contrast *out,
                           hipStream_t stream) {
  hipLaunchKernelGGL(k_contrast, dim3(n), dim3(kCystThreads), 0, stream, env, nz, cs, out);
  return hipGetLastError();
}

hipError_t launch_resolution(const float *env, int nx, int nz, float dx, float dz,
                             const TargetSet &ts, int n, pwbf_resolution *out,
                             hipStream_t stream) {
  hipLaunchKernelGGL(k_resolution, dim3(n), dim3(kThreads), 0, stream, env, nx, nz, dx, dz, ts,
                     out);
  return hipGetLastError();
}

}  // namespace pwbf

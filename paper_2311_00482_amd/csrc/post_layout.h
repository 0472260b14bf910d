#pragma once
// How the depth post-processing splits columns over threads, for host and device
// code: a column of n = 2^L samples belongs to n / 8 threads with 8 samples each.

#if defined(__HIPCC__)
#define PWBF_POST_HD __host__ __device__
#else
#define PWBF_POST_HD
#endif

namespace pwbf {

PWBF_POST_HD constexpr int fft_log2_points(int L) { return L >= 3 ? 3 : L; }
PWBF_POST_HD constexpr int fft_threads(int L) { return 1 << (L - fft_log2_points(L)); }

// Threads of a post-processing block of a batch, and the columns of 2^L samples
// that a block holds. A single-frame block holds the columns of one wavefront
// (several short ones), or one column of two, four or eight wavefronts.
constexpr int kPostThreads = 512;
PWBF_POST_HD constexpr int post_columns(int L, int block_threads) {
  return block_threads / fft_threads(L);
}
PWBF_POST_HD constexpr int post_block(int L) { return fft_threads(L) > 64 ? fft_threads(L) : 64; }

}  // namespace pwbf

// First-level histogram of the selection (Eq. 2), shared by the selection kernels and by the
// score kernels that build it while the scores are still on chip.
#pragma once
#include "esa_common.h"

namespace esa {

constexpr int kRadixBins = 2048;
// Copies of the global histogram; workgroup w adds into copy w % kHistReplicas and a reader sums the copies.
// Adds to one address are served one after the other (about 30 ns each, measured), and where most scores share
// a bin every workgroup adds to the same few: 250 workgroups on one copy cost 5 us, on four copies 0.4 us.
constexpr int kHistReplicas = 4;
constexpr int kHistWords = kHistReplicas * kRadixBins;       // of one batch row

// Rows up to this long are selected from by one workgroup that keeps the row's keys in registers (no global
// histogram).  Measured: 4.8 / 5.5 / 7.2 / 13.2 us for up to 2 / 4 / 8 / 16 thousand scores (its LDS histogram is one
// compute unit's work), the two passes of longer rows 8 us and a launch boundary at any of these lengths.
constexpr int kSelectSmallThreads = 1024;
constexpr int kSelectSmallItems = 8;                         // keys per thread
constexpr int64_t kSelectSmallMax = kSelectSmallThreads * kSelectSmallItems;

// Bin of a value, given its order-preserving key: thirty-two bins per power of two and sign from 2^-16 to 2^16, the bins at
// the ends take what lies beyond.  The value is the score plus a shift of its row (TopkLayout::shift) that brings the bulk
// of the row near zero, where bins are narrow: a row's scores F = S - mu lie together far below zero when one token stands
// out (mu = 500 and a spread of 11 in a decode step on a long document), and binned as they are a bin there held several
// thousand of 260k keys, more than the lists of topk_compact: 264 us for that step against 39 us.  Any shift gives the same
// selection: adding a number and rounding keeps the order.
constexpr uint32_t kNegBins = 1024, kNegFirst = (127 - 16) << 5;         // magnitude >> 18 of the finest negative bin
constexpr uint32_t kPosBins = kRadixBins - kNegBins, kPosFirst = (127 - 16) << 5;
__device__ __forceinline__ uint32_t score_bin(uint32_t key) {
  const bool pos = key >= 0x80000000u;
  const int32_t unit = (int32_t)(pos ? (key - 0x80000000u) >> 18 : (0x7FFFFFFFu - key) >> 18);
  int32_t b = unit - (int32_t)(pos ? kPosFirst : kNegFirst);
  const int32_t most = (int32_t)(pos ? kPosBins : kNegBins) - 1;
  b = b < 0 ? 0 : (b > most ? most : b);
  return pos ? kNegBins + (uint32_t)b : kNegBins - 1 - (uint32_t)b;
}
__device__ __forceinline__ uint32_t shifted_bin(float score, float shift) { return score_bin(ordered_key(score + shift)); }
// The shift from a row maximum of S (none where that is not a number to add).
__device__ __forceinline__ float shift_of(float mu) { return fabsf(mu) < 1e30f ? mu : 0.f; }
// Smallest and largest key of an unshifted bin.
__device__ __forceinline__ void bin_keys(uint32_t bin, uint32_t* lo, uint32_t* hi) {
  const bool pos = bin >= kNegBins;
  const uint32_t b = pos ? bin - kNegBins : kNegBins - 1 - bin, last = (pos ? kPosBins : kNegBins) - 1;
  const int shift = 18;
  const uint32_t first = pos ? kPosFirst : kNegFirst;
  const uint32_t m_lo = b == 0 ? 0u : (first + b) << shift;
  const uint32_t m_hi = b == last ? 0x7FFFFFFFu : ((first + b + 1) << shift) - 1;
  *lo = pos ? 0x80000000u + m_lo : 0x7FFFFFFFu - m_hi;
  *hi = pos ? 0x80000000u + m_hi : 0x7FFFFFFFu - m_lo;
}

// Workspace of one batch row of the selection, in uint32 words.
struct TopkLayout {
  static constexpr int hist = 0;                              // [kHistReplicas][kRadixBins]
  static constexpr int pick = kHistWords;                     // [3]: bin of the k-th score, keys in it, its rank inside the bin
  static constexpr int shift = kHistWords + 3;                // fp32: written with the histogram
  static constexpr int blk = kHistWords + 4;                  // [2][nblk]: per workgroup, scores above the bin / inside it
  // then [nblk][cap]: keys inside the bin
};

// One LDS-histogram increment per lane.  With bins this fine a wave's 64 scores fall into dozens of them; folding the
// lanes that share the first lane's bin into one atomic, which paid when four fifths of a row shared a bin, cost more
// than the few lanes served one after the other.
__device__ __forceinline__ void hist_add(uint32_t* h, bool active, uint32_t bin) {
  if (active) atomicAdd(&h[bin], 1u);
}

// A workgroup's finished LDS histogram h, added to its copy of the global histogram gh ([kHistReplicas][kRadixBins]).
__device__ __forceinline__ void hist_flush(uint32_t* __restrict__ gh, const uint32_t* h, int wg, int tid, int n_threads) {
  uint32_t* g = gh + (wg % kHistReplicas) * kRadixBins;
  for (int i = tid; i < kRadixBins; i += n_threads)
    if (h[i]) atomicAdd(&g[i], h[i]);
}

// Words of one batch row's selection workspace and the stride between rows (host side).
int64_t topk_row_stride_words(int64_t n, int batch);
// Tiles of 1024 scores that a workgroup of the selection takes (host side).
int topk_tiles_per_wg(int64_t n, int batch);

}  // namespace esa

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

// Bin of a score, given its order-preserving key: monotone, and much finer than the key's leading bits where the
// scores of Eq. 4 are (F = S - mu <= 0, most of it within a few powers of two): sixty-four bins per power of two for
// negative scores from 2^-12 to 2^12, sixteen per power of two for positive ones from 2^-16 to 2^16, the bins at the
// ends take what lies beyond.  A bin of the leading eleven key bits (four per power of two) held up to four fifths of a
// row; the bin of the k-th score now holds well under one per cent of it (a few hundred of 128k), so that the keys inside
// it can be listed and the exact threshold picked from the list.
constexpr uint32_t kNegBins = 1536, kNegFirst = (127 - 12) << 6;         // magnitude >> 17 of the finest negative bin
constexpr uint32_t kPosBins = kRadixBins - kNegBins, kPosFirst = (127 - 16) << 4;     // magnitude >> 19
__device__ __forceinline__ uint32_t score_bin(uint32_t key) {
  const bool pos = key >= 0x80000000u;
  const int32_t unit = (int32_t)(pos ? (key - 0x80000000u) >> 19 : (0x7FFFFFFFu - key) >> 17);
  int32_t b = unit - (int32_t)(pos ? kPosFirst : kNegFirst);
  const int32_t most = (int32_t)(pos ? kPosBins : kNegBins) - 1;
  b = b < 0 ? 0 : (b > most ? most : b);
  return pos ? kNegBins + (uint32_t)b : kNegBins - 1 - (uint32_t)b;
}
// Smallest and largest key of a bin.
__device__ __forceinline__ void bin_keys(uint32_t bin, uint32_t* lo, uint32_t* hi) {
  const bool pos = bin >= kNegBins;
  const uint32_t b = pos ? bin - kNegBins : kNegBins - 1 - bin, last = (pos ? kPosBins : kNegBins) - 1;
  const int shift = pos ? 19 : 17;
  const uint32_t first = pos ? kPosFirst : kNegFirst;
  const uint32_t m_lo = b == 0 ? 0u : (first + b) << shift;
  const uint32_t m_hi = b == last ? 0x7FFFFFFFu : ((first + b + 1) << shift) - 1;
  *lo = pos ? 0x80000000u + m_lo : 0x7FFFFFFFu - m_hi;
  *hi = pos ? 0x80000000u + m_hi : 0x7FFFFFFFu - m_lo;
}

// Workspace of one batch row of the selection, in uint32 words.
struct TopkLayout {
  static constexpr int hist = 0;                              // [kHistReplicas][kRadixBins]
  static constexpr int pick = kHistWords;                     // [4]: bin of the k-th score, its rank inside the bin
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

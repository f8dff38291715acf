// Histograms of the selection (Eq. 2): the first digit's, shared by the selection kernels of long rows and by the score
// kernels that build it while the scores are still on chip, and the finer bins of the rows that one workgroup takes.
#pragma once
#include "esa_common.h"

namespace esa {

constexpr int kRadixBins = 2048;        // 11-bit digits (the last pass uses 10 bits of them)
// Copies of the global histogram; workgroup w adds into copy w % kHistReplicas and a reader sums the copies.
// Adds to one address are served one after the other (about 30 ns each, measured), and where most scores share
// a digit every workgroup adds to the same few: 250 workgroups on one copy cost 5 us, on four copies 0.4 us.
constexpr int kHistReplicas = 4;
constexpr int kHistWords = 3 * kHistReplicas * kRadixBins;   // the three passes' histograms of one batch row

// Rows up to this long are selected from by one workgroup that keeps the row's keys in registers (no global
// histogram).  Measured: 6.0 / 7.8 us for 3.8 / 8.2 thousand N(0,1) scores, 5 to 12 us for crowded ones and 28 where all
// are equal (its LDS histogram is one compute unit's work); the passes of longer rows take 15 us at any of these lengths.
constexpr int kSelectSmallThreads = 1024;
constexpr int kSelectSmallItems = 8;                         // keys per thread
constexpr int64_t kSelectSmallMax = kSelectSmallThreads * kSelectSmallItems;

// Digit of the first histogram of a long row, given a score's order-preserving key.
__device__ __forceinline__ uint32_t score_digit(uint32_t key) { return key >> 21; }

// Bin of a score in a short row's first histogram, given its key: thirty-two bins per power of two and sign from 2^-16 to
// 2^16, the bins at the ends take what lies beyond.
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
// Smallest and largest key of a bin.
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
  static constexpr int hist = 0;                              // [3][kHistReplicas][kRadixBins]
  static constexpr int pick = kHistWords;                     // [2][2]: (bin, remaining rank) chosen in the first / second histogram
  static constexpr int blk = kHistWords + 4;                  // [2][nblk]: per workgroup, scores above the 22-bit prefix / sharing it
  // then [nblk][cap] uint16: last digits of the scores sharing the prefix, cap = scores per workgroup
};

// One LDS-histogram increment per lane, with the lanes of a wave that hit the leader's bin folded into a single atomic
// (scores of one row share their exponent, so in the first pass almost every lane hits the same bin).  Every lane of the
// wave must call it.
__device__ __forceinline__ void hist_add(uint32_t* h, bool active, uint32_t bin) {
  const uint64_t act = __ballot(active);
  if (act == 0ull) return;
  const int leader = __ffsll((long long)act) - 1;
  const uint32_t lead_bin = (uint32_t)__builtin_amdgcn_readlane((int)bin, leader);     // leader is the same in every lane
  const uint64_t same = __ballot(active && bin == lead_bin);
  if ((int)(__builtin_amdgcn_workitem_id_x() & 63) == leader) atomicAdd(&h[lead_bin], (uint32_t)__popcll(same));
  if (active && bin != lead_bin) atomicAdd(&h[bin], 1u);
}
// The same without folding, for a short row's finer bins: a wave's 64 scores fall into dozens of them, and folding cost more
// than the few lanes served one after the other (8192 scores: 7.2 against 6.0 us).
__device__ __forceinline__ void bin_add(uint32_t* h, bool active, uint32_t bin) {
  if (active) atomicAdd(&h[bin], 1u);
}

// A first histogram in LDS of which every fourth lane has a copy of its own, [kRadixBins][kLaneCopies], 16-byte aligned: the scores of
// a row crowd into some five bins, and lanes of one instruction that add to one address are served one after the other.  A
// sixteenth of a wave in turn costs less than two ballots and what folding the leader's bin leaves: score_finish of sixteen rows of 260k
// scores 13.8 -> 10.8 us (13.0 with both), of four rows of 100k 6.1 -> 5.6, of one row the same (four times the words to clear).
constexpr int kLaneCopies = 4;
__device__ __forceinline__ void lane_copies_clear(uint32_t* h, int tid, int n_threads) {
  for (int i = tid; i < kRadixBins; i += n_threads) ((uint4*)h)[i] = make_uint4(0u, 0u, 0u, 0u);
}
__device__ __forceinline__ void lane_copies_add(uint32_t* h, bool active, uint32_t bin, int lane) {
  if (active) atomicAdd(&h[bin * kLaneCopies + (lane & (kLaneCopies - 1))], 1u);
}
__device__ __forceinline__ void lane_copies_flush(uint32_t* __restrict__ gh, const uint32_t* h, int wg, int tid, int n_threads) {
  uint32_t* g = gh + (wg % kHistReplicas) * kRadixBins;
  for (int i = tid; i < kRadixBins; i += n_threads) {
    const uint4 c = ((const uint4*)h)[i];
    const uint32_t sum = c.x + c.y + c.z + c.w;
    if (sum) atomicAdd(&g[i], sum);
  }
}

// A workgroup's finished LDS histogram h, added to its copy of one pass's global histogram gh ([kHistReplicas][kRadixBins]).
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

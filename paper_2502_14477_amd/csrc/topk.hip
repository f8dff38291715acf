// Token-level top-k over the middle-token scores (Eq. 2): exact selection on order-preserving 32-bit keys, then an
// ordered compaction (ascending positions; equal scores: the lower position wins).
//
// Rows of up to kSelectSmallMax scores: one workgroup per row keeps the row's keys in registers and does everything
// in one launch (select_small), including what the score call would otherwise need a pass of its own for (mu of a
// single current token, Eq. 8's pooling).
//
// Longer rows: three histogram passes (11 + 11 + 10 bits, most significant first) pin down the key T of the k-th
// largest score and how many scores equal to T are still needed; the first histogram is built by the kernel that writes
// the scores where that can.  A writing pass then emits the positions.  For its output offsets a workgroup of it needs
// the number of selected scores in the workgroups before it; the third histogram pass leaves that per workgroup in two
// pieces: the count of scores above the 22-bit prefix fixed so far (selected whatever the last digit of T turns out to
// be), and the list of the last digits of the scores that share the prefix (usually a handful), which the writing pass
// compares with T's last digit once it knows it.
// Why digits of the key and not finer bins: no bin that is fixed before the scores are known is fine enough for every
// row.  One histogram of 32 bins per power of two around an estimate of the row's bulk, and lists of the keys in the
// threshold's bin, save a pass where the selected tokens stand clear of all others (260k scores: 25.0 against 27.3 us for
// a decode step's score and selection) and lose wherever they do not: N(0,1) scores 30.9 against 27.7 us, a passage of
// 3000 tokens of similar score 275 against 15, a chunk whose first query is fifty times the others 446 against 139.
// All cross-block traffic is integer atomics and plain stores, so the result is deterministic.
// No workgroup ever waits for another: what one pass leaves in global memory (a 2048-bin histogram, or the per-workgroup
// counts) is re-read and scanned by EVERY workgroup of the next launch, redundantly, instead of being finished by a
// last-arriving workgroup: a launch is then one round trip to memory plus a little LDS work, which is what bounds this
// latency-bound call.
#include <atomic>

#include "esa_common.h"
#include "radix_hist.h"

namespace esa {
namespace {

constexpr int kThreads = 512;
constexpr int kItems = 2;                       // scores per thread and tile
constexpr int kTile = kThreads * kItems;        // scores per block
constexpr int kBins = kRadixBins;
constexpr int kBinsPerThread = kBins / kThreads;

struct TopkPlan {
  int64_t sub;      // tiles of kTile scores per workgroup
  int64_t nblk;     // workgroups per row
};
// One tile of kTile scores per workgroup while that keeps the chip busy (a call is latency-bound
// then); with many rows a workgroup takes several tiles, so that the fixed work per workgroup
// (prefix resolution, histogram flush) is paid by fewer of them.
__host__ inline TopkPlan topk_plan(int64_t n, int batch) {
  const int64_t tiles = (n + kTile - 1) / kTile;
  int64_t sub = (tiles * batch + 767) / 768;
  sub = sub < 1 ? 1 : (sub > 8 ? 8 : sub);
  TopkPlan p;
  p.sub = sub;
  p.nblk = (tiles + sub - 1) / sub;
  return p;
}
__host__ inline int64_t topk_row_words(const TopkPlan& p) {
  const int64_t cand_words = (p.nblk * p.sub * kTile + 1) / 2;
  return TopkLayout::blk + 2 * p.nblk + cand_words;
}

// Inclusive prefix sum over the 64 lanes of a wave in the vector unit: shifts inside the 16-lane rows, then the
// last lane of row 0 / 2 is added into row 1 / 3 and lane 31 into the upper half (every lane of the wave must be
// active).  The LDS-routed shuffles this replaces cost a crossbar round trip per step.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);   // row_shr:1 (lanes without a source add 0)
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);   // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);   // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);   // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1 and 3
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2 and 3
  return v;
}

// Exclusive prefix sum of one value per thread over the block.
template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* wave_sums) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t incl = wave_incl_scan(v);
  __syncthreads();                       // wave_sums may still be read from a previous call
  if (lane == 63) wave_sums[w] = incl;
  __syncthreads();
  uint32_t base = 0;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) base += i < w ? wave_sums[i] : 0u;
  return base + incl - v;
}

// Where rank k_rem falls in a histogram of 2048 bins, walking from the top bin down: the bin, its population, and
// the rank inside it.  Thread t owns bins kBins - 1 - t * PER .. downwards, c[0] the highest.  Every thread of the
// block gets the result.
struct BinPick {
  uint32_t bin, count, k_rem;
};
template <int NT>
__device__ __forceinline__ BinPick pick_bin(const uint32_t (&c)[kBins / NT], uint32_t k_rem, uint32_t* wave_sums,
                                            uint32_t* result) {
  constexpr int kPer = kBins / NT;
  const int top = kBins - 1 - threadIdx.x * kPer;
  uint32_t mine = 0;
#pragma unroll
  for (int e = 0; e < kPer; ++e) mine += c[e];
  const uint32_t above = block_excl_scan<NT>(mine, wave_sums);
  if (above < k_rem && k_rem <= above + mine) {          // exactly one thread
    uint32_t cum = above;
    bool done = false;
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      if (!done && cum + c[e] >= k_rem) {
        result[0] = (uint32_t)(top - e);
        result[1] = c[e];
        result[2] = k_rem - cum;
        done = true;
      }
      cum += c[e];
    }
  }
  __syncthreads();
  const BinPick r = {result[0], result[1], result[2]};
  __syncthreads();                       // result[] is free for the next pick
  return r;
}
// This thread's bins of a histogram in LDS.
template <int NT>
__device__ __forceinline__ void lds_bins(const uint32_t* h, uint32_t (&c)[kBins / NT]) {
#pragma unroll
  for (int e = 0; e < kBins / NT; ++e) c[e] = h[kBins - 1 - (int)threadIdx.x * (kBins / NT) - e];
}

// Keys in [lo, hi] of which the k_rem largest are wanted, narrowed until they all are or only one value is left:
// the caller then takes every key above hi and the first k_rem keys (by position) in [lo, hi].
// add(lo, hi, shift) adds the digits ((key - lo) >> shift) of the keys in [lo, hi] to the histogram.
struct Narrowed {
  uint32_t lo, hi, k_rem;
};
template <int NT, typename Add>
__device__ __forceinline__ Narrowed narrow(Narrowed r, uint32_t count, uint32_t* h, uint32_t* wave_sums, uint32_t* result,
                                           Add&& add) {
  while (r.lo != r.hi && count != r.k_rem) {             // the same in every thread
    const int bits = 32 - __clz(r.hi - r.lo), shift = bits > 11 ? bits - 11 : 0;
    for (int i = threadIdx.x; i < kBins; i += NT) h[i] = 0u;
    __syncthreads();
    add(r.lo, r.hi, shift);
    __syncthreads();
    uint32_t c[kBins / NT];
    lds_bins<NT>(h, c);
    const BinPick p = pick_bin<NT>(c, r.k_rem, wave_sums, result);
    const uint32_t lo = r.lo + (p.bin << shift), last = lo + ((1u << shift) - 1u);
    r.hi = last < r.hi ? last : r.hi;
    r.lo = lo;
    r.k_rem = p.k_rem;
    count = p.count;
  }
  return r;
}

// This thread's share of a finished histogram in global memory ([kHistReplicas][kBins]); thread 0 owns the highest bins.
__device__ __forceinline__ void load_slice(const uint32_t* __restrict__ gh, uint32_t (&c)[kBinsPerThread]) {
  static_assert(kBinsPerThread == 4, "one 16-byte load per copy");
  const uint4* lowest = (const uint4*)gh + (kThreads - 1 - threadIdx.x);      // bins top-3 .. top of this thread
  uint4 copy[kHistReplicas];
#pragma unroll
  for (int r = 0; r < kHistReplicas; ++r) copy[r] = lowest[r * (kBins / 4)];
  uint4 t = copy[0];
#pragma unroll
  for (int r = 1; r < kHistReplicas; ++r) {
    t.x += copy[r].x; t.y += copy[r].y; t.z += copy[r].z; t.w += copy[r].w;
  }
  c[0] = t.w; c[1] = t.z; c[2] = t.y; c[3] = t.x;
}

// Key bits fixed by the passes before PASS, and the rank still to find below them.  A pass picks one histogram itself
// (the one the pass before it filled) and reads what the earlier passes picked from the workspace, where the pass that
// made the pick left it (every workgroup writes the same two words); all of it is one round trip.
template <int PASS>
__device__ __forceinline__ void resolve_prefix(uint32_t* __restrict__ w, uint32_t k, uint32_t* wave_sums,
                                               uint32_t* result, uint32_t* prefix, uint32_t* k_rem) {
  *prefix = 0;
  *k_rem = k;
  if constexpr (PASS > 0) {
    uint32_t c[kBinsPerThread];
    load_slice(w + TopkLayout::hist + (PASS - 1) * kHistReplicas * kBins, c);
    uint32_t bin[3] = {0, 0, 0}, rank = k;
#pragma unroll
    for (int p = 0; p < PASS - 1; ++p) {
      bin[p] = w[TopkLayout::pick + 2 * p];
      rank = w[TopkLayout::pick + 2 * p + 1];
    }
    const BinPick b = pick_bin<kThreads>(c, rank, wave_sums, result);
    bin[PASS - 1] = b.bin;
    if (PASS < 3 && threadIdx.x == 0) {
      w[TopkLayout::pick + 2 * (PASS - 1)] = b.bin;
      w[TopkLayout::pick + 2 * (PASS - 1) + 1] = b.k_rem;
    }
    *prefix = (bin[0] << 21) | (bin[1] << 10) | bin[2];
    *k_rem = b.k_rem;
  }
}

__global__ void topk_init(uint32_t* ws, int64_t row_words) {
  uint32_t* w = ws + (int64_t)blockIdx.y * row_words;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < kHistWords; i += gridDim.x * blockDim.x) w[i] = 0u;
}

// PASS 0: bits 31..21, PASS 1: bits 20..10, PASS 2: bits 9..0.  SUB: tiles of a workgroup, all of whose scores are requested in front
// of the prefix resolution (sixteen rows of 260k: 7.3 and 7.7 us a pass with a tile requested at a time, 6.6 and 7.6 now).
template <int PASS, int SUB>
__global__ __launch_bounds__(kThreads) void topk_hist(const float* __restrict__ score, int64_t n, int64_t score_bs,
                                                      uint32_t* __restrict__ ws, int64_t row_words, int nblk,
                                                      uint32_t k) {
  __shared__ uint32_t h[kBins];
  __shared__ uint32_t wave_sums[kThreads / 64];
  __shared__ uint32_t result[3];
  __shared__ uint32_t n_above, n_cand;             // PASS 2: this workgroup's scores above / sharing the prefix
  const float* row = score + (int64_t)blockIdx.y * score_bs;
  uint32_t* w = ws + (int64_t)blockIdx.y * row_words;
  constexpr int kMine = kItems * SUB;
  const int64_t first = (int64_t)blockIdx.x * kTile * SUB + threadIdx.x;
  float v[kMine];                                  // unconditional loads: a position past the end reads score 0 instead
#pragma unroll
  for (int e = 0; e < kMine; ++e) v[e] = row[first + e * kThreads < n ? first + e * kThreads : 0];
  for (int i = threadIdx.x; i < kBins; i += kThreads) h[i] = 0u;
  if (threadIdx.x == 0) {
    n_above = 0u;
    n_cand = 0u;
  }
  uint32_t prefix, k_rem;
  resolve_prefix<PASS>(w, k, wave_sums, result, &prefix, &k_rem);
  __syncthreads();
  uint16_t* cand = (uint16_t*)(w + TopkLayout::blk + 2 * nblk) + (int64_t)blockIdx.x * kTile * SUB;
  uint32_t above = 0;
#pragma unroll
  for (int e = 0; e < kMine; ++e) {
    const bool ok = first + e * kThreads < n;
    const uint32_t key = ordered_key(v[e]);
    if (PASS == 0) {
      hist_add(h, ok, score_digit(key));
    } else if (PASS == 1) {
      hist_add(h, ok && (key >> 21) == (prefix >> 21), (key >> 10) & 2047u);
    } else {
      const bool shares = ok && (key >> 10) == (prefix >> 10);
      hist_add(h, shares, key & 1023u);
      above += (ok && (key >> 10) > (prefix >> 10)) ? 1u : 0u;
      if (shares) cand[atomicAdd(&n_cand, 1u)] = (uint16_t)(key & 1023u);   // order does not matter: they are counted
    }
  }
  if (PASS == 2) {
    above = wave_incl_scan(above);                 // lane 63 holds the wave's total
    if ((threadIdx.x & 63) == 63) atomicAdd(&n_above, above);
  }
  __syncthreads();
  hist_flush(w + TopkLayout::hist + PASS * kHistReplicas * kBins, h, blockIdx.x, threadIdx.x, kThreads);
  if (PASS == 2 && threadIdx.x == 0) {
    w[TopkLayout::blk + blockIdx.x] = n_above;
    w[TopkLayout::blk + nblk + blockIdx.x] = n_cand;
  }
}

// A wave owns consecutive scores, a lane every 64th of them, so that two ballots per 64 scores give every selected one its place
// and the waves meet once, whatever SUB (the tiles of a workgroup) is.  What bounds it: two round trips, the prefix resolution, a barrier.
// With a block scan per tile and consecutive scores to a lane it took 11.9 us for sixteen rows of 260k scores (SUB 6), 9.1 now, and
// 4.2 / 4.2 for one row; with the histogram passes as they are now a call 34.9 -> 30.2, 64 rows of 100k 49.9 -> 45.0.
template <int SUB>
__global__ __launch_bounds__(kThreads) void topk_write(const float* __restrict__ score, int64_t n, int64_t score_bs,
                                                       uint32_t* __restrict__ ws, int64_t row_words, int nblk,
                                                       int64_t base, int32_t* __restrict__ idx, int64_t idx_bs,
                                                       uint32_t k) {
  constexpr int kW = kThreads / 64, kMine = kItems * SUB;
  __shared__ uint32_t wave_sums[kW];
  __shared__ uint32_t result[3];
  __shared__ uint32_t before[2][kW], mine[2][kW];        // selected / equal to T: in earlier workgroups, in this one's waves
  const float* row = score + (int64_t)blockIdx.y * score_bs;
  uint32_t* w = ws + (int64_t)blockIdx.y * row_words;
  int32_t* out = idx + (int64_t)blockIdx.y * idx_bs;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t first = (int64_t)blockIdx.x * kTile * SUB + wave * (64 * kMine) + lane;
  const int left = (int)(n - first < 64 * kMine ? n - first : 64 * kMine);   // 64 * e < left: the lane has an e-th score
  uint32_t key[kMine];
  {
    float v[kMine];                                      // unconditional loads: a position past the end reads score 0 instead
#pragma unroll
    for (int e = 0; e < kMine; ++e) v[e] = row[64 * e < left ? first + 64 * e : 0];
#pragma unroll
    for (int e = 0; e < kMine; ++e) key[e] = ordered_key(v[e]);
  }
  // What the third histogram pass left about the first workgroup this thread looks at: requested
  // before T is resolved, so that the two round trips overlap.
  constexpr int kPeek = 4;
  const uint16_t* cand_all = (const uint16_t*)(w + TopkLayout::blk + 2 * nblk);
  constexpr int64_t cap = (int64_t)kTile * SUB;
  uint32_t c0 = 0, above0 = 0, peek[kPeek];
#pragma unroll
  for (int j = 0; j < kPeek; ++j) peek[j] = 0u;
  if ((int)threadIdx.x < (int)blockIdx.x) {
    above0 = w[TopkLayout::blk + threadIdx.x];
    c0 = w[TopkLayout::blk + nblk + threadIdx.x];
    // read whether or not that workgroup left so many (its slots exist either way; the count decides below what
    // is used): asking for the count first would put a second round trip in front of them
    static_assert(kPeek <= kTile, "a workgroup's candidate slots");
#pragma unroll
    for (int j = 0; j < kPeek; ++j) peek[j] = cand_all[threadIdx.x * cap + j];
  }
  uint32_t T, need;                                      // need: equal-to-T scores to take, lowest positions first
  resolve_prefix<3>(w, k, wave_sums, result, &T, &need);
  // scores above / equal to T in the workgroups before this one: those above the 22-bit prefix, plus
  // those sharing it whose last digit is above / equal to T's
  const uint32_t t_digit = T & 1023u;
  uint32_t my_gt = 0, my_eq = 0;
  for (int i = threadIdx.x; i < (int)blockIdx.x; i += kThreads) {
    const bool head = i == (int)threadIdx.x;
    uint32_t c = head ? c0 : w[TopkLayout::blk + nblk + i];
    c = c < (uint32_t)cap ? c : (uint32_t)cap;           // a workgroup cannot have left more than its scores: the reads below stay inside its slots
    my_gt += head ? above0 : w[TopkLayout::blk + i];
    uint32_t j0 = 0;
    if (head) {
#pragma unroll
      for (int j = 0; j < kPeek; ++j) {
        my_gt += ((uint32_t)j < c && peek[j] > t_digit) ? 1u : 0u;
        my_eq += ((uint32_t)j < c && peek[j] == t_digit) ? 1u : 0u;
      }
      j0 = kPeek;
    }
    for (uint32_t j = j0; j < c; ++j) {
      const uint32_t dgt = cand_all[i * cap + j];
      my_gt += dgt > t_digit ? 1u : 0u;
      my_eq += dgt == t_digit ? 1u : 0u;
    }
  }
  my_gt = wave_incl_scan(my_gt);                         // lane 63 holds the wave's total
  my_eq = wave_incl_scan(my_eq);
  uint32_t gt = 0, eq = 0;                               // of the wave
#pragma unroll
  for (int e = 0; e < kMine; ++e) {
    const bool ok = 64 * e < left;
    gt += (uint32_t)__popcll(__ballot(ok && key[e] > T));
    eq += (uint32_t)__popcll(__ballot(ok && key[e] == T));
  }
  if (lane == 63) {
    before[0][wave] = my_gt;
    before[1][wave] = my_eq;
    mine[0][wave] = gt;
    mine[1][wave] = eq;
  }
  __syncthreads();
  uint32_t g0 = 0, e0 = 0;
#pragma unroll
  for (int i = 0; i < kW; ++i) {
    g0 += before[0][i] + (i < wave ? mine[0][i] : 0u);
    e0 += before[1][i] + (i < wave ? mine[1][i] : 0u);
  }
  if (gt + eq == 0u) return;                             // the same in every lane
  const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
  for (int e = 0; e < kMine; ++e) {
    const bool ok = 64 * e < left;
    const bool is_gt = ok && key[e] > T, is_eq = ok && key[e] == T;
    const uint64_t mg = __ballot(is_gt), me = __ballot(is_eq);
    const uint32_t gb = g0 + (uint32_t)__popcll(mg & below), eb = e0 + (uint32_t)__popcll(me & below);
    if (is_gt || (is_eq && eb < need)) {
      const uint32_t slot = gb + (eb < need ? eb : need);
      if (slot < k) out[slot] = (int32_t)(base + first + 64 * e);
    }
    g0 += (uint32_t)__popcll(mg);
    e0 += (uint32_t)__popcll(me);
  }
}

// A whole row in one workgroup: wave w holds scores [64 * ITEMS * w, ...), lane l of it every 64th, so that loads are
// coalesced and (item, lane) is position order inside the wave.  Before the selection it finishes the scores where
// that is left to do (see ScoreTail): pooling over +-eps, minus mu = the largest of n_part partial maxima.
// What bounds it: round trips and barriers (two loads deep, a histogram or two, one scan): 5.5 us at 3.8k scores
// where the four launches it replaces (subtract mu, two histogram passes, write) took 13.7 us.
template <int ITEMS>
__global__ __launch_bounds__(kSelectSmallThreads) void select_small(ScoreTail t, float* __restrict__ score, int64_t score_bs,
                                                                    int n, int64_t base, int32_t* __restrict__ idx,
                                                                    int64_t idx_bs, uint32_t k) {
  constexpr int NT = kSelectSmallThreads, kW = NT / 64;
  extern __shared__ float staged[];              // [n] unpooled scores when pooling
  __shared__ uint32_t h[kBins];
  __shared__ uint32_t wave_sums[2 * kW];
  __shared__ uint32_t result[3];
  const float* in = t.in + (int64_t)blockIdx.x * t.in_bs;
  int32_t* out = idx + (int64_t)blockIdx.x * idx_bs;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int first = wave * 64 * ITEMS + lane;
  float x[ITEMS];
#pragma unroll
  for (int e = 0; e < ITEMS; ++e) x[e] = in[first + 64 * e < n ? first + 64 * e : 0];
  float mu = 0.f;
  if (t.part) {
    const float* part = t.part + (int64_t)blockIdx.x * t.n_part;
    float m = -INFINITY;
    for (int i = tid; i < t.n_part; i += NT) m = fmaxf(m, part[i]);
    m = wave_max(m);
    if (lane == 0) wave_sums[wave] = __float_as_uint(m);
  }
  for (int i = tid; i < kBins; i += NT) h[i] = 0u;
  if (t.eps > 0) {
#pragma unroll
    for (int e = 0; e < ITEMS; ++e)
      if (first + 64 * e < n) staged[first + 64 * e] = x[e];
  }
  __syncthreads();
  if (t.part) {
    mu = __uint_as_float(wave_sums[0]);
#pragma unroll
    for (int i = 1; i < kW; ++i) mu = fmaxf(mu, __uint_as_float(wave_sums[i]));
  }
  uint32_t key[ITEMS];
#pragma unroll
  for (int e = 0; e < ITEMS; ++e) {
    const int i = first + 64 * e;
    const bool ok = i < n;
    float f = x[e];
    if (t.eps > 0 && ok) {                       // max - mu rounds as the max over the rounded differences does
      const int a = i - t.eps > 0 ? i - t.eps : 0, b = i + t.eps < n - 1 ? i + t.eps : n - 1;
      for (int j = a; j <= b; ++j) f = fmaxf(f, staged[j]);
    }
    if (t.part) f -= mu;
    if (ok && score) score[(int64_t)blockIdx.x * score_bs + i] = f;
    key[e] = ordered_key(f);
    bin_add(h, ok, score_bin(key[e]));
  }
  __syncthreads();
  uint32_t c[kBins / NT];
  lds_bins<NT>(h, c);
  const BinPick p = pick_bin<NT>(c, k, wave_sums, result);
  Narrowed r;
  bin_keys(p.bin, &r.lo, &r.hi);
  r.k_rem = p.k_rem;
  r = narrow<NT>(r, p.count, h, wave_sums, result, [&](uint32_t lo, uint32_t hi, int shift) {
#pragma unroll
    for (int e = 0; e < ITEMS; ++e)
      bin_add(h, first + 64 * e < n && key[e] >= lo && key[e] <= hi, (key[e] - lo) >> shift);
  });
  uint32_t gt = 0, eq = 0;                       // of the wave
#pragma unroll
  for (int e = 0; e < ITEMS; ++e) {
    const bool ok = first + 64 * e < n;
    gt += (uint32_t)__popcll(__ballot(ok && key[e] > r.hi));
    eq += (uint32_t)__popcll(__ballot(ok && key[e] >= r.lo && key[e] <= r.hi));
  }
  if (lane == 0) {
    wave_sums[wave] = gt;
    wave_sums[kW + wave] = eq;
  }
  __syncthreads();
  uint32_t g0 = 0, e0 = 0;
#pragma unroll
  for (int i = 0; i < kW; ++i) {
    g0 += i < wave ? wave_sums[i] : 0u;
    e0 += i < wave ? wave_sums[kW + i] : 0u;
  }
  const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
  for (int e = 0; e < ITEMS; ++e) {
    const bool ok = first + 64 * e < n;
    const bool is_gt = ok && key[e] > r.hi, is_eq = ok && !is_gt && key[e] >= r.lo;
    const uint64_t mg = __ballot(is_gt), me = __ballot(is_eq);
    const uint32_t gb = g0 + (uint32_t)__popcll(mg & below), eb = e0 + (uint32_t)__popcll(me & below);
    if (is_gt || (is_eq && eb < r.k_rem)) {
      const uint32_t slot = gb + (eb < r.k_rem ? eb : r.k_rem);
      if (slot < k) out[slot] = (int32_t)(base + first + 64 * e);
    }
    g0 += (uint32_t)__popcll(mg);
    e0 += (uint32_t)__popcll(me);
  }
}

// k >= n: every middle token is selected.
__global__ void topk_all(int64_t n, int64_t base, int32_t* idx, int64_t idx_bs) {
  int32_t* out = idx + (int64_t)blockIdx.y * idx_bs;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    out[i] = (int32_t)(base + i);
}

// The passes of long rows, with SUB tiles to a workgroup.
template <int SUB>
void launch_passes(const float* score, int64_t n, int64_t score_bs, uint32_t* w, int64_t row_words, dim3 grid, int64_t base,
                   int32_t* idx, int64_t idx_bs, uint32_t k, bool first_hist_ready, hipStream_t st) {
  const int nblk = (int)grid.x;
  if (!first_hist_ready) topk_hist<0, SUB><<<grid, kThreads, 0, st>>>(score, n, score_bs, w, row_words, nblk, k);
  topk_hist<1, SUB><<<grid, kThreads, 0, st>>>(score, n, score_bs, w, row_words, nblk, k);
  topk_hist<2, SUB><<<grid, kThreads, 0, st>>>(score, n, score_bs, w, row_words, nblk, k);
  topk_write<SUB><<<grid, kThreads, 0, st>>>(score, n, score_bs, w, row_words, nblk, base, idx, idx_bs, k);
}

}  // namespace

// ---------------------------------------------------------------- library-owned scratch (no caller workspace)
// For callers that cannot allocate.  One array per GPU, held until the process ends; every call on
// a GPU shares it, so calls that overlap in time on one GPU race.  In host code the array's name is
// only a handle: its device address is looked up once per device and that address is what the
// kernels are given.
constexpr size_t kStaticScratchBytes = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
static std::atomic<void*> g_scratch_addr[kMaxDevices];

// Device address of `scratch` on the current device (looked up on first use).
static int static_scratch(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_failed(e, "hipGetDevice");
  if (dev < 0 || dev >= kMaxDevices) ESA_FAIL(ESA_EUNSUPPORTED, "device ordinal %d beyond %d", dev, kMaxDevices - 1);
  void* p = g_scratch_addr[dev].load(std::memory_order_acquire);
  if (!p) {
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return hip_failed(e, "hipGetSymbolAddress(scratch)");
    g_scratch_addr[dev].store(p, std::memory_order_release);     // every thread finds the same address
  }
  *out = p;
  return ESA_OK;
}

size_t topk_static_capacity() { return kStaticScratchBytes; }

int topk_static_prepare() {
  void* p;
  return static_scratch(&p);
}

int launch_topk_static(const float* score, int64_t n, int k, int64_t base, int32_t* idx, int batch, int64_t score_bs,
                       int64_t idx_bs, hipStream_t st) {
  const size_t need = topk_workspace_bytes(n, k, batch);
  if (need > kStaticScratchBytes)
    ESA_FAIL(ESA_EWORKSPACE, "esa_select_topk_static: %lld scores x %d rows need %zu bytes of scratch, the library holds %zu",
             (long long)n, batch, need, kStaticScratchBytes);
  void* ws = nullptr;
  const int rc = static_scratch(&ws);
  if (rc != ESA_OK) return rc;
  return launch_topk(score, n, k, base, idx, batch, score_bs, idx_bs, ws, kStaticScratchBytes, st, false);
}

size_t topk_workspace_bytes(int64_t n, int k, int batch) {
  if (n <= 0 || k <= 0 || batch <= 0 || k >= n) return 256;
  return align_up((size_t)topk_row_words(topk_plan(n, batch)) * sizeof(uint32_t), 256) * (size_t)batch;
}

int64_t topk_row_stride_words(int64_t n, int batch) {
  return (int64_t)(align_up((size_t)topk_row_words(topk_plan(n, batch)) * sizeof(uint32_t), 256) / sizeof(uint32_t));
}

int topk_tiles_per_wg(int64_t n, int batch) {
  static_assert(kTile == 1024, "tiles of the kernels that write the scores");
  return (int)topk_plan(n, batch).sub;
}

int launch_select_small(const ScoreTail& tail, float* score, int64_t score_bs, int64_t n, int k, int64_t base, int32_t* idx,
                        int64_t idx_bs, int batch, hipStream_t st) {
  const size_t lds = tail.eps > 0 ? (size_t)n * sizeof(float) : 0;
  const auto kernel = n <= kSelectSmallThreads * 2   ? select_small<2>
                      : n <= kSelectSmallThreads * 4 ? select_small<4>
                                                     : select_small<kSelectSmallItems>;
  kernel<<<batch, kSelectSmallThreads, lds, st>>>(tail, score, score_bs, (int)n, base, idx, idx_bs, (uint32_t)k);
  ESA_LAUNCH_CHECK("select_small");
  return ESA_OK;
}

int launch_topk(const float* score, int64_t n, int k, int64_t base, int32_t* idx, int batch, int64_t score_bs,
                int64_t idx_bs, void* ws, size_t ws_bytes, hipStream_t st, bool first_hist_ready) {
  if (k >= n) {
    const int blocks = (int)((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024);
    topk_all<<<dim3(blocks, batch), 256, 0, st>>>(n, base, idx, idx_bs);
    ESA_LAUNCH_CHECK("topk_all");
    return ESA_OK;
  }
  if (n <= kSelectSmallMax) {
    ScoreTail whole = {score, score_bs, nullptr, 0, 0};
    return launch_select_small(whole, nullptr, 0, n, k, base, idx, idx_bs, batch, st);
  }
  const TopkPlan plan = topk_plan(n, batch);
  const int sub = (int)plan.sub, nblk = (int)plan.nblk;
  const int64_t row_words = topk_row_stride_words(n, batch);
  uint32_t* w = (uint32_t*)ws;
  const dim3 grid(nblk, batch);
  // otherwise the score call has zeroed the histograms and filled the first one
  if (!first_hist_ready) topk_init<<<dim3(3 * kHistReplicas, batch), 1024, 0, st>>>(w, row_words);
  const auto passes = sub == 1   ? launch_passes<1>
                      : sub == 2 ? launch_passes<2>
                      : sub == 3 ? launch_passes<3>
                      : sub == 4 ? launch_passes<4>
                      : sub == 5 ? launch_passes<5>
                      : sub == 6 ? launch_passes<6>
                      : sub == 7 ? launch_passes<7>
                                 : launch_passes<8>;
  passes(score, n, score_bs, w, row_words, grid, base, idx, idx_bs, (uint32_t)k, first_hist_ready, st);
  ESA_LAUNCH_CHECK("topk");
  return ESA_OK;
}

}  // namespace esa

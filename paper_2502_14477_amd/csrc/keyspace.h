// The virtual key sequence one ESA step attends over (Eq. 1):
//   [ I | M_k | L | C ]  =  cache rows [0, i_end) ++ selected rows [0, n_sel) ++ cache rows [l_start, t0 + l_c).
// M_k is read either from the gathered buffers or, through an index list, from the caches themselves.
// Current token c sees virtual keys [0, n_fixed + c], n_fixed = i_end + n_sel + (t0 - l_start).
#pragma once
#include "esa_common.h"

namespace esa {

struct KeySpace {
  const char* k_cache;
  const char* v_cache;
  const char* k_sel;
  const char* v_sel;
  const int32_t* sel_idx; // non-null: selected row j is cache row sel_idx[j] (no gathered buffers)
  int64_t tok_bytes;      // cache token stride in bytes
  int64_t sel_bytes;      // gathered-row stride in bytes
  int64_t i_end, n_sel, l_start;
};

// Address of virtual key j's row (all KV heads) in the key or value storage.
__device__ __forceinline__ const char* key_row(const KeySpace& ks, int64_t j, bool values) {
  if (j < ks.i_end) return (values ? ks.v_cache : ks.k_cache) + j * ks.tok_bytes;
  j -= ks.i_end;
  if (j < ks.n_sel) {
    if (ks.sel_idx) {
      int64_t row = ks.sel_idx[j];                       // a middle token: clamped so that a bad index cannot leave the cache
      row = row < 0 ? 0 : (row < ks.l_start ? row : ks.l_start - 1);
      return (values ? ks.v_cache : ks.k_cache) + row * ks.tok_bytes;
    }
    return (values ? ks.v_sel : ks.k_sel) + j * ks.sel_bytes;
  }
  j -= ks.n_sel;
  return (values ? ks.v_cache : ks.k_cache) + (ks.l_start + j) * ks.tok_bytes;
}

// What the workgroups of a launch of the tiled kernels attend to: a query tensor and a virtual key sequence.  A launch
// carries two views; the usual one uses view 0 only, the re-encoded attention of Section 3.2 gives the local keys
// (their own encoding of queries and keys, causal) to view 0 and the initial and selected keys (queries at the fixed
// position, every key visible) to view 1, so that both parts run in one launch.  Keys and values have strides of
// their own: the re-encoded local keys are a dense copy, their values stay in the caller's cache.
struct KeyView {
  const char* q;
  const char* k_cache;
  const char* v_cache;
  int64_t q_bs, k_bs_bytes, v_bs_bytes;   // batch strides (queries: elements)
  uint32_t k_bytes, v_bytes;              // row strides of the caches
  uint32_t i_end, n_sel, l_start;
  uint32_t n_fixed;                       // keys every row sees
  const int32_t* sel_idx;                 // not null: the n_sel selected rows are cache rows sel_idx[0..n_sel), not a gathered buffer
  int64_t idx_bs;                         // batch stride of the index list
  uint32_t idx_limit;                     // indices are clamped into [0, idx_limit)
  int with_chunk;                         // 1: the virtual sequence ends with the current chunk (causal); 0: every key is visible to every row
  // The split-key kernel's, whose views have slices of their own (beside the views, in arguments of their own, they cost each of its launches
  // 0.2 us: one token 8.06 -> 8.28 us); the matrix-core kernel lays its views' tiles end to end.
  int n_split;                            // slices of this view (view 0's slices come first)
  uint32_t split_step;                    // 2^32 / n_split, rounded up
  int slot0;                              // partial results of slice s go to slot slot0 + s
};

static inline uint32_t split_step(int n_split) {
  return n_split > 1 ? (uint32_t)((((uint64_t)1 << 32) + n_split - 1) / n_split) : 0u;
}
static inline void set_splits(KeyView* v, int n_split, int slot0) {
  v->n_split = n_split;
  v->split_step = split_step(n_split);
  v->slot0 = slot0;
}
// First of n_tiles tiles of slice s (s = n_split: behind the last): n_tiles s / n_split without a division, which as a 64-bit
// one was a third of the instructions in front of a kernel's first load.
__device__ __forceinline__ uint32_t slice_tile(uint32_t n_tiles, uint32_t s, int n_split, uint32_t step) {
  return s >= (uint32_t)n_split ? n_tiles : __umulhi(n_tiles, s * step);
}

// The grid of the tiled kernels: workgroups of one (batch entry, KV head) pair on one XCD (workgroup w runs on XCD w % 8) where
// the pairs are a multiple of eight, decoded without a division (what is left is that of a pair into entry and head).  x: 8 row tiles' worth of XCDs, or the row tiles; y: slices;
// z: pairs / 8, or the pairs.
struct PairGrid {
  int xcd_log2;                           // 3, or 0
  int pair0;                              // first pair of this launch
};
template <typename Launch>                // launch(grid, PairGrid)
static inline void for_pair_grids(int64_t pairs, int64_t row_tiles, int n_slices, Launch&& launch) {
  PairGrid g = {pairs % 8 == 0 ? 3 : 0, 0};
  const int64_t z = pairs >> g.xcd_log2;
  for (int64_t z0 = 0; z0 < z; z0 += 65535) {         // (65535: the most that a grid takes in z)
    g.pair0 = (int)(z0 << g.xcd_log2);
    launch(dim3((unsigned)(row_tiles << g.xcd_log2), (unsigned)n_slices, (unsigned)(z - z0 < 65535 ? z - z0 : 65535)), g);
  }
}
struct Placed {
  int pair, row_tile, slice;
};
__device__ __forceinline__ Placed place_in(const PairGrid& g) {
  return {g.pair0 + (int)((blockIdx.z << g.xcd_log2) | (blockIdx.x & ((1u << g.xcd_log2) - 1))), (int)(blockIdx.x >> g.xcd_log2), (int)blockIdx.y};
}

struct CacheRef {               // cache rows as a launch function gets them (strides in elements)
  const void *k, *v;
  int64_t k_stride, v_stride, k_bs, v_bs;
};
static inline KeyView make_view(const void* q, int64_t q_bs, const CacheRef& c, int64_t esz, int64_t i_end, int64_t n_sel,
                                int64_t l_start, int64_t n_fixed, int with_chunk, int n_split, int slot0,
                                const int32_t* sel_idx = nullptr, int64_t idx_bs = 0, int64_t idx_limit = 1) {
  KeyView v;
  v.q = (const char*)q;
  v.q_bs = q_bs;
  v.k_cache = (const char*)c.k;
  v.v_cache = (const char*)c.v;
  v.k_bs_bytes = c.k_bs * esz;
  v.v_bs_bytes = c.v_bs * esz;
  v.k_bytes = (uint32_t)(c.k_stride * esz);
  v.v_bytes = (uint32_t)(c.v_stride * esz);
  v.i_end = (uint32_t)i_end;
  v.n_sel = (uint32_t)n_sel;
  v.l_start = (uint32_t)l_start;
  v.n_fixed = (uint32_t)n_fixed;
  v.sel_idx = n_sel > 0 ? sel_idx : nullptr;
  v.idx_bs = idx_bs;
  v.idx_limit = (uint32_t)(idx_limit > 0 ? idx_limit : 1);
  v.with_chunk = with_chunk;
  set_splits(&v, n_split, slot0);
  return v;
}
// Field-wise select of the view a workgroup works on (not an indexed load): every kernel argument is then fetched in
// the first round trip.
__device__ __forceinline__ KeyView pick_view(const KeyView (&view)[2], bool second) {
  const KeyView &v0 = view[0], &v1 = view[1];
  KeyView V;
  V.q = second ? v1.q : v0.q;
  V.k_cache = second ? v1.k_cache : v0.k_cache;
  V.v_cache = second ? v1.v_cache : v0.v_cache;
  V.q_bs = second ? v1.q_bs : v0.q_bs;
  V.k_bs_bytes = second ? v1.k_bs_bytes : v0.k_bs_bytes;
  V.v_bs_bytes = second ? v1.v_bs_bytes : v0.v_bs_bytes;
  V.k_bytes = second ? v1.k_bytes : v0.k_bytes;
  V.v_bytes = second ? v1.v_bytes : v0.v_bytes;
  V.i_end = second ? v1.i_end : v0.i_end;
  V.n_sel = second ? v1.n_sel : v0.n_sel;
  V.l_start = second ? v1.l_start : v0.l_start;
  V.n_fixed = second ? v1.n_fixed : v0.n_fixed;
  V.sel_idx = second ? v1.sel_idx : v0.sel_idx;
  V.idx_bs = second ? v1.idx_bs : v0.idx_bs;
  V.idx_limit = second ? v1.idx_limit : v0.idx_limit;
  V.with_chunk = second ? v1.with_chunk : v0.with_chunk;
  V.n_split = second ? v1.n_split : v0.n_split;
  V.split_step = second ? v1.split_step : v0.split_step;
  V.slot0 = second ? v1.slot0 : v0.slot0;
  return V;
}

}  // namespace esa

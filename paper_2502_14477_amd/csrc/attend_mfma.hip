// Selected attention (Eq. 1) on the matrix cores: bf16 storage, head sizes 128 and 64.
//
// Work decomposition.  The query heads of one KV group share keys and values, so a workgroup
// owns up to 256 "rows" (128 where plan_one_call finds that quicker) = (up to 256/G consecutive current tokens) x (heads of one KV
// group), numbered token by token, and one slice of the virtual key sequence [I | M_k | L | C]; slices of one row tile
// are merged afterwards with the log-sum-exp rule of Algorithm 1 (esa_attend_merge).  The chunk's tokens are
// shared out evenly over the row tiles, in units of a wave's 32 rows, and a wave without rows, or whose rows see
// no key of a tile, leaves the tile's arithmetic out.  Eight waves of 32 rows each, two waves
// per SIMD, so that one wave's softmax arithmetic overlaps the other's matrix instructions; the
// kernel stays under 256 registers per lane for that.  Workgroups are numbered so that all
// workgroups of one (batch element, KV head) land on the same XCD and share its L2.
//
// Matrix-core formulation (v_mfma_f32_32x32x16_bf16, D[32x32] += A[32x16] B[16x32]; lane l feeds
// A row l%32 / B column l%32 with eight consecutive reduction elements chosen by l/32, and owns
// D[8*(v/4) + 4*(l/32) + v%4][l%32] in accumulator register v).  Both products are computed
// transposed so that a lane always stands for one query:
//     S^T [keys x queries] = K_tile [keys x d] . Q^T [d x queries]        A = K (LDS), B = Q (registers)
//     O^T [d x queries]   += V_tile^T [d x keys] . P^T [keys x queries]   A = V^T (LDS), B = P (registers)
// so the softmax over keys is an in-lane reduction over accumulator registers plus one exchange
// between the two half-waves, and S^T's accumulator layout is directly P^T's B-operand layout once
// the reduction slots of the second product are assigned to keys accordingly.
//
// Tiles of 64 keys stand three deep in LDS and arrive there without passing through registers:
// global_load_lds_dwordx4 deposits 16 bytes per lane at consecutive LDS addresses, so one wave
// instruction brings four 256-byte rows, and which 16 bytes of its row a lane fetches is chosen
// such that the rows land XOR-swizzled (K: 16-byte pieces by row % 16, V: 64-byte chunks by
// row % 4; with head size 64, where two rows share the 256 bytes that the banks cover, by the same bits of
// row / 2), which makes the fragment reads below free of bank conflicts without padding.  K
// fragments are plain 16-byte reads.  V stays row-major [key][dim]; its transposed fragments (eight
// keys of one head dimension per lane) come from ds_read_b64_tr_b16, which hands lane i of a 16-lane
// group element i%4 of the 8 bytes addressed by lanes 4e + i/4 (e = 0..3): sixteen lanes that point
// at a 4-key x 16-dim block receive one dimension each, four consecutive keys of it.
// One barrier per tile; the next two tiles' loads are in flight during the current tile's math, counted by hand.
//
// What bounds it: with all compute units busy the clock falls, on random operands further than on constant ones (a matrix
// instruction takes a SIMD 13.4 ns on one workgroup, 13.7 to 15.2 on 256 with constant operands, 18.9 to 20.0 with N(0,1)
// ones, that is 1.28 us for the 64 of a tile's two waves), so the loop's instructions count more than their order.  Time of a call against
// its number of tiles, merge included: 1.35 us a tile + 10 on 16 workgroups, 1.74 + 21.5 on 256 (512 tokens, 8 KV heads, 17 to 57
// tiles a slice); with a maximum taken from every tile and every row's address computed by every lane, 180 vector instructions a
// tile and wave where 130 stand now, 1.52 + 9.5 and 1.78 + 23 on the same card (1024 tokens with 8192 selected and 8192 local ones: 431 -> 410 us a
// step).  A tile takes 3250 cycles (2048 of them matrix instructions) at 1.8 GHz.  Steps of half a tile that carry the first product of
// the next half, the exponentials of their own and the second product of the last take 3050, but the clock falls to 1.7 GHz: the same time.
#include "attend_mfma.h"
#include "keyspace.h"

#include <float.h>
#include <stddef.h>
#include <type_traits>

namespace esa {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef short i16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
typedef __attribute__((address_space(3))) unsigned char lds_byte;

constexpr int kKT = 64;             // virtual keys per tile
constexpr int kRows = 256;          // query rows per workgroup
constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kMaxSlots = 32;           // partial results per row
constexpr int kMaxSplits = 16;          // slices of the key sequence, two-call form
constexpr int kMaxSelSplits = 8;        // two-call form: at most half as many local slices, then the selected ones
constexpr int kStages = 3;
constexpr int kMinLc = 16;          // shorter chunks go to the split-key kernel (attend_split.hip)
constexpr float kLog2e = 1.4426950408889634f;
// A lane's sixteen exponentials of half a tile add up to at most this, or the softmax reference moves to the running maximum: it lags
// by at most 2^8, harmless in bf16 and fp32, and the accumulators are rescaled in the first tiles of a slice and rarely after them.
constexpr float kMostSum = 256.f;
constexpr uint32_t kFollow = 2;
constexpr float kNoKey = -FLT_MAX;  // reference of a row that has seen no key: finite, so that differences stay numbers
constexpr float kLn2 = 0.6931471805599453f;

struct AttendArgs {
  KeyView view[2];
  bf16_t* out;
  float* lse;
  void* part_o;       // [batch][n_slot][l_c][h][D] partial outputs, un-normalised: fp16, scaled by 2^-E per row (D = 128), or fp32
  float* part_ml;     // [batch][n_slot][l_c][h][2]   softmax reference (log2 domain) + E, and sum * 2^-E (fp32 partials: E = 0)
  const char* k_sel;
  const char* v_sel;
  uint32_t sel_bytes;               // row stride of the gathered buffers
  int l_c, h, h_kv, group, group_log2;
  int qpt, n_qt;                    // tokens per row tile (a whole number of waves' rows, at most 256 rows), row tiles
  int batch;
  PairGrid grid;
  int n_split;        // slices of the launch's views, laid end to end
  uint32_t split_step;
  int slot0;          // slice s leaves its partial results in slot slot0 + s ...
  int n_slot;         // ... of so many per row
  uint32_t follow;    // tiles of a slice at whose end the softmax reference moves to the running maximum (head size 128)
  int to_slots;       // 1: write partial results even when the launch has a single slice
  int stream_slices;  // head size 64: slices leave non-temporally, as whole rows (see kStreamSlices)
  float c2;           // scale * log2(e)
  int64_t out_bs, sel_bs_bytes;
};

// Maximum / sum of a value over the two lanes 32 places apart: a lane swap in the vector unit.  (A general
// shuffle goes through the LDS crossbar, and the wait for it is a wait for every LDS read in flight.)
__device__ __forceinline__ float halves_max(float v) {
  const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));     // lower half's value, upper half's value
}
__device__ __forceinline__ float halves_sum(float v) {
  const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  f32x2 f = {lo, hi};
  bf16x2 b = __builtin_convertvector(f, bf16x2);
  return *(uint32_t*)&b;
}

__device__ __forceinline__ uint32_t pack_f16x2(float lo, float hi) {
  f16x2 h = {(_Float16)lo, (_Float16)hi};
  return *(uint32_t*)&h;
}

// Swizzles of the LDS tiles: the 16-byte slot of piece p of K row R is p ^ k_swizzle(R), the 64-byte slot of chunk c
// of V row R is c ^ v_swizzle(R).
template <int D> __device__ __forceinline__ uint32_t k_swizzle(uint32_t row) { return D == 128 ? row & 15 : (row >> 1) & 7; }
template <int D> __device__ __forceinline__ uint32_t v_swizzle(uint32_t row) { return D == 128 ? row & 3 : (row >> 1) & 1; }

// Head size 64 keeps what it computes in fp32: a probability goes into the second product as three bf16 terms, which
// together are its fp32 value, and the results of a slice are stored as they were accumulated.  (One term and fp16 slices,
// as for head size 128, put the outputs 2.3e-3 from the 64-bit result where rounding them to bf16 alone makes 1.66e-3; a
// step of 512 tokens at 32k takes 80 us for it, 63 with the narrow formats.)
template <int D> constexpr bool kFp32Probs = D == 64;
// Natural-log normaliser from a reference in the log2 domain and the sum of exponentials relative to it.  The fp32 form
// adds the logarithm in its own domain, one rounding of the sum instead of two.
template <int D> __device__ __forceinline__ float lse_of(float m, float l) {
  return kFp32Probs<D> ? __builtin_fmaf(m, kLn2, logf(l)) : (m + __builtin_amdgcn_logf(l)) * kLn2;
}

// View `part` of the kernel's arguments, read where they lie: by a select of every field, the loop over the views kept both in
// scalar registers, half of them spilled (1.3 us in front of the first load).
__device__ __forceinline__ KeyView view_argument(int part) {
  typedef __attribute__((address_space(4))) const KeyView argument;
  argument& v = ((argument*)((__attribute__((address_space(4))) const char*)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(AttendArgs, view)))[part];
  KeyView V;
  V.q = v.q;
  V.k_cache = v.k_cache;
  V.v_cache = v.v_cache;
  V.q_bs = v.q_bs;
  V.k_bs_bytes = v.k_bs_bytes;
  V.v_bs_bytes = v.v_bs_bytes;
  V.k_bytes = v.k_bytes;
  V.v_bytes = v.v_bytes;
  V.i_end = v.i_end;
  V.n_sel = v.n_sel;
  V.l_start = v.l_start;
  V.n_fixed = v.n_fixed;
  V.sel_idx = v.sel_idx;
  V.idx_bs = v.idx_bs;
  V.idx_limit = v.idx_limit;
  V.with_chunk = v.with_chunk;
  return V;
}

// LISTED: selected rows come from the cache, through an index list; otherwise from the gathered buffers.  Neither form pays for
// the other's rows (one kernel for both, with base and stride chosen per row: 285 us against 279 for 1024 queries with 8192
// gathered rows).
template <int D, bool LISTED>
__global__ __launch_bounds__(kThreads) void attend_mfma_bf16(AttendArgs a) {       // (the only argument: view_argument)
  static_assert(D == 64 || D == 128, "swizzles and store patterns");
  constexpr int kTileElems = kKT * D;     // one K or V tile in LDS: 64 unpadded rows, swizzled
  constexpr int kPieces = D / 8;          // 16-byte pieces of a row
  constexpr int kLoadRows = 64 / kPieces; // rows that one wave instruction brings
  constexpr int kMyRows = kKT / (kLoadRows * kWaves);   // rows of a tile that a lane fetches a piece of (2 or 1)
  constexpr int kRowStep = kLoadRows * kWaves;          // distance between them
  constexpr int kKS = D / 16;             // reduction steps of the first product
  constexpr int kMD = D / 32;             // 32-dim tiles of the second product
  // Three stages of a K tile, then three of a V tile, then room for the query rows, which come in through the last V stage and
  // what is behind it.  Two buffers of each wave's index entries, for eight tiles each.
  __shared__ __attribute__((aligned(1024))) bf16_t st[(2 * kStages + 3) * kTileElems];
  __shared__ __attribute__((aligned(1024))) int32_t idx_st[2][LISTED ? kWaves : 1][64];
  constexpr int kQPlace = (2 * kStages - 1) * kTileElems * 2;       // byte offset of the query rows

  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, hi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);        // uniform: scalar address arithmetic

  // ---- which (batch element, KV head, row tile, key slice) is this workgroup
  const Placed at = place_in(a.grid);
  const int b = at.pair / a.h_kv, g = at.pair - b * a.h_kv, qt = at.row_tile, split = at.slice;

  // ---- this workgroup's rows, and its slice of the tiles of both views
  const int q0 = qt * a.qpt;
  const int c_last = (q0 + a.qpt < a.l_c ? q0 + a.qpt : a.l_c) - 1;
  auto keys_of_last_row = [&](const KeyView& V) { return V.n_fixed + (V.with_chunk ? c_last + 1 : 0); };
  const uint32_t tiles_0 = (keys_of_last_row(a.view[0]) + kKT - 1) / kKT;
  const uint32_t tiles_all = tiles_0 + (keys_of_last_row(a.view[1]) + kKT - 1) / kKT;
  const uint32_t slice_begin = slice_tile(tiles_all, split, a.n_split, a.split_step);
  const uint32_t slice_end = slice_tile(tiles_all, split + 1, a.n_split, a.split_step);

  // ---- this wave's 32 rows (32/G consecutive current tokens, the group's heads of each), one per lane (both half-waves)
  const int row_in_tile = wave * 32 + r;
  const int head = g * a.group + (row_in_tile & (a.group - 1));
  const int c = q0 + (row_in_tile >> a.group_log2);
  const bool c_ok = c <= c_last;
  const int cc = c_ok ? c : c_last;                                // rows past the tile repeat its last token
  const bool wave_has_rows = q0 + ((wave * 32) >> a.group_log2) <= c_last;
  bf16x8 qf[kKS];

  f32x16 o[kMD];
#pragma unroll
  for (int md = 0; md < kMD; ++md)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[md][v] = 0.f;
  float m_run = kNoKey, l_run = 0.f;

  // ---- staging of one tile: global -> LDS directly, 16 bytes per lane.  A wave instruction fills 1 KB =
  // four rows of 256 bytes or eight of 128; wave w brings row groups w and (head size 128) w + 8 of K and of V.
  // Lane l fills one 16-byte slot of a row of its group; the piece of the global row it fetches for that slot undoes
  // the swizzle.
  const uint32_t st_row = kLoadRows * wave + lane / kPieces;       // first of this lane's rows (second: + 32)
  const uint32_t st_slot = lane % kPieces;
  const uint32_t kcol = (st_slot ^ k_swizzle<D>(st_row)) * 16;     // byte column of the piece fetched for K
  const uint32_t vcol = ((((st_slot >> 2) ^ v_swizzle<D>(st_row)) << 2) | (st_slot & 3)) * 16;   // ... for V
  const uint32_t st_lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_byte*)st) + wave * 1024;    // 1 KB per row group
  const uint32_t idx_lds = LISTED ? __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_byte*)idx_st) + wave * (kKT * 4) : 0u;
  // At most LEFT vector-memory operations of this wave are outstanding (they complete in order; the other counters are
  // left alone).
  auto loads_landed = [&](auto left_c) __attribute__((always_inline)) {
    constexpr int kLeft = decltype(left_c)::value;
    static_assert(kLeft < 16, "the counter's low bits");
    __builtin_amdgcn_s_waitcnt(0x0F70 | kLeft);
  };
  // A barrier without the fences of __syncthreads(), which wait for every load in flight.  The wave's LDS reads are
  // complete: their results have been used.
  auto all_waves = [&]() __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  // Lane constants of the transposed V reads: inside its 16-lane group lane i points at key i/4 of a
  // four-key block and at four consecutive dims 4*(i%4).. of the group's sixteen.
  const int tr_key = (lane & 15) >> 2;
  const int tr_dim = ((lane >> 4) & 1) * 16 + 4 * (lane & 3);

  // Byte offsets of the fragments in a stage; what comes on top, which stage and which keys, is constant and goes into the read
  // instruction.
  uint32_t k_at[kKS], v_at[kMD];
#pragma unroll
  for (int ks16 = 0; ks16 < kKS; ++ks16) k_at[ks16] = (r * D + (((2 * ks16 + hi) ^ k_swizzle<D>(r)) << 3)) * 2;
  // row key of the V tile holds chunk c (dims 32c .. 32c+31) at chunk slot c ^ v_swizzle(key), which keys 4 apart share
#pragma unroll
  for (int md = 0; md < kMD; ++md) v_at[md] = (kStages * kTileElems + (4 * hi + tr_key) * D + ((md ^ v_swizzle<D>(tr_key)) << 5) + tr_dim) * 2;
  // Keeps the compiler from folding a stage's place into the offsets outside the loop: twelve registers, not thirty-six.
  auto pin_offsets = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int ks16 = 0; ks16 < kKS; ++ks16) asm volatile("" : "+v"(k_at[ks16]));
#pragma unroll
    for (int md = 0; md < kMD; ++md) asm volatile("" : "+v"(v_at[md]));
  };

  // ---- the slice's tiles of one view after those of the other.  Sums and reference run on: a softmax does not mind in which
  // order, or with which encoding of the query, its logits were made.  (With slices of their own, Section 3.2's two parts were
  // three of 24 tiles and one of 34 where four of 26.5 are possible: 512 tokens behind a window of 4096.)
#pragma unroll 1
  for (int part = 0; part < 2; ++part) {
  const KeyView V = view_argument(part);
  const uint32_t before = part ? tiles_0 : 0, up_to = part ? tiles_all : tiles_0;
  if (slice_end <= before || slice_begin >= up_to) continue;
  const uint32_t tile_begin = (slice_begin > before ? slice_begin : before) - before;
  const uint32_t tile_end = (slice_end < up_to ? slice_end : up_to) - before;
  const uint32_t n_vis = keys_of_last_row(V);                      // keys the tile's last token sees
  const uint32_t k_end = tile_end * kKT < n_vis ? tile_end * kKT : n_vis;
  const char* kc = V.k_cache + (int64_t)b * V.k_bs_bytes + (int64_t)g * D * 2;
  const char* vc = V.v_cache + (int64_t)b * V.v_bs_bytes + (int64_t)g * D * 2;
  const char* ksl = a.k_sel + (V.n_sel ? (int64_t)b * a.sel_bs_bytes + (int64_t)g * D * 2 : 0);
  const char* vsl = a.v_sel + (V.n_sel ? (int64_t)b * a.sel_bs_bytes + (int64_t)g * D * 2 : 0);
  const uint32_t vis = V.n_fixed + (V.with_chunk ? cc + 1 : 0);
  const uint32_t lim = vis < k_end ? vis : k_end;                  // first virtual key this lane's query may NOT see
  const uint32_t lim_lo = __builtin_amdgcn_readlane(lim, 0);       // smallest limit in the wave (r = 0)
  const uint32_t lim_hi = wave_has_rows ? __builtin_amdgcn_readlane(lim, 31) : 0;      // largest; 0 for a wave without rows
  if (part && slice_begin < tiles_0) all_waves();                  // every wave is done with the other view's last tile
  // Loads into LDS are written out: the compiler, which cannot tell the stages apart, would put a wait for all of them in
  // front of every LDS read.  (They have no result registers that it could reuse under way.)  Every wave issues the same
  // number per turn and waits by count.
  // (The compiler warns that it does not keep m0's value across them: it has none there.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
  auto dma16 = [&](const char* src, uint32_t dst) __attribute__((always_inline)) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(dst), "v"(src) : "memory", "m0");
  };
  // The rows that this lane fetches pieces of, eight tiles at a time: the lanes of a row's group (sixteen of them with two rows each,
  // or eight with one) hold the offsets of one row of one tile each, and a tile's offsets are broadcast to the group when its turn
  // comes: 14 vector instructions a tile and wave, where every lane of a group finding every tile's rows took 40 (a chunk of 1024
  // with 8192 selected and 8192 local tokens: 1.04 of the step's time).
  // Index-driven selected rows (the gather folded into this kernel): the entries for eight tiles go to LDS eight tiles ahead.  A
  // list without entries: the cache's first word.
  const bool entries = LISTED && V.n_sel;
  const int32_t* list = entries ? V.sel_idx + (int64_t)b * V.idx_bs : (const int32_t*)kc;
  const uint32_t list_last = entries ? V.n_sel - 1 : 0;
  const uint32_t row_of_lane = st_row + kRowStep * (kMyRows == 2 ? lane & 1 : 0);
  const uint32_t key_of_lane = (tile_begin + (kMyRows == 2 ? (lane & 15) >> 1 : lane & 7)) * kKT + row_of_lane;
  auto idx_load = [&](uint32_t eight) __attribute__((always_inline)) {
    if constexpr (LISTED) {
      const int32_t js = (int32_t)(eight * (8 * kKT) + key_of_lane - V.i_end);
      const uint32_t at = js < 0 ? 0u : (uint32_t)js < list_last ? (uint32_t)js : list_last;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" : : "s"(idx_lds + (eight & 1) * (kWaves * 256)), "v"(list + at) : "memory", "m0");
    }
  };
#pragma clang diagnostic pop
  const uint32_t past_sel = V.l_start - V.i_end - V.n_sel;                // from a virtual key behind the selected ones to its row
  int64_t k_row = 0, v_row = 0;       // byte offsets from kc and vc (LISTED: the same)
  auto find_rows = [&](uint32_t eight) __attribute__((always_inline)) {
    uint32_t j = eight * (8 * kKT) + key_of_lane;
    j = j < k_end ? j : k_end - 1;                                        // the tail repeats a key; masked below
    if constexpr (LISTED) {
      // a middle token's position, clamped so that a bad index cannot leave the cache
      const int32_t entry = idx_st[eight & 1][wave][lane], most = (int32_t)V.idx_limit - 1;
      const uint32_t selected = entry < 0 ? 0 : entry < most ? entry : most;
      const uint32_t row = j - V.i_end < V.n_sel ? selected : j < V.i_end ? j : j + past_sel;
      k_row = (int64_t)((uint64_t)row * V.k_bytes);
    } else {
      const bool sel = j - V.i_end < V.n_sel;
      const uint64_t row = sel ? j - V.i_end : j < V.i_end ? j : j + past_sel;
      k_row = sel ? (ksl - kc) + (int64_t)(row * a.sel_bytes) : (int64_t)(row * V.k_bytes);
      v_row = sel ? (vsl - vc) + (int64_t)(row * a.sel_bytes) : (int64_t)(row * V.v_bytes);
    }
  };
  auto of_lane = [&](int64_t x, auto control) __attribute__((always_inline)) {       // every lane reads another of its sixteen
    constexpr int kControl = decltype(control)::value;
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, kControl, 0xF, 0xF, true);
    const uint32_t hi32 = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)((uint64_t)x >> 32), kControl, 0xF, 0xF, true);
    return (int64_t)((uint64_t)hi32 << 32 | lo);
  };
  auto of_group = [&](int64_t x, auto first) __attribute__((always_inline)) {        // row `first` of the group's next tile
    constexpr int kFirst = decltype(first)::value;
    if constexpr (kMyRows == 2) return of_lane(x, std::integral_constant<int, 0x150 + kFirst>());    // row_newbcast
    const int64_t low = of_lane(x, std::integral_constant<int, 0x150>()), up = of_lane(x, std::integral_constant<int, 0x158>());
    return lane & 8 ? up : low;
  };
  uint32_t fetched = 0;
  // the next tile, keys and values
  auto tile_load = [&](int stage) __attribute__((always_inline)) {
    const uint32_t k_dst = st_lds + stage * (kTileElems * 2), v_dst = k_dst + kStages * (kTileElems * 2);
    if ((fetched & 7) == 0) {
      find_rows(fetched >> 3);
      idx_load((fetched >> 3) + 1);
    }
    ++fetched;
    const int64_t k0 = of_group(k_row, std::integral_constant<int, 0>()), v0 = LISTED ? k0 : of_group(v_row, std::integral_constant<int, 0>());
    if constexpr (kMyRows == 2) {
      const int64_t k1 = of_group(k_row, std::integral_constant<int, 1>()), v1 = LISTED ? k1 : of_group(v_row, std::integral_constant<int, 1>());
      dma16(kc + kcol + k0, k_dst);
      dma16(kc + kcol + k1, k_dst + kWaves * 1024);
      dma16(vc + vcol + v0, v_dst);
      dma16(vc + vcol + v1, v_dst + kWaves * 1024);
    } else {
      dma16(kc + kcol + k0, k_dst);
      dma16(vc + vcol + v0, v_dst);
    }
    k_row = of_lane(k_row, std::integral_constant<int, 0x100 + kMyRows>());         // row_shl: the tile after it comes to the front
    if constexpr (!LISTED) v_row = of_lane(v_row, std::integral_constant<int, 0x100 + kMyRows>());
  };
  // ---- one tile: S^T = K Q^T, online softmax, O^T += V^T P^T, the probabilities in fp32 (head size 64)
  auto tile_math = [&](uint32_t t, int stage) __attribute__((always_inline)) {
    const uint32_t j0 = t * kKT;
    if (j0 >= lim_hi) return;           // no row of this wave sees any of the tile's keys
    f32x16 s[2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int v = 0; v < 16; ++v) s[mt][v] = 0.f;
    // The K fragments of the tile are requested half of them ahead of the matrix instructions that use
    // them (the order is pinned below): LDS latency is paid once per tile, not once per reduction step.
    bf16x8 kf[kKS][2];
#pragma unroll
    for (int ks16 = 0; ks16 < kKS; ++ks16)
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
        kf[ks16][mt] = *(const bf16x8*)((const char*)st + k_at[ks16] + (stage * kKT + 32 * mt) * D * 2);
#pragma unroll
    for (int ks16 = 0; ks16 < kKS; ++ks16)
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
        s[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks16][mt], qf[ks16], s[mt], 0, 0, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, kKS, 0);
#pragma unroll
    for (int i = 0; i < kKS / 2; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, kKS, 0);

    // ---- mask keys beyond each query's limit (causal diagonal, end of the slice)
    if (j0 + kKT > lim_lo) {
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const uint32_t j = j0 + 32 * mt + 8 * (v / 4) + 4 * hi + (v % 4);
          if (j >= lim) s[mt][v] = -INFINITY;
        }
    }

    // The V fragments of sixteen keys (two reads for each 32 dims) are requested two such groups ahead of their use.
    bf16x8 vf[4][kMD];
    auto request_values = [&](int kp, int md) __attribute__((always_inline)) {
      const char* vp = (const char*)st + v_at[md] + (stage * kKT + 16 * kp) * D * 2;
      const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)vp);                 // keys 16kp + 4hi + 0..3
      const i16x4 up = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(vp + 8 * D * 2));  // keys 16kp + 8 + 4hi + 0..3
      vf[kp][md] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, up, 0, 1, 2, 3, 4, 5, 6, 7));
    };
#pragma unroll
    for (int kp = 0; kp < 2; ++kp)
#pragma unroll
      for (int md = 0; md < kMD; ++md) request_values(kp, md);
    __builtin_amdgcn_sched_barrier(0);

    // ---- online softmax, one query per lane
    float mx = s[0][0];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int v = 0; v < 16; ++v) mx = fmaxf(mx, s[mt][v]);
    // The reference m_run of the exponentials follows the running maximum at once: the sum stays small, and its logarithm
    // as exact as the normaliser can hold.
    const float cand = halves_max(mx) * a.c2, m_old = m_run;
    const bool moved = cand > m_run;
    m_run = moved ? cand : m_run;
    float corr = 1.f;
    if (__ballot(moved) != 0ull) {
      corr = __builtin_amdgcn_exp2f(m_old - m_run);
#pragma unroll
      for (int md = 0; md < kMD; ++md)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[md][v] *= corr;
    }
    float psum = 0.f;
    // Accumulator register v = 8*(e/4) + e%4 (+ 4*hi in the key number): fragment kp of P^T is S^T's
    // registers 8*(kp%2) .. + 7 of key tile kp/2, i.e. keys 16*kp + 4*hi + {0..3} and 16*kp + 8 + 4*hi + {0..3}.
    constexpr int kTerms = kFp32Probs<D> ? 3 : 1;
    uint32_t pf[4][kTerms][4];
    // The eight keys of a lane in group kp, pair by pair in pieces: exponentials (E), then operands of the second product (O), in
    // the order E0 E1 O0 E2 O1 E3 O2 O3.
    auto piece = [&](int kp, int at) __attribute__((always_inline)) {
      const bool exps = at == 0 || at == 1 || at == 3 || at == 5;
      const int e = at < 2 ? at : at == 7 ? 3 : at / 2 + (exps ? 1 : -1);
      f32x16& sx = s[kp >> 1];
      const int v = (kp & 1) * 8 + 2 * e;
      if (exps) {
        sx[v] = __builtin_amdgcn_exp2f(__builtin_fmaf(sx[v], a.c2, -m_run));
        sx[v + 1] = __builtin_amdgcn_exp2f(__builtin_fmaf(sx[v + 1], a.c2, -m_run));
      } else {
        float x = sx[v], y = sx[v + 1];
        psum += x;
        psum += y;
#pragma unroll
        for (int term = 0; term < kTerms; ++term) {
          const uint32_t w = pack_bf16x2(x, y);
          pf[kp][term][e] = w;
          if (term + 1 < kTerms) {          // what the term leaves, exactly
            x -= __uint_as_float(w << 16);
            y -= __uint_as_float(w & 0xFFFF0000u);
          }
        }
      }
    };
#pragma unroll
    for (int at = 0; at < 8; ++at) piece(0, at);
    __builtin_amdgcn_sched_barrier(0);

    // ---- O^T += V^T P^T, sixteen keys at a time; beside each matrix instruction a share of the next sixteen's exponentials and
    // of the fragment reads for the sixteen after them.  (The order is pinned: left to itself, or with groups of instruction
    // kinds to follow, the scheduler puts the fragment reads next to their use: 1.57 to 1.81 us a tile.)
    constexpr int kMat = kTerms * kMD;
#pragma unroll
    for (int kp = 0; kp < 4; ++kp)
#pragma unroll
      for (int j = 0; j < kMat; ++j) {
        const int term = j / kMD, md = j % kMD;
        const uint4 w = make_uint4(pf[kp][term][0], pf[kp][term][1], pf[kp][term][2], pf[kp][term][3]);
        o[md] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[kp][md], *(const bf16x8*)&w, o[md], 0, 0, 0);
        if (kp + 2 < 4 && j < kMD) request_values(kp + 2, j);
#pragma unroll
        for (int at = 0; at < 8; ++at)
          if (kp + 1 < 4 && at * kMat / 8 == j) piece(kp + 1, at);
        __builtin_amdgcn_sched_barrier(0);
      }
    l_run = __builtin_fmaf(l_run, corr, psum);          // rounded once
  };

  // ---- the same with probabilities in one bf16 term (head size 128), in two halves of 32 keys, so that the exponentials of one half
  // stand beside the matrix instructions of the other.  No maximum is looked for: the exponentials are taken against the
  // reference as it is, and where a lane's sum over a half exceeds kMostSum (infinite where the row has no reference yet) the half is
  // done again against its maximum, with what has been summed so far rescaled.  (The 27 instructions of the maximum stood between
  // the products, where nothing hid them: 1.53 -> 1.48 us a tile on 16 workgroups.)
  auto half_tiles = [&](uint32_t t, int stage, auto&& loads) __attribute__((always_inline)) {
    const uint32_t j0 = t * kKT;
    const char* kt = (const char*)st + stage * kKT * D * 2;
    bf16x8 kf[2][kKS];
    auto request_keys = [&](int mt, int ks16) __attribute__((always_inline)) {
      kf[mt][ks16] = *(const bf16x8*)(kt + k_at[ks16] + 32 * mt * D * 2);
    };
#pragma unroll
    for (int ks16 = 0; ks16 < kKS; ++ks16) request_keys(0, ks16);
    __builtin_amdgcn_sched_barrier(0);
    loads();
    if (j0 >= lim_hi) return;           // no row of this wave sees any of the tile's keys
    f32x16 s[2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int v = 0; v < 16; ++v) s[mt][v] = 0.f;
    bf16x8 vf[4][kMD];
    auto request_values = [&](int kp, int md) __attribute__((always_inline)) {
      const char* vp = (const char*)st + v_at[md] + (stage * kKT + 16 * kp) * D * 2;
      const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)vp);
      const i16x4 up = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(vp + 8 * D * 2));
      vf[kp][md] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, up, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    auto mask = [&](int mt) __attribute__((always_inline)) {
      if (j0 + 32 * mt + 32 > lim_lo) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (j0 + 32 * mt + 8 * (v / 4) + 4 * hi + (v % 4) >= lim) s[mt][v] = -INFINITY;
      }
    };
    float psum[2] = {0.f, 0.f};
    uint32_t pf[4][4];
    float p[2][16];
    auto piece = [&](int mt, int at) __attribute__((always_inline)) {    // at: 0 .. 15
      const int kp = at / 8, a8 = at % 8;
      const bool exps = a8 == 0 || a8 == 1 || a8 == 3 || a8 == 5;
      const int e = a8 < 2 ? a8 : a8 == 7 ? 3 : a8 / 2 + (exps ? 1 : -1);
      const int v = kp * 8 + 2 * e;
      if (exps) {
        p[mt][v] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[mt][v], a.c2, -m_run));
        p[mt][v + 1] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[mt][v + 1], a.c2, -m_run));
      } else {
        psum[mt] += p[mt][v];
        psum[mt] += p[mt][v + 1];
        pf[2 * mt + kp][e] = pack_bf16x2(p[mt][v], p[mt][v + 1]);
      }
    };
    // (A sum that is no number does not exceed it: the row's output is none either way.)  In the first tiles, two of a slice or `follow` of
    // them, the reference moves to the largest logit in any case: the keys that it has stood at have exact probabilities, and a slice's largest of
    // 128 keys weighs more than its largest of 32.  Distance from the 64-bit result, mean over eleven calls of 20 to 700 tokens, four
    // seeds: 2.295e-3, 2.330 without (2.308 with the maximum of every tile and up to sixteen slices); steps 0 to 1.5 % longer.
    auto settle = [&](int mt) __attribute__((always_inline)) {
      if (__builtin_expect(__ballot(psum[mt] > kMostSum) != 0ull || (mt == 1 && t < tile_begin + a.follow), 0)) {
        float mx = s[mt][0];
#pragma unroll
        for (int v = 0; v < 16; ++v) mx = fmaxf(mx, s[mt][v]);
        const float m_old = m_run;
        m_run = fmaxf(m_run, halves_max(mx) * a.c2);
        const float corr = __builtin_amdgcn_exp2f(m_old - m_run);
        if (mt || t != tile_begin || part) {              // (nothing has been summed yet)
#pragma unroll
          for (int md = 0; md < kMD; ++md)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[md][v] *= corr;
        }
        l_run *= corr;
        if (mt) psum[0] *= corr;
        psum[mt] = 0.f;
#pragma unroll
        for (int at = 0; at < 16; ++at) piece(mt, at);
      }
    };
    auto second = [&](int kp, int md) __attribute__((always_inline)) {
      const uint4 w = make_uint4(pf[kp][0], pf[kp][1], pf[kp][2], pf[kp][3]);
      o[md] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[kp][md], *(const bf16x8*)&w, o[md], 0, 0, 0);
    };
    // (The order is pinned: left to itself the scheduler puts the fragment reads next to their use.)
    // keys 0 ... 31: first product
#pragma unroll
    for (int i = 0; i < kKS; ++i) {
      s[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0][i], qf[i], s[0], 0, 0, 0);
      request_keys(1, i);
      __builtin_amdgcn_sched_barrier(0);
    }
    mask(0);
    // keys 32 ... 63; beside it the exponentials of the first half
#pragma unroll
    for (int i = 0; i < kKS; ++i) {
      s[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[1][i], qf[i], s[1], 0, 0, 0);
      request_values(i / kMD, i % kMD);
#pragma unroll
      for (int at = 0; at < 16; ++at)
        if (1 + at * (kKS - 1) / 16 == i) piece(0, at);
      __builtin_amdgcn_sched_barrier(0);
    }
    settle(0);
    mask(1);
    // second product of the first half; beside it the exponentials of the second
#pragma unroll
    for (int i = 0; i < 2 * kMD; ++i) {
      second(i / kMD, i % kMD);
      request_values(2 + i / kMD, i % kMD);
#pragma unroll
      for (int at = 0; at < 16; ++at)
        if (1 + at * (2 * kMD - 1) / 16 == i) piece(1, at);
      __builtin_amdgcn_sched_barrier(0);
    }
    settle(1);
#pragma unroll
    for (int i = 0; i < 2 * kMD; ++i) {
      second(2 + i / kMD, i % kMD);
      __builtin_amdgcn_sched_barrier(0);
    }
    l_run += psum[0] + psum[1];
  };

  // Turn t: tile t, requested two turns before (a turn takes 2 us, a tile that comes from HBM sometimes longer).  Its own requests
  // are tile t + 2 and, every eighth turn, index entries; tile n is in stage (n - tile_begin) % 3.  At its barrier every wave is
  // done with the stage that these overwrite.
  idx_load(0);
  // The wave's 32 query rows, through LDS like a K tile: whole rows, four or eight to an instruction.  (Fetched as
  // fragments, 16 bytes of 32 rows to an instruction, they were 32 cache lines each.)
  constexpr int kQLoads = 32 / kLoadRows;
  uint32_t lane_now = lane;                      // hidden from the compiler: the rows' addresses would be kept across both views' loops
  asm volatile("" : "+v"(lane_now));
#pragma unroll
  for (int i = 0; i < kQLoads; ++i) {
    const uint32_t qr = kLoadRows * i + lane_now / kPieces, in_tile = wave * 32 + qr;
    const int qc = q0 + (int)(in_tile >> a.group_log2);
    const int64_t at = (int64_t)b * V.q_bs + ((int64_t)(qc < c_last ? qc : c_last) * a.h + g * a.group + (in_tile & (a.group - 1))) * D;
    dma16(V.q + (at + ((lane_now % kPieces) ^ k_swizzle<D>(qr)) * 8) * 2, st_lds - wave * 1024 + kQPlace + wave * (32 * D * 2) + 1024 * i);
  }
  if constexpr (LISTED) loads_landed(std::integral_constant<int, kQLoads>());
  tile_load(0);
  tile_load(1);
  loads_landed(std::integral_constant<int, 4 * kMyRows>());
#pragma unroll
  for (int ks16 = 0; ks16 < kKS; ++ks16) qf[ks16] = *(const bf16x8*)((const char*)st + kQPlace + wave * (32 * D * 2) + k_at[ks16]);
  // arrived before the barrier of the first turn, behind which other waves overwrite the rows
#pragma unroll
  for (int ks16 = 0; ks16 < kKS; ++ks16) asm volatile("" : "+v"(qf[ks16]));
  auto turn = [&](uint32_t t, int s0, int s2) __attribute__((always_inline)) {        // stages of tiles t and t + 2
    loads_landed(std::integral_constant<int, 2 * kMyRows>());
    all_waves();
    if constexpr (kFp32Probs<D>) {
      tile_load(s2);
      pin_offsets();
      tile_math(t, s0);
    } else {
      pin_offsets();
      half_tiles(t, s0, [&]() __attribute__((always_inline)) { tile_load(s2); });
    }
  };
  for (uint32_t t = tile_begin; t < tile_end; t += 3) {
    turn(t, 0, 2);
    if (t + 1 < tile_end) {
      turn(t + 1, 1, 0);
      if (t + 2 < tile_end) turn(t + 2, 2, 1);
    }
  }
  loads_landed(std::integral_constant<int, 0>());
  }

  // ---- results.  Accumulator register v of tile md is head-dim 32*md + 8*(v/4) + 4*hi + v%4 of this
  // lane's query, so a lane holds its whole output row in 8-byte pieces.  The rows are narrowed to 16
  // bits and turned into whole rows in LDS (free by now), from where each wave writes its own
  // 32 rows with fully coalesced 16-byte stores.  Final outputs are normalised and rounded to bf16.
  // Partial results of a key slice stay un-normalised and are stored as fp16 with a per-row power-of-two
  // scale 2^-E that brings the row's largest magnitude to about 2^13 (fp16's 11-bit significand keeps the
  // rounding well below that of the bf16 output, and any magnitude bf16 inputs can produce fits); beside
  // them go m + E and l * 2^-E, so that the merge's sums of 2^(m+E-M) * (O 2^-E) and 2^(m+E-M) * (l 2^-E)
  // are the plain log-sum-exp combination of Algorithm 1 with no trace of E.  Head size 64 stores its slices in fp32: many bytes as whole
  // rows too and non-temporally, few as each lane holds them.
  const float l_tot = halves_sum(l_run);
  const bool final_out = a.n_split == 1 && !a.to_slots;
  float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  float m_store = m_run, l_store = l_tot;
  if constexpr (kFp32Probs<D>) {
    if (!final_out) {
      const int64_t prow0 = ((int64_t)(b * a.n_slot + a.slot0 + split) * a.l_c) * a.h;
      if (hi == 0 && c_ok) *(float2*)(a.part_ml + (prow0 + (int64_t)c * a.h + head) * 2) = make_float2(m_run, l_tot);
      if (!a.stream_slices) {
        if (c_ok) {
          float* dst = (float*)a.part_o + (prow0 + (int64_t)c * a.h + head) * D + 4 * hi;
#pragma unroll
          for (int md = 0; md < kMD; ++md)
#pragma unroll
            for (int vg = 0; vg < 4; ++vg) {
              const f32x4 w = {o[md][4 * vg], o[md][4 * vg + 1], o[md][4 * vg + 2], o[md][4 * vg + 3]};
              *(f32x4*)(dst + 32 * md + 8 * vg) = w;
            }
        }
        return;
      }
      __syncthreads();                   // every wave is done with the last tile
      float* mine = (float*)st + wave * 32 * D;
#pragma unroll
      for (int md = 0; md < kMD; ++md)
#pragma unroll
        for (int vg = 0; vg < 4; ++vg) {
          const f32x4 w = {o[md][4 * vg], o[md][4 * vg + 1], o[md][4 * vg + 2], o[md][4 * vg + 3]};
          *(f32x4*)(mine + r * D + (((8 * md + 2 * vg + hi) ^ (r & 15)) << 2)) = w;      // 16-byte slots swizzled
        }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int rw = 4 * i + lane / 16, piece = lane % 16;
        const int row = wave * 32 + rw, tok = q0 + (row >> a.group_log2), hd = g * a.group + (row & (a.group - 1));
        if (tok <= c_last)
          __builtin_nontemporal_store(*(const f32x4*)(mine + rw * D + ((piece ^ (rw & 15)) << 2)),
                                      (f32x4*)((float*)a.part_o + (prow0 + (int64_t)tok * a.h + hd) * D + piece * 4));
      }
      return;
    }
  }
  if (!final_out) {
    float amax = 0.f;
#pragma unroll
    for (int md = 0; md < kMD; ++md)
#pragma unroll
      for (int v = 0; v < 16; ++v) amax = fmaxf(amax, __builtin_fabsf(o[md][v]));
    amax = halves_max(amax);
    int s_exp = 267 - (int)((__float_as_uint(amax) >> 23) & 0xFFu);      // biased exponent of 2^-E
    s_exp = s_exp < 17 ? 17 : (s_exp > 167 ? 167 : s_exp);              // 2^-110 .. 2^40
    inv = __uint_as_float((uint32_t)s_exp << 23);
    m_store = m_run - (float)(s_exp - 127);
    l_store = l_tot * inv;
  }
  __syncthreads();                       // every wave is done with the last tile
  {
    // 16-byte slots swizzled as in a K tile
    uint16_t* ot = (uint16_t*)st + (wave * 32 + r) * D;
#pragma unroll
    for (int md = 0; md < kMD; ++md)
#pragma unroll
      for (int vg = 0; vg < 4; ++vg) {
        uint2 w;
        if (final_out) {
          w.x = pack_bf16x2(o[md][4 * vg + 0] * inv, o[md][4 * vg + 1] * inv);
          w.y = pack_bf16x2(o[md][4 * vg + 2] * inv, o[md][4 * vg + 3] * inv);
        } else {
          w.x = pack_f16x2(o[md][4 * vg + 0] * inv, o[md][4 * vg + 1] * inv);
          w.y = pack_f16x2(o[md][4 * vg + 2] * inv, o[md][4 * vg + 3] * inv);
        }
        *(uint2*)(ot + (((4 * md + vg) ^ k_swizzle<D>(r)) << 3) + 4 * hi) = w;
      }
  }
  __syncthreads();
  uint16_t* dst;
  if (final_out) {
    dst = (uint16_t*)a.out + (int64_t)b * a.out_bs;
  } else {
    const int64_t prow0 = ((int64_t)(b * a.n_slot + a.slot0 + split) * a.l_c) * a.h;
    dst = (uint16_t*)a.part_o + prow0 * D;
    if (hi == 0 && c_ok) {
      float2 ml = {m_store, l_store};
      *(float2*)(a.part_ml + (prow0 + (int64_t)c * a.h + head) * 2) = ml;
    }
  }
#pragma unroll
  for (int i = 0; i < kPieces / 2; ++i) {
    const int rw = kLoadRows * i + lane / kPieces, piece = lane % kPieces;
    const int row = wave * 32 + rw, tok = q0 + (row >> a.group_log2), hd = g * a.group + (row & (a.group - 1));
    if (tok <= c_last) {
      const uint4 w = *(const uint4*)((const uint16_t*)st + (wave * 32 + rw) * D + ((piece ^ k_swizzle<D>(rw)) << 3));
      *(uint4*)(dst + ((int64_t)tok * a.h + hd) * D + piece * 8) = w;
    }
  }
  if (final_out && a.lse && hi == 0 && c_ok)
    a.lse[(int64_t)b * a.l_c * a.h + (int64_t)c * a.h + head] = lse_of<D>(m_run, l_tot);
}

// Algorithm 1's merge over partial results (un-normalised outputs and sums, both relative to the slice's
// reference m_s): weights 2^(m_s - M) with the maximum subtracted first.
// The slots in use are [0, ns_a) and [slot_b, slot_b + ns_b) of n_slot.  Sixteen lanes per row (16 bytes of partials
// each: eight head-dims in fp16, four in fp32), sixteen rows per workgroup.
// NS: slots in use, a constant: with a run-time number every slot's loads stood behind a branch, which made each a round
// trip of its own, and vector instructions were issued for sixteen slots whatever their number (1.2 % of a step with
// four slices, 16.9 MB of partials for 512 tokens).
template <int D, int NS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, NS > 16 ? 2 : NS > 8 ? 4 : 8)))   // registers for all loads
void esa_attend_merge(const void* __restrict__ part_o, const float* __restrict__ part_ml, int n_slot, int ns_a,
                      int slot_b, int64_t rows, bf16_t* __restrict__ out, float* __restrict__ lse, int64_t out_bs,
                      int64_t lse_bs) {
  constexpr int kPer = kFp32Probs<D> ? 4 : 8;     // head-dims of a lane
  constexpr int kLanes = D / kPer;
  const int64_t row = (int64_t)blockIdx.x * (256 / kLanes) + threadIdx.x / kLanes;
  const int dim = (threadIdx.x % kLanes) * kPer;
  const int b = blockIdx.y;
  if (row >= rows) return;
  // Every load of the row goes out before the first use (one round trip): the slices' (maximum, sum)
  // pairs and their outputs.  A slice that saw no key of this row stored zeros and sum 0.
  float2 ml[NS];
  uint4 po[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    const int64_t prow = ((int64_t)b * n_slot + (i < ns_a ? i : slot_b + i - ns_a)) * rows + row;
    ml[i] = *(const float2*)(part_ml + prow * 2);
    po[i] = *(const uint4*)((const char*)part_o + (prow * D + dim) * (16 / kPer));
  }
  float M = kNoKey;
#pragma unroll
  for (int i = 0; i < NS; ++i) M = fmaxf(M, ml[i].x);
  float L = 0.f;
  float acc[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) acc[i] = 0.f;
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    const float w = __builtin_amdgcn_exp2f(ml[i].x - M);
    const uint32_t u[4] = {po[i].x, po[i].y, po[i].z, po[i].w};
    L += w * ml[i].y;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (kFp32Probs<D>) {
        acc[e] += w * __uint_as_float(u[e]);
      } else {
        const f16x2 p = *(const f16x2*)&u[e];
        acc[2 * e] += w * (float)p[0];
        acc[2 * e + 1] += w * (float)p[1];
      }
    }
  }
  const float inv = 1.f / L;
  uint32_t w[kPer / 2];
#pragma unroll
  for (int e = 0; e < kPer / 2; ++e) w[e] = pack_bf16x2(acc[2 * e] * inv, acc[2 * e + 1] * inv);
  bf16_t* dst = out + (int64_t)b * out_bs + row * D + dim;
  if constexpr (kPer == 8) *(uint4*)dst = make_uint4(w[0], w[1], w[2], w[3]);
  else *(uint2*)dst = make_uint2(w[0], w[1]);
  if (lse && dim == 0) lse[(int64_t)b * lse_bs + row] = lse_of<D>(M, L);
}

// Row tiles: as few as hold the chunk at most_rows rows each, the tokens shared out evenly in units of a wave's 32 rows.
struct RowTiles {
  int n_qt, qpt;
};
RowTiles row_tiles(int l_c, int group, int most_rows = kRows) {
  const int most = most_rows / group, unit = 32 / group;
  RowTiles t;
  t.n_qt = (l_c + most - 1) / most;
  t.qpt = ((l_c + t.n_qt - 1) / t.n_qt + unit - 1) / unit * unit;
  return t;
}

int choose_splits(int l_c, int group, int h_kv, int batch) {
  const int64_t tiles = (int64_t)row_tiles(l_c, group).n_qt * h_kv * batch;
  const int64_t ns = (256 + tiles - 1) / tiles;
  return (int)(ns < 1 ? 1 : (ns > kMaxSplits ? kMaxSplits : ns));
}

// ---- one-call form: row tiles of 256 or of 128 rows, and the number of slices.  A compute unit holds one workgroup, so a workgroup
// more than 256 costs another round of them (160 tokens of eight KV heads in eleven slices of three row tiles, 264 workgroups: 38.5 us a
// call, 23.6 as chosen here), and a number far below leaves compute units idle.  With 128 rows a SIMD has one wave instead of
// two, which takes 0.6 of the time a tile.  A merge of more than sixteen slots has few rows and waits for its loads; a slice that
// holds the end of Section 3.2's first part and the start of its second has the queries to fetch again, about a tile's time.
// The constants of the cost are a fit to 375 calls, every number of slices of each (17 to 1000 tokens; 32 heads of 8, 16 of 2 and 8 of 8;
// head sizes 128 and 64; 3 to 16 thousand keys; one to four sequences; one view and two): the plan takes 1.004 of the best one's time
// in the mean, 1.065 at most.  (Fitted on one view of one sequence of eight KV heads, without the second part's start: 1.016 and 1.13.)
// Calls, us, with 256 rows and 256 / tiles slices rounded up, at most sixteen (and the kernel of whole tiles), and as chosen here: 4 thousand
// keys of eight KV heads, 17 tokens 14.9 / 14.4, 48 19.7 / 16.5, 77 21.8 / 18.7, 128 25.1 / 22.2, 200 28.8 / 28.5, 300 50.4 / 34.2, 384
// 55.5 / 39.3, 512 48.1 / 46.8, 700 95.5 / 68.5; 16 thousand, 17 27.4 / 21.6, 77 38.3 / 34.8, 300 137 / 84.7, 700 305 / 190; three sequences of 4
// thousand, 48 36.5 / 23.6, 256 93.5 / 68.8; Section 3.2, 6 thousand, 48 33.1 / 29.9, 200 44.3 / 44.9, 300 73.5 / 52.4.
// Slices that a launch over this many (row tile, pair)s may have: one round of workgroups where that fills nine tenths of the compute
// units, three otherwise.  (Known without the number of keys, so that the workspace is.)
int most_slices(int64_t base) {
  const int64_t one = 256 / base, ns = one * base >= 230 ? one : 768 / base;
  return (int)(ns < 1 ? 1 : ns > kMaxSlots ? kMaxSlots : ns);
}
struct Plan {
  RowTiles rows;
  int n_split;
  uint32_t follow;
};
// keys: in front of the chunk's own; second_keys: of Section 3.2's second part, -1 where there is one view only.
Plan plan_one_call(int l_c, int h, int h_kv, int batch, int64_t keys, int64_t second_keys) {
  const int group = h / h_kv;
  auto tiles_of = [](int64_t n) { return (uint32_t)((n + kKT - 1) / kKT); };
  const uint32_t second = second_keys > 0 ? tiles_of(second_keys) : 0;
  const uint32_t tiles = tiles_of(keys + l_c) + second, first = tiles_of(keys + 1) + second;
  Plan best = {row_tiles(l_c, group), 1, kFollow};
  float least = FLT_MAX;
  for (int most_rows = kRows; most_rows >= kRows / 2; most_rows /= 2) {
    const RowTiles r = row_tiles(l_c, group, most_rows);
    const int64_t base = (int64_t)r.n_qt * h_kv * batch;
    const bool one_wave = r.qpt * group <= kRows / 2;                    // a SIMD's waves with rows
    const uint32_t most = (uint32_t)most_slices(base) < first ? most_slices(base) : first;
    // The longest slice, of the first row tile or the last.
    auto longest = [&](uint32_t ns) {
      uint32_t most_tiles = 0;
      for (int64_t seen : {keys + (r.qpt < l_c ? r.qpt : l_c), keys + l_c}) {
        const uint32_t end = tiles_of(seen), all = end + second;
        uint32_t n = (all + ns - 1) / ns;
        if (second) {
          const uint32_t s = ((end + 1) * ns - 1) / all, lo = all * s / ns, hi = all * (s + 1) / ns;     // the slice of the second part's first tile
          if (lo < end && hi - lo + 1 > n) n = hi - lo + 1;
        }
        most_tiles = n > most_tiles ? n : most_tiles;
      }
      return most_tiles;
    };
    for (uint32_t ns = 1;;) {
      const float n = (float)longest(ns);
      float t = (float)((base * ns + 255) / 256) * (one_wave ? 0.8f + 1.f * n : 2.f + 1.4f * n);
      if (ns > 1) t += 4.f + 9.8e-5f * (float)l_c * h * batch * ns + (ns > 16 ? 0.08f * (ns - 16) : 0.f);
      if (one_wave && second_keys >= 0) t *= 1.05f;
      if (t < least) {
        least = t;
        best = {r, (int)ns, kFollow};
      }
      if (ns >= most) break;
      ns += ns < 16 ? 1 : 4;
      ns = ns < most ? ns : most;
    }
  }
  // Every slice has its own reference, so a row has the fewer exact probabilities the fewer slices it is cut into.  Where they are fewer than
  // one round of workgroups of 256 rows would take, the reference follows the maximum for more tiles, the same number in all.  Distance from
  // the 64-bit result, 1e-3, with that many slices, with fewer and two tiles, and so: 300 tokens of 16 heads of two 2.290 / 2.308 / 2.276, 128 tokens of 32 heads of eight
  // 2.294 / 2.305 / 2.283, 512 of eight of eight 2.299 / 2.311 / 2.291; none of 80 calls of 17 to 1024 tokens is further from it than with that
  // many slices.  The calls concerned take 1 to 3 % longer.
  const int round = choose_splits(l_c, group, h_kv, batch), whole = (uint32_t)round < tiles ? round : (int)tiles;
  if (best.n_split < whole) best.follow = (uint32_t)(kFollow * whole + best.n_split / 2) / best.n_split;
  return best;
}

// Head size 64: bytes of a launch's slices (256 a row) from which on they leave as whole rows and non-temporally.  As each lane holds them / so, us: 0.8 MB
// (17 tokens, 8 heads) 9.5 / 11.0, 2.1 (17, 32) 11.1 / 12.2, 3.1 (100, 8) 11.7 / 12.3, 3.9 (64, 16) 12.46 / 12.40, 4.6 (40, 32) 14.69 / 14.69, 5.2 (2 x 40, 32)
// 19.3 / 18.6, 5.7 (400, 8) 18.0 / 16.7, 6.3 (64, 16) 14.25 / 14.26, 6.6 (100, 32) 17.0 / 15.6, 13.1 (200, 32) 29.3 / 27.3, 16.8 (512, 32) 50.1 / 47.5.  Whole
// rows by ordinary stores take what a lane's own pieces take, or 0.5 more.  (The fp16 slices of head size 128, 16.8 MB: 45.8 / 45.7, a step 0.994 to 1.006.)
constexpr int64_t kStreamSlices = 5000000;

void launch_tiles(AttendArgs& a, int d, int n_split, int slot0, hipStream_t st) {
  a.n_split = n_split;
  a.stream_slices = (int64_t)n_split * a.batch * a.l_c * a.h * 256 >= kStreamSlices;
  a.split_step = split_step(n_split);
  a.slot0 = slot0;
  for_pair_grids((int64_t)a.batch * a.h_kv, a.n_qt, n_split, [&](dim3 grid, PairGrid placed) {
    a.grid = placed;
    const auto kernel = a.view[0].sel_idx ? (d == 128 ? attend_mfma_bf16<128, true> : attend_mfma_bf16<64, true>)
                                          : (d == 128 ? attend_mfma_bf16<128, false> : attend_mfma_bf16<64, false>);
    kernel<<<grid, kThreads, 0, st>>>(a);
  });
}

template <int D, int NS = 1>
void launch_merge(const AttendArgs& a, int ns_a, int slot_b, int ns_b, hipStream_t st) {
  if (ns_a + ns_b != NS) {                       // 1 ... kMaxSlots slots in all
    if constexpr (NS < kMaxSlots) launch_merge<D, NS + 1>(a, ns_a, slot_b, ns_b, st);
    return;
  }
  const int64_t rows = (int64_t)a.l_c * a.h;
  constexpr int kRowsPerWg = 256 / (D / (kFp32Probs<D> ? 4 : 8));
  esa_attend_merge<D, NS><<<dim3((unsigned)((rows + kRowsPerWg - 1) / kRowsPerWg), a.batch), 256, 0, st>>>(
      a.part_o, a.part_ml, a.n_slot, ns_a, slot_b, rows, a.out, a.lse, a.out_bs, rows);
}

}  // namespace

bool attend_mfma_supported(int l_c, int h, int h_kv, int d, int dtype) {
  if (dtype != ESA_BF16 || (d != 128 && d != 64) || l_c < kMinLc || h % h_kv != 0) return false;
  const int group = h / h_kv;
  return group == 1 || group == 2 || group == 4 || group == 8;
}

namespace {

// Planned slice counts of the two-call form: the local part [ I | L | C ] runs beside other work, so it gets fewer, longer slices than
// the selected part, which is on the critical path and should cover the chip by itself.
struct SplitPlan {
  int local, sel;
};
SplitPlan plan_splits(int l_c, int group, int h_kv, int batch) {
  SplitPlan p;
  const int all = choose_splits(l_c, group, h_kv, batch);
  p.sel = all < kMaxSelSplits ? all : kMaxSelSplits;
  p.local = p.sel > 1 ? p.sel / 2 : 1;
  return p;
}

size_t part_o_bytes(size_t rows, int d) { return align_up(rows * d * (d == 64 ? sizeof(float) : sizeof(uint16_t)), 256); }
size_t slots_bytes(int64_t slots, int h, int d) {          // slots: of a token's h rows
  const size_t rows = (size_t)slots * h;
  return part_o_bytes(rows, d) + align_up(rows * 2 * sizeof(float), 256);
}

}  // namespace

// Covers every shorter chunk (of kMinLc tokens or more) and fewer sequences too, so that a workspace for the longest chunk serves the last one: more than one
// slice are at most 768 workgroups (most_slices; the two-call form's slots are at most one and a half times ceil(256 / base)) of
// at most kRows rows, and at most kMaxSlots of them; one slice of the two-call form's parts each are two slots.
size_t attend_mfma_workspace_bytes(int l_c, int h, int h_kv, int d, int batch) {
  const int64_t tokens = (int64_t)l_c * batch, round = (int64_t)768 * kRows / h, all = tokens * kMaxSlots;
  const int64_t split = round < all ? round : all;
  return slots_bytes(split > 2 * tokens ? split : 2 * tokens, h, d);
}

namespace {

int clamp_splits(int ns, int64_t keys_of_first_tile) {
  const int64_t tiles = (keys_of_first_tile + kKT - 1) / kKT;
  return (int)(ns > tiles ? (tiles > 0 ? tiles : 1) : ns);
}

}  // namespace

int launch_attend_mfma(int part, int split, const void* q, int l_c, int h, int h_kv, int d, const void* k_cache,
                       const void* v_cache, int64_t tok_stride, int64_t t0, int64_t i_end, int64_t l_start,
                       const void* k_sel, const void* v_sel, int n_sel, const int32_t* sel_idx, int64_t idx_bs,
                       float scale, void* out, float* lse, int batch, int64_t q_bs, int64_t cache_bs, int64_t sel_bs,
                       int64_t out_bs, void* ws, size_t ws_bytes, hipStream_t st) {
  if (!(scale > 0.f)) ESA_FAIL(ESA_EINVAL, "esa_attend: scale must be positive");
  if (t0 + l_c >= ((int64_t)1 << 31) || tok_stride * 2 >= ((int64_t)1 << 32))
    ESA_FAIL(ESA_EUNSUPPORTED, "esa_attend: positions beyond 2^31 are not supported by the matrix-core kernel");
  AttendArgs a;
  a.out = (bf16_t*)out;
  a.lse = lse;
  a.k_sel = (const char*)k_sel;
  a.v_sel = (const char*)v_sel;
  a.sel_bytes = (uint32_t)((int64_t)h_kv * d * 2);
  a.l_c = l_c;
  a.h = h;
  a.h_kv = h_kv;
  a.group = h / h_kv;
  a.group_log2 = __builtin_ctz(a.group);
  const int64_t n_fixed = i_end + n_sel + (t0 - l_start);
  const Plan one = part == kAttendAll ? plan_one_call(l_c, h, h_kv, batch, n_fixed, -1) : Plan{row_tiles(l_c, a.group), 0, kFollow};
  const RowTiles tiles = one.rows;
  a.follow = one.follow;
  a.qpt = tiles.qpt;
  a.n_qt = tiles.n_qt;
  a.batch = batch;
  a.c2 = scale * kLog2e;
  a.out_bs = out_bs;
  a.sel_bs_bytes = sel_bs * 2;

  const SplitPlan plan = plan_splits(l_c, a.group, h_kv, batch);
  const int first_rows = l_c < a.qpt ? l_c : a.qpt;
  // slices in use: one call -> ns_all; two calls -> local in slots [0, ns_local), selected in [plan.local, +ns_sel)
  const int ns_all = one.n_split;
  // split == ESA_SPLIT_ALGORITHM1 moves the initial tokens from the early part to the late one
  const int64_t i_early = split == ESA_SPLIT_ALGORITHM1 ? 0 : i_end, i_late = i_end - i_early;
  const int ns_local = clamp_splits(plan.local, i_early + (t0 - l_start) + first_rows);
  const int ns_sel = i_late + n_sel > 0 ? clamp_splits(plan.sel, i_late + n_sel) : 0;
  const int n_slot = part == kAttendAll ? ns_all : plan.local + plan.sel;

  a.part_o = nullptr;
  a.part_ml = nullptr;
  if (part != kAttendAll || ns_all > 1) {
    const size_t need = slots_bytes((int64_t)batch * n_slot * l_c, h, d);
    if (!ws || ws_bytes < need) ESA_FAIL(ESA_EWORKSPACE, "esa_attend: workspace needs %zu bytes", need);
    const size_t rows = (size_t)batch * n_slot * l_c * h;
    a.part_o = ws;
    a.part_ml = (float*)((char*)ws + part_o_bytes(rows, d));
  }
  a.n_slot = n_slot;
  const CacheRef cache = {k_cache, v_cache, tok_stride, tok_stride, cache_bs, cache_bs};
  a.view[1] = make_view(q, q_bs, cache, 2, 0, 0, 0, 0, 0, 0, 0);   // unused
  auto launch = [&](int n_split, int slot0) { launch_tiles(a, d, n_split, slot0, st); };
  auto merge = [&](int ns_a, int slot_b, int ns_b) {
    if (d == 128) launch_merge<128>(a, ns_a, slot_b, ns_b, st);
    else launch_merge<64>(a, ns_a, slot_b, ns_b, st);
  };
  if (part == kAttendAll) {
    a.view[0] = make_view(q, q_bs, cache, 2, i_end, n_sel, l_start, i_end + n_sel + (t0 - l_start), 1, 0, 0, sel_idx, idx_bs,
                          l_start);
    a.to_slots = 0;
    launch(ns_all, 0);
    if (ns_all > 1) merge(ns_all, 0, 0);
  } else if (part == kAttendLocal) {
    a.view[0] = make_view(q, q_bs, cache, 2, i_early, 0, l_start, i_early + (t0 - l_start), 1, 0, 0);
    a.to_slots = 1;
    launch(ns_local, 0);
  } else {
    if (ns_sel > 0) {
      a.view[0] = make_view(q, q_bs, cache, 2, i_late, n_sel, 0, i_late + n_sel, 0, 0, 0, sel_idx, idx_bs, l_start);
      a.to_slots = 1;
      launch(ns_sel, plan.local);
    }
    merge(ns_local, plan.local, ns_sel);
  }
  ESA_LAUNCH_CHECK("attend_mfma");
  return ESA_OK;
}

// Section 3.2 in one launch: the local keys (dense re-encoded copy, rows [0, n_loc + l_c), causal; their values where
// they are in the caller's cache) with the queries q_loc, and the initial and selected keys (caller's un-encoded cache
// and gathered rows, every key visible) with the queries q_glob; the slices of both share the launch and the merge.
int launch_attend_mfma_two_views(const void* q_loc, const void* q_glob, int64_t qw_bs, int l_c, int h, int h_kv, int d,
                                 const CacheRef& local, int64_t n_loc, const CacheRef& cache, int64_t i_end,
                                 const void* k_sel, const void* v_sel, int n_sel, int64_t sel_bs, float scale, void* out,
                                 float* lse, int batch, int64_t out_bs, void* ws, size_t ws_bytes, hipStream_t st) {
  if (!(scale > 0.f)) ESA_FAIL(ESA_EINVAL, "esa_attend: scale must be positive");
  if (n_loc + l_c >= ((int64_t)1 << 31) || cache.k_stride * 2 >= ((int64_t)1 << 32))
    ESA_FAIL(ESA_EUNSUPPORTED, "esa_attend: positions beyond 2^31 are not supported by the matrix-core kernel");
  AttendArgs a;
  a.out = (bf16_t*)out;
  a.lse = lse;
  a.k_sel = (const char*)k_sel;
  a.v_sel = (const char*)v_sel;
  a.sel_bytes = (uint32_t)((int64_t)h_kv * d * 2);
  a.l_c = l_c;
  a.h = h;
  a.h_kv = h_kv;
  a.group = h / h_kv;
  a.group_log2 = __builtin_ctz(a.group);
  // slices of the two parts' tiles laid end to end
  const int64_t keys_b = i_end + n_sel;
  const Plan plan = plan_one_call(l_c, h, h_kv, batch, n_loc, keys_b);
  a.qpt = plan.rows.qpt;
  a.n_qt = plan.rows.n_qt;
  a.follow = plan.follow;
  a.batch = batch;
  a.c2 = scale * kLog2e;
  a.out_bs = out_bs;
  a.sel_bs_bytes = sel_bs * 2;
  const int n_slot = plan.n_split;
  const size_t need = slots_bytes((int64_t)batch * n_slot * l_c, h, d);
  a.part_o = nullptr;
  a.part_ml = nullptr;
  if (n_slot > 1) {
    if (!ws || ws_bytes < need) ESA_FAIL(ESA_EWORKSPACE, "esa_attend: workspace needs %zu bytes", need);
    const size_t rows = (size_t)batch * n_slot * l_c * h;
    a.part_o = ws;
    a.part_ml = (float*)((char*)ws + part_o_bytes(rows, d));
  }
  a.n_slot = n_slot;
  a.to_slots = 0;
  a.view[0] = make_view(q_loc, qw_bs, local, 2, 0, 0, 0, n_loc, 1, 0, 0);
  a.view[1] = make_view(q_glob, qw_bs, cache, 2, i_end, n_sel, 0, keys_b, 0, 0, 0);
  launch_tiles(a, d, n_slot, 0, st);
  if (n_slot > 1) {
    if (d == 128) launch_merge<128>(a, n_slot, 0, 0, st);
    else launch_merge<64>(a, n_slot, 0, 0, st);
  }
  ESA_LAUNCH_CHECK("attend_mfma (two views)");
  return ESA_OK;
}

}  // namespace esa

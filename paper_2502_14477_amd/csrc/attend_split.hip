// Selected attention (Eq. 1) with the key sequence split over waves: bf16 storage with fewer than 16 current tokens
// (decode, drafts; head sizes 64 and 128) and fp32 storage (any chunk; head sizes 32, 64 and 128).
//
// A decode step reads every attended key and value once (17 MB per sequence at the Llama shape) for a few hundred
// floating-point operations per byte less than the matrix cores need, so what counts is that many independent
// requests are in flight and that the current tokens share them.  A workgroup owns 32 "rows" = (current tokens x query
// heads of one KV head, numbered token by token) and a slice of the virtual key sequence [I | M_k | L | C]; its four or five
// waves take the slice's 32-key tiles in turn, each with staging space of its own, so that no barrier stands in the
// tile loop: a wave waits for its own keys, and while its values are still arriving requests the next tile's keys.
// The waves' results meet in LDS, the slices' in a second small kernel (Algorithm 1's log-sum-exp rule).
// (One token at a time through vector arithmetic, five drafted tokens read every key five times: 53 us for four
// sequences of 4229 keys, 69 MB.)
//
// Matrix-core formulation as in attend_mfma.hip: S^T = K Q^T, O^T += V^T P^T, a lane stands for one row; the layout of
// S^T's accumulator is the second product's operand layout.  bf16: v_mfma_f32_32x32x16_bf16; fp32:
// v_mfma_f32_32x32x2_f32, exact fp32 products and sums, four of which consume the same 16 bytes of a key row that one
// bf16 instruction does, so that staging and fragment reads are the same for both.
#include "attend_split.h"

#include <type_traits>

namespace esa {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) double f64x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef short i16x8 __attribute__((ext_vector_type(8)));

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) unsigned char lds_byte;
typedef __attribute__((address_space(1))) const void global_void;

constexpr int kKT = 32;             // keys per tile
constexpr int kRows = 32;           // rows per workgroup
constexpr int kWavesOfTwo = 4;      // waves of a workgroup of which a compute unit holds two ...
constexpr int kWavesOfOne = 5;      // ... and of one that has it to itself (see waves_of)
constexpr int kMaxSplits = 64;
constexpr int kTargetWorkgroups = 512;   // two per compute unit: 64 KB of staging each at 256-byte rows
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Exponentials of the softmax: base 2 on the hardware instruction for bf16 storage, full-precision base e for fp32.
template <typename T> __device__ __forceinline__ float exp_of(float x) { return __builtin_amdgcn_exp2f(x); }
template <> __device__ __forceinline__ float exp_of<float>(float x) { return expf(x); }
// (the normaliser of the base-2 form adds the logarithm in its own domain: one rounding of the sum instead of two)
template <typename T> __device__ __forceinline__ float lse_of(float m, float l) { return __builtin_fmaf(m, kLn2, logf(l)); }
template <> __device__ __forceinline__ float lse_of<float>(float m, float l) { return m + logf(l); }

__device__ __forceinline__ float halves_max(float v) {
  const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
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

struct SplitArgs {
  KeyView view[2];
  void* out;
  float* lse;
  float* part_o;      // [batch][l_c][h][n_slot][D] un-normalised
  float* part_ml;     // [batch][l_c][h][n_slot][2]  largest logit (base 2 for bf16), sum of exponentials relative to it
  const char* k_sel;
  const char* v_sel;
  uint32_t sel_bytes;
  int l_c, h, h_kv, n_rt;             // n_rt: row tiles of a KV head
  int group, group_log2;              // query heads of a KV head, their logarithm (-1: no power of two)
  int n_slot, to_slots;
  PairGrid grid;
  float scale;                        // includes log2(e) for bf16
  int64_t out_bs, sel_bs_bytes;
  const double* turns;                // TURNED
};

// Wait until at most N vector-memory operations are outstanding (the other counters are left alone).  The builtin, not
// an instruction written out: the compiler takes it into account where it places waits of its own.
template <int N> __device__ __forceinline__ void wait_loads() {
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Fragment reads of the tile loop are instructions written out, each group followed by its own wait: an LDS read that the
// compiler generates while loads into LDS are outstanding is preceded by a wait for all of these (it does not tell which
// of them fill what it reads), which would put a tile's round trip in front of the previous tile's arithmetic.  LDS
// operations complete in order: "at most N outstanding" means everything but the N newest has arrived.
__device__ __forceinline__ u32x4 lds_read16(uint32_t at) {
  u32x4 x;
  asm volatile("ds_read_b128 %0, %1" : "=v"(x) : "v"(at));
  return x;
}
template <int OFF> __device__ __forceinline__ i16x4 lds_read_tr(uint32_t at) {
  i16x4 x;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(x) : "v"(at), "n"(OFF));
  return x;
}
__device__ __forceinline__ float lds_read4(uint32_t at) {
  float x;
  asm volatile("ds_read_b32 %0, %1" : "=v"(x) : "v"(at));
  return x;
}
template <int N, typename X> __device__ __forceinline__ void arrived4(X& a, X& b, X& c, X& d) {
  asm volatile("s_waitcnt lgkmcnt(%c4)" : "+v"(a), "+v"(b), "+v"(c), "+v"(d) : "n"(N));
}

__device__ __forceinline__ void lds_write4(uint32_t at, uint32_t x) { asm volatile("ds_write_b32 %0, %1" : : "v"(at), "v"(x)); }

// TURNED: the first view's keys are un-encoded.  When a tile of them has arrived its wave turns it where it lies in LDS, key j by j
// positions, in fp64 and rounded once: the keys are then those that esa_rope writes.  A lane has two neighbouring pairs of D / 8
// consecutive keys (half a tile, a quarter with head size 64): it takes their first turn from the table, and the next key's from the
// last two (cos(a + x) = 2 cos x cos a - cos(a - x)), whose error grows to some 2^-46 over sixteen keys.
// Where a tile's turns begin in the table, which starts with the turn by one position.
constexpr int kTurnBytes = 2048;                   // of a tile: 256 / D rows of D / 2 pairs of fp64 cosine and sine
constexpr uint64_t turn_offset(uint32_t tile, int d) { return 8u * d + (uint64_t)tile * kTurnBytes; }
static_assert(turn_offset((1u << 31) / kKT, 128) == 1024 + (((1ull << 31) / kKT) << 11), "the last tile of the longest window, beyond 32 bits");

// (A re-encoded copy of the local keys is a read, a write and another read of them, 67 MB more for eight sequences behind a window of
// 2048: step at 64 thousand tokens 129.4 us copied, 121.2 turned here.  What turning costs is 25 vector instructions a pair, 0.8 us a tile
// and SIMD with the SIMDs busy, 1.5 us of a call that has a tile a wave.  In fp32, by products of two turns in registers, it cost
// half of that (117.1), but put an element of every hundredth key on the other side of its rounding.)
// STREAM: keys and values are fetched non-temporally (see streams).
template <typename T, int D, int kWaves, bool TURNED = false, bool STREAM = false>
__global__ __launch_bounds__(64 * kWaves, D * sizeof(T) > 256 || kWaves > kWavesOfTwo ? 1 : 2) __attribute__((amdgpu_waves_per_eu(D * sizeof(T) > 256 ? 1 : 2)))
void attend_split(SplitArgs a) {
  static_assert(!TURNED || sizeof(T) == 2, "the table's order");
  constexpr bool kBf16 = sizeof(T) == 2;
  constexpr int kRowBytes = D * (int)sizeof(T);
  constexpr int kPieces = kRowBytes / 16;          // 16-byte pieces of a row
  constexpr int kLoadRows = 64 / kPieces;          // rows that one load instruction of the wave brings
  constexpr int kLoads = kKT / kLoadRows;          // load instructions of a tile (keys or values)
  constexpr int kKS = kPieces / 2;                 // fragment reads of the first product
  constexpr int kMD = D / 32;                      // 32-dim tiles of the second product
  constexpr int kTileBytes = kKT * kRowBytes;
  __shared__ __attribute__((aligned(1024))) unsigned char k_st[kWaves][kTileBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char v_st[kWaves][kTileBytes];
  __shared__ __attribute__((aligned(8))) float ml[kWaves][kRows][2];
  __shared__ __attribute__((aligned(1024))) unsigned char turn_st[TURNED ? kWaves : 1][TURNED ? kTurnBytes : 1];

  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, hi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // ---- which (batch element, KV head, row tile, slice)
  const int n_slices = a.view[0].n_split + a.view[1].n_split;
  const Placed at = place_in(a.grid);
  const int b = at.pair / a.h_kv, g = at.pair - b * a.h_kv, rt = at.row_tile, slice = at.slice;
  const bool second = slice >= a.view[0].n_split;
  const KeyView V = pick_view(a.view, second);
  const int split = slice - (second ? a.view[0].n_split : 0);
  const char* kc = V.k_cache + (int64_t)b * V.k_bs_bytes + (int64_t)g * kRowBytes;
  const char* vc = V.v_cache + (int64_t)b * V.v_bs_bytes + (int64_t)g * kRowBytes;
  const bool gathered = V.n_sel && (TURNED || !V.sel_idx);      // (Section 3.2's selected rows are always gathered ones)
  const char* ksl = a.k_sel + (gathered ? (int64_t)b * a.sel_bs_bytes + (int64_t)g * kRowBytes : 0);
  const char* vsl = a.v_sel + (gathered ? (int64_t)b * a.sel_bs_bytes + (int64_t)g * kRowBytes : 0);
  const int32_t* sidx = !TURNED && V.sel_idx ? V.sel_idx + (int64_t)b * V.idx_bs : nullptr;

  // ---- rows: one per lane (both half-waves)
  const int n_rows = a.l_c * a.group;
  const int row = rt * kRows + r, rr = row < n_rows ? row : n_rows - 1;     // rows past the end repeat the last one
  const int c = a.group_log2 >= 0 ? rr >> a.group_log2 : rr / a.group, head = g * a.group + rr - c * a.group;
  const int row_last = rt * kRows + kRows - 1 < n_rows ? rt * kRows + kRows - 1 : n_rows - 1;
  const uint32_t n_vis = V.n_fixed + (V.with_chunk ? (a.group_log2 >= 0 ? row_last >> a.group_log2 : row_last / a.group) + 1 : 0);     // keys the tile's last row sees
  const uint32_t n_tiles = (n_vis + kKT - 1) / kKT;
  const uint32_t tile_begin = slice_tile(n_tiles, split, V.n_split, V.split_step);
  const uint32_t tile_end = slice_tile(n_tiles, split + 1, V.n_split, V.split_step);
  const uint32_t k_end = tile_end * kKT < n_vis ? tile_end * kKT : n_vis;
  const uint32_t vis = V.n_fixed + (V.with_chunk ? c + 1 : 0);
  const uint32_t lim = vis < k_end ? vis : k_end;                           // first virtual key this lane's row may NOT see
  const uint32_t lim_lo = __builtin_amdgcn_readlane(lim, 0);

  // ---- staging.  A wave instruction deposits 1 KB of LDS at consecutive addresses, lane by lane: kLoadRows rows.
  // Which 16 bytes of its row a lane fetches is chosen such that the rows land swizzled (keys: 16-byte pieces by the
  // row's number, or half of it where two rows share the 256 bytes that the banks cover; bf16 values: 64-byte chunks).
  const uint32_t st_row = lane / kPieces, st_slot = lane % kPieces;
  auto k_swizzle = [](uint32_t key) -> uint32_t { return kRowBytes >= 256 ? key & 15 : (key >> 1) & 7; };
  auto v_swizzle = [](uint32_t key) -> uint32_t { return !kBf16 ? 0 : kRowBytes >= 256 ? key & 3 : (key >> 1) & 1; };
  // Lane l stands for key l%32 of a tile.  Its entry of the index list is requested (lookup) a tile ahead of its use
  // (place_of): the number of its cache row, or the complement of its number among the gathered rows.
  auto virtual_key = [&](uint32_t t) {
    const uint32_t j = t * kKT + r;
    return j < k_end ? j : k_end - 1;                                       // the tail repeats a key; masked below
  };
  auto lookup = [&](uint32_t t) -> int32_t {
    if (!sidx) return 0;
    const uint32_t js = virtual_key(t) - V.i_end;
    return sidx[js < V.n_sel ? js : 0];
  };
  auto place_of = [&](uint32_t t, int32_t v) -> int32_t {
    const uint32_t j = virtual_key(t), js = j - V.i_end;
    if (j >= V.i_end && js < V.n_sel) {
      if (!sidx) return ~(int32_t)js;
      return v < 0 ? 0 : ((uint32_t)v < V.idx_limit ? v : (int32_t)V.idx_limit - 1);   // clamped so that a bad index cannot leave the cache
    }
    return (int32_t)(j < V.i_end ? j : js - V.n_sel + V.l_start);
  };
  // The places of the rows this lane fetches a piece of, from the lanes that stand for their keys.
  auto spread = [&](int32_t place, int32_t (&mine)[kLoads]) {
#pragma unroll
    for (int i = 0; i < kLoads; ++i) mine[i] = __shfl(place, kLoadRows * i + (int)st_row, 64);
    __builtin_amdgcn_sched_barrier(0);
  };
  constexpr int kTurnLoads = TURNED ? kTurnBytes / 1024 : 0;
  auto load_turn = [&](uint32_t tile) {            // the second view's tiles have none of their own and take the first
    if constexpr (TURNED) {
      const char* src = (const char*)a.turns + turn_offset(second ? 0 : tile, D) + lane * 16;
#pragma unroll
      for (int i = 0; i < kTurnLoads; ++i)
        __builtin_amdgcn_global_load_lds((global_void*)(src + i * 1024), (lds_void*)(turn_st[wave] + i * 1024), 16, 0, 0);
    }
  };
  auto load_tile = [&](const int32_t (&mine)[kLoads], bool values) {
    unsigned char* dst = values ? v_st[wave] : k_st[wave];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const uint32_t key = kLoadRows * i + st_row;
      const int32_t p = mine[i];
      const uint32_t piece = values ? ((((st_slot >> 2) ^ v_swizzle(key)) << 2) | (st_slot & 3)) : st_slot ^ k_swizzle(key);
      const char* src = p < 0 ? (values ? vsl : ksl) + (uint64_t)(uint32_t)~p * a.sel_bytes
                              : (values ? vc : kc) + (uint64_t)(uint32_t)p * (values ? V.v_bytes : V.k_bytes);
      __builtin_amdgcn_global_load_lds((global_void*)(src + piece * 16), (lds_void*)(dst + i * 1024), 16, 0, STREAM ? kNonTemporal : 0);
    }
  };

  // Requested in the order of need: the first tile's places, the row's query fragments (piece 2 ks + hi), the tile.
  uint32_t t = tile_begin + wave;
  const bool has_tile = t < tile_end;
  int32_t next = 0;                                                         // index entry of the wave's next tile
  int32_t mine[kLoads];
  u32x4 qf[kKS];
  double step[TURNED ? 4 : 1];                     // cosine and sine of the lane's two pairs' turn by one position
  if (has_tile) {
    const int32_t first = lookup(t);
    const char* qp = V.q + ((int64_t)b * V.q_bs + ((int64_t)c * a.h + head) * D) * (int64_t)sizeof(T) + hi * 16;
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) qf[ks] = *(const u32x4*)(qp + ks * 32);
    if (t + kWaves < tile_end) next = lookup(t + kWaves);
    if constexpr (TURNED) {
#pragma unroll
      for (int i = 0; i < 4; ++i) step[i] = a.turns[lane % (D / 4) * 4 + i];
    }
    __builtin_amdgcn_sched_barrier(0);
    spread(place_of(t, first), mine);
    load_turn(t);
    load_tile(mine, false);
    load_tile(mine, true);
    if constexpr (TURNED) {                        // (a use that the compiler saw first in the loop it would put behind all loads)
      wait_loads<kTurnLoads + 2 * kLoads>();
#pragma unroll
      for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(step[i]));
    }
  }
  f32x16 o[kMD];
#pragma unroll
  for (int md = 0; md < kMD; ++md)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[md][v] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  if (has_tile) {
    const uint32_t k_at = (uint32_t)(uintptr_t)(lds_byte*)k_st[wave] + r * kRowBytes + ((hi ^ k_swizzle(r)) << 4);
    uint32_t v_at[kMD];
    {
      const int tr_key = (lane & 15) >> 2, tr_dim = ((lane >> 4) & 1) * 16 + 4 * (lane & 3);   // transposed reads: see attend_mfma.hip
      const uint32_t v0 = (uint32_t)(uintptr_t)(lds_byte*)v_st[wave];
#pragma unroll
      for (int md = 0; md < kMD; ++md)
        v_at[md] = kBf16 ? v0 + ((4 * hi + tr_key) * D + ((md ^ v_swizzle(tr_key)) << 5) + tr_dim) * 2
                         : v0 + 4 * hi * kRowBytes + (32 * md + r) * 4;
    }
    auto turn_keys = [&]() __attribute__((always_inline)) {
      constexpr int kMine = D / 8;                                          // keys of a lane
      const uint32_t block = lane / (D / 4), dword = lane % (D / 4);
      const uint32_t first = (uint32_t)(uintptr_t)(lds_byte*)k_st[wave] + block * (kMine * kRowBytes) +
                             (((dword >> 2) ^ (D == 64 ? (block & 1) << 2 : 0)) << 4) + (dword & 3) * 4;
      auto place = [&](uint32_t key) { return (first ^ ((D == 128 ? key : key >> 1) << 4)) + key * kRowBytes; };   // upper half: ^ D
      const uint32_t turn_at = (uint32_t)(uintptr_t)(lds_byte*)turn_st[wave] + lane * 32;
      u32x4 turn[2];
      asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %2 offset:16\n\ts_waitcnt lgkmcnt(0)" : "=&v"(turn[0]), "=&v"(turn[1]) : "v"(turn_at));
      double c[2], sn[2], c_before[2], sn_before[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        c[e] = __builtin_bit_cast(f64x2, turn[e])[0];
        sn[e] = __builtin_bit_cast(f64x2, turn[e])[1];
        c_before[e] = c[e] * step[2 * e] + sn[e] * step[2 * e + 1];
        sn_before[e] = sn[e] * step[2 * e] - c[e] * step[2 * e + 1];
      }
      // Four keys a turn of a loop: a copy of its code for every key would be cold for longer than it takes.
#pragma unroll 1
      for (uint32_t key = 0; key < kMine; key += 4) {
        uint32_t at[4], x[4], y[4];                                         // the keys' lower and upper halves
#pragma unroll
        for (int k = 0; k < 4; ++k) at[k] = place(key + k);
        asm volatile("ds_read_b32 %0, %8\n\tds_read_b32 %4, %12\n\tds_read_b32 %1, %9\n\tds_read_b32 %5, %13\n\t"
                     "ds_read_b32 %2, %10\n\tds_read_b32 %6, %14\n\tds_read_b32 %3, %11\n\tds_read_b32 %7, %15\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(y[0]), "=&v"(y[1]), "=&v"(y[2]), "=&v"(y[3])
                     : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "v"(at[0] ^ D), "v"(at[1] ^ D), "v"(at[2] ^ D), "v"(at[3] ^ D));
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          double turned[4];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const double av = __uint_as_float(e ? x[k] & 0xFFFF0000u : x[k] << 16), bv = __uint_as_float(e ? y[k] & 0xFFFF0000u : y[k] << 16);
            turned[e] = av * c[e] - bv * sn[e];
            turned[2 + e] = bv * c[e] + av * sn[e];
            const double twice = 2.0 * step[2 * e], c_next = twice * c[e] - c_before[e], sn_next = twice * sn[e] - sn_before[e];
            c_before[e] = c[e];
            sn_before[e] = sn[e];
            c[e] = c_next;
            sn[e] = sn_next;
          }
          float f[4];
          narrow_for_bf16(turned, f);
          lds_write4(at[k], pack_bf16x2(f[0], f[1]));
          lds_write4(at[k] ^ D, pack_bf16x2(f[2], f[3]));
        }
      }
    };
    for (; t < tile_end; t += kWaves) {
      const bool more = t + kWaves < tile_end;
      const uint32_t j0 = t * kKT;
      wait_loads<kLoads>();                                                 // the keys; the values may still be on their way
      // bf16: two chains (even and odd fragments), each of half the sum: a logit is rounded at its full size once
      f32x16 s, s_odd;
#pragma unroll
      for (int v = 0; v < 16; ++v) s[v] = s_odd[v] = 0.f;
      if constexpr (TURNED) {
        if (!second) turn_keys();
      }
      u32x4 kf[kKS];
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) kf[ks] = lds_read16(k_at ^ (ks << 5));
#pragma unroll
      for (int g4 = 0; g4 < kKS; g4 += 4) {
        if (g4 + 4 < kKS) {
#pragma unroll
          for (int ks = g4 + 4; ks < g4 + 8; ++ks) kf[ks] = lds_read16(k_at ^ (ks << 5));
          arrived4<4>(kf[g4], kf[g4 + 1], kf[g4 + 2], kf[g4 + 3]);
        } else {
          arrived4<0>(kf[g4], kf[g4 + 1], kf[g4 + 2], kf[g4 + 3]);
        }
#pragma unroll
        for (int ks = g4; ks < g4 + 4; ++ks) {
          if constexpr (kBf16) {
            f32x16& chain = ks & 1 ? s_odd : s;
            chain = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[ks]), __builtin_bit_cast(bf16x8, qf[ks]), chain, 0, 0, 0);
          } else {
            const f32x4 k4 = __builtin_bit_cast(f32x4, kf[ks]), q4 = __builtin_bit_cast(f32x4, qf[ks]);
#pragma unroll
            for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(k4[e], q4[e], s, 0, 0, 0);
          }
        }
      }
      if constexpr (kBf16) s += s_odd;
      __builtin_amdgcn_sched_barrier(0);
      if (more) {
        spread(place_of(t + kWaves, next), mine);
        load_turn(t + kWaves);
        load_tile(mine, false);                                             // over the keys just consumed
      }
      __builtin_amdgcn_sched_barrier(0);
      if (j0 + kKT > lim_lo) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (j0 + 8 * (v / 4) + 4 * hi + (v % 4) >= lim) s[v] = -INFINITY;
      }
      float mx = s[0];
#pragma unroll
      for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[v]);
      mx = halves_max(mx) * a.scale;
      const float m_new = fmaxf(m_run, mx), m_use = m_new == -INFINITY ? 0.f : m_new;
      const float corr = exp_of<T>(m_run - m_use);
      m_run = m_new;
      float psum = 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        s[v] = exp_of<T>(__builtin_fmaf(s[v], a.scale, -m_use));
        psum += s[v];
      }
      l_run = l_run * corr + psum;
      if (__ballot(corr != 1.f) != 0ull) {
#pragma unroll
        for (int md = 0; md < kMD; ++md)
#pragma unroll
          for (int v = 0; v < 16; ++v) o[md][v] *= corr;
      }
      __builtin_amdgcn_sched_barrier(0);
      if (more) wait_loads<kLoads + kTurnLoads>();                          // the values; the next keys may be on their way
      else wait_loads<0>();
      if constexpr (kBf16) {
        i16x4 vf[2][kMD][2];
        auto request = [&](auto kp_c) {
          constexpr int kp = decltype(kp_c)::value;
#pragma unroll
          for (int md = 0; md < kMD; ++md) {
            vf[kp][md][0] = lds_read_tr<kp * 16 * D * 2>(v_at[md]);               // keys 16kp + 4hi + 0..3
            vf[kp][md][1] = lds_read_tr<(kp * 16 + 8) * D * 2>(v_at[md]);         // keys 16kp + 8 + 4hi + 0..3
          }
        };
        auto multiply = [&](auto kp_c) {
          constexpr int kp = decltype(kp_c)::value;
          constexpr int kNewer = kp == 0 ? 2 * kMD : 0;
#pragma unroll
          for (int md = 0; md < kMD; md += 2) arrived4<kNewer>(vf[kp][md][0], vf[kp][md][1], vf[kp][md + 1][0], vf[kp][md + 1][1]);
          // A probability goes in as three bf16 terms, each the rounded value of what the ones before it leave: together
          // they are its fp32 value, at a price in matrix instructions that a kernel waiting for memory hardly notices (6k
          // decode step 26.2 -> 26.6 us).  Two terms, sixteen bits, left ten times as many outputs off the nearest bf16
          // number: 2.3e-3 of them.
          bf16x8 pf, rest, last;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            pf[e] = (__bf16)s[8 * kp + e];
            const float left = s[8 * kp + e] - (float)pf[e];
            rest[e] = (__bf16)left;
            last[e] = (__bf16)(left - (float)rest[e]);
          }
#pragma unroll
          for (int md = 0; md < kMD; ++md) {
            const i16x8 both = __builtin_shufflevector(vf[kp][md][0], vf[kp][md][1], 0, 1, 2, 3, 4, 5, 6, 7);
            o[md] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), pf, o[md], 0, 0, 0);
            o[md] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), rest, o[md], 0, 0, 0);
            o[md] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), last, o[md], 0, 0, 0);
          }
        };
        request(std::integral_constant<int, 0>());
        request(std::integral_constant<int, 1>());
        multiply(std::integral_constant<int, 0>());
        multiply(std::integral_constant<int, 1>());
      } else {
        // step v multiplies keys 8*(v/4) + v%4 (lower half-wave) and + 4 (upper): the keys of S^T's register v
        float vf[2][4];
        auto request = [&](int e0) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int v = (e0 + i) / kMD, md = (e0 + i) % kMD;
            vf[(e0 / 4) & 1][i] = lds_read4(v_at[md] + (8 * (v / 4) + v % 4) * kRowBytes);
          }
        };
        request(0);
#pragma unroll
        for (int e0 = 0; e0 < 16 * kMD; e0 += 4) {
          float(&x)[4] = vf[(e0 / 4) & 1];
          if (e0 + 4 < 16 * kMD) {
            request(e0 + 4);
            arrived4<4>(x[0], x[1], x[2], x[3]);
          } else {
            arrived4<0>(x[0], x[1], x[2], x[3]);
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) o[(e0 + i) % kMD] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i], s[(e0 + i) / kMD], o[(e0 + i) % kMD], 0, 0, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if (more) {
        // the index entries of the tile after the next are requested in front of the values, so that nothing newer than
        // the values is outstanding at the wait in front of the next tile
        if (t + 2 * kWaves < tile_end) next = lookup(t + 2 * kWaves);
        load_tile(mine, true);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // ---- the waves' results meet in LDS, in the space each has staged its tiles in: rows 0..15 in the keys' part, the
  // others in the values', 16-byte slots swizzled by row.  Accumulator register v of tile md is dim
  // 32 md + 8 (v/4) + 4 hi + v%4.
  const int rows_here = n_rows - rt * kRows < kRows ? n_rows - rt * kRows : kRows;
  l_run = halves_sum(l_run);
  if (hi == 0) {
    ml[wave][r][0] = m_run;
    ml[wave][r][1] = l_run;
  }
  if (has_tile && r < rows_here) {
    unsigned char* ot = (r < 16 ? k_st[wave] : v_st[wave]) + (r & 15) * (D * 4);
#pragma unroll
    for (int md = 0; md < kMD; ++md)
#pragma unroll
      for (int vg = 0; vg < 4; ++vg) {
        const f32x4 w = {o[md][4 * vg], o[md][4 * vg + 1], o[md][4 * vg + 2], o[md][4 * vg + 3]};
        *(f32x4*)(ot + (((8 * md + 2 * vg + hi) ^ (r & 7)) << 4)) = w;
      }
  }
  __syncthreads();
  const bool final_out = n_slices == 1 && !a.to_slots;
  for (int e = tid; e < rows_here * (D / 4); e += 64 * kWaves) {
    const int q = e / (D / 4), p = e % (D / 4);
    // Everything is read before the first use, and a wave that saw no key of this row, which left no output, is not counted by a select (a sum
    // that is no number counts): behind a branch each wave's reads were a round trip to LDS of their own (from the barrier to the last store, one
    // token 0.75 -> 0.56 us, five 1.57 -> 1.15, 128 of fp32 1.26 -> 1.02).
    float2 of[kWaves];
    f32x4 part[kWaves];
    const unsigned char* ot = (q < 16 ? k_st[0] : v_st[0]) + (q & 15) * (D * 4) + ((p ^ (q & 7)) << 4);
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      of[w] = *(const float2*)ml[w][q];
      part[w] = *(const f32x4*)(ot + w * kTileBytes);
    }
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) M = fmaxf(M, of[w].x);
    float L = 0.f;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const bool counts = of[w].y != 0.f;
      const float wt = exp_of<T>(of[w].x - M);
      L = counts ? __builtin_fmaf(wt, of[w].y, L) : L;
#pragma unroll
      for (int i = 0; i < 4; ++i) sum[i] = counts ? __builtin_fmaf(wt, part[w][i], sum[i]) : sum[i];
    }
    const int qrow = rt * kRows + q, qc = a.group_log2 >= 0 ? qrow >> a.group_log2 : qrow / a.group, qh = g * a.group + qrow - qc * a.group;
    const int64_t orow = (int64_t)qc * a.h + qh, prow = (int64_t)b * a.l_c * a.h + orow;
    if (final_out) {
      const float inv = 1.f / L;
      T* dst = (T*)a.out + (int64_t)b * a.out_bs + orow * D + p * 4;
      if constexpr (kBf16) {
        *(uint2*)dst = make_uint2(pack_bf16x2(sum[0] * inv, sum[1] * inv), pack_bf16x2(sum[2] * inv, sum[3] * inv));
      } else {
        *(f32x4*)dst = sum * inv;
      }
      if (a.lse && p == 0) a.lse[prow] = lse_of<T>(M, L);
    } else {
      const int64_t slot = prow * a.n_slot + V.slot0 + split;
      *(f32x4*)(a.part_o + slot * D + p * 4) = sum;
      if (p == 0) *(float2*)(a.part_ml + slot * 2) = make_float2(M, L);
    }
  }
}

// Slices combined by their maxima and sums, WPR waves per output row.  Round trips are all this costs: every lane
// requests the (maximum, sum) pairs of the row and, without waiting for them, the partial outputs of its wave's slices
// (wave w takes slices w, w + WPR, ...), eight at a time; the waves' shares meet in LDS in a fixed order.
template <typename T, int D, int WPR>
__global__ __launch_bounds__(WPR == 1 ? 256 : 64 * WPR) void attend_split_merge(const float* __restrict__ part_o,
                                                                                const float* __restrict__ part_ml, int splits,
                                                                                int stride, int64_t rows, int64_t rows_per_batch,
                                                                                T* __restrict__ out, int64_t out_bs,
                                                                                float* __restrict__ lse) {
  constexpr int kPer = D >= 128 ? 2 : 1;              // dims per lane (D = 32: half the lanes repeat the others)
  static_assert(kMaxSplits <= 64, "two pairs per lane cover both parts of a two-call attention");
  __shared__ float red[WPR == 1 ? 1 : WPR][D];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t row = WPR == 1 ? (int64_t)blockIdx.x * 4 + wave : blockIdx.x;
  if (WPR == 1 && row >= rows) return;
  const int w0 = WPR == 1 ? 0 : wave, dim = (lane * kPer) % D;
  const float2* ml = (const float2*)(part_ml + row * stride * 2);   // slots [0, splits) of `stride` are in use
  float2 a0 = make_float2(-INFINITY, 0.f), a1 = make_float2(-INFINITY, 0.f);
  if (lane < splits) a0 = ml[lane];
  if (lane + 64 < splits) a1 = ml[lane + 64];
  const float* po = part_o + row * stride * D + dim;
  float o[8][kPer];
  auto request = [&](int s0) {                         // a slice past the end re-reads slice 0 and gets weight 0
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int s = s0 + WPR * u;
#pragma unroll
      for (int e = 0; e < kPer; ++e) o[u][e] = po[(int64_t)(s < splits ? s : 0) * D + e];
    }
  };
  request(w0);
  const float m = wave_max(fmaxf(a0.x, a1.x));
  const float f0 = a0.y != 0.f ? exp_of<T>(a0.x - m) : 0.f, f1 = a1.y != 0.f ? exp_of<T>(a1.x - m) : 0.f;
  const float l = wave_sum(__fmaf_rn(f0, a0.y, f1 * a1.y));
  float acc[kPer] = {};
  for (int s0 = w0; s0 < splits; s0 += 8 * WPR) {
    if (s0 != w0) request(s0);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int s = s0 + WPR * u;
      const float ws = __shfl(s < 64 ? f0 : f1, s & 63, 64);
      const float w = s < splits ? ws : 0.f;
#pragma unroll
      for (int e = 0; e < kPer; ++e) acc[e] += w != 0.f ? w * o[u][e] : 0.f;     // slices past the causal limit hold no output
    }
  }
  if constexpr (WPR > 1) {
#pragma unroll
    for (int e = 0; e < kPer; ++e) red[wave][dim + e] = acc[e];
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      acc[e] = 0.f;
#pragma unroll
      for (int i = 0; i < WPR; ++i) acc[e] += red[i][dim + e];
    }
  }
  const float inv = 1.f / l;
  T* dst = out + row / rows_per_batch * out_bs + row % rows_per_batch * D + dim;
  if (lane * kPer < D) {
    if constexpr (sizeof(T) == 2 && kPer == 2) {
      *(uint32_t*)dst = pack_bf16x2(acc[0] * inv, acc[1] * inv);
    } else {
#pragma unroll
      for (int e = 0; e < kPer; ++e) store_f32<T>(dst + e, acc[e] * inv);
    }
  }
  if (lse && lane == 0) lse[row] = lse_of<T>(m, l);
}

int row_tiles(int l_c, int h, int h_kv) { return (l_c * (h / h_kv) + kRows - 1) / kRows; }

// Most slices of a view: enough for about kTargetWorkgroups workgroups (known without the number of keys, so that the
// workspace is).
int split_limit(int l_c, int h, int h_kv, int batch) {
  const int64_t per_slice = (int64_t)row_tiles(l_c, h, h_kv) * h_kv * batch;
  const int64_t ns = kTargetWorkgroups / per_slice;
  return (int)(ns < 1 ? 1 : (ns > kMaxSplits ? kMaxSplits : ns));
}
// Slices of n_keys keys: a tile per wave at least.
int split_count(int limit, int64_t n_keys, int waves = kWavesOfTwo) {
  const int64_t most = (n_keys + kKT * waves - 1) / (kKT * waves);
  return (int)(most < 1 ? 1 : (most < limit ? most : limit));
}
// Waves of a workgroup: five where workgroups of four with a tile per wave are a few more than the compute units and those of five are not.
// A compute unit takes 64 KB of tiles in 0.9 us and 128 KB in 2.3 (a row at a time into LDS), so that the sixteen that got two workgroups
// of 272 kept the others waiting: one token over 4225 keys of 8 KV heads 7.35 -> 6.6 us from first entry to last store (8.3 -> 7.4 on a
// long document), a step 41.5 -> 40.35, re-encoded 46.9 -> 45.6.
int waves_of(int64_t groups, int64_t n_keys0, int64_t n_keys1) {
  auto workgroups = [&](int w) { return groups * ((n_keys0 + kKT * w - 1) / (kKT * w) + (n_keys1 + kKT * w - 1) / (kKT * w)); };
  return workgroups(kWavesOfTwo) > 256 && workgroups(kWavesOfOne) <= (256 < groups * kMaxSplits ? 256 : groups * kMaxSplits) ? kWavesOfOne : kWavesOfTwo;
}

size_t ml_offset(int64_t rows, int n_slot, int d) { return align_up((size_t)rows * n_slot * d * sizeof(float), 256); }
size_t slots_bytes(int64_t rows, int n_slot, int d) {
  return ml_offset(rows, n_slot, d) + align_up((size_t)rows * n_slot * 2 * sizeof(float), 256);
}

SplitArgs make_args(const SplitCall& c) {
  const int64_t esz = c.dtype == ESA_F32 ? 4 : 2;
  SplitArgs a = {};
  a.out = c.out;
  a.lse = c.lse;
  a.k_sel = (const char*)c.k_sel;
  a.v_sel = (const char*)c.v_sel;
  a.sel_bytes = (uint32_t)((int64_t)c.h_kv * c.d * esz);
  a.l_c = c.l_c;
  a.h = c.h;
  a.h_kv = c.h_kv;
  a.group = c.h / c.h_kv;
  a.n_rt = row_tiles(c.l_c, c.h, c.h_kv);
  a.group_log2 = (a.group & (a.group - 1)) == 0 ? __builtin_ctz(a.group) : -1;
  a.scale = c.dtype == ESA_F32 ? c.scale : c.scale * kLog2e;
  a.out_bs = c.out_bs;
  a.sel_bs_bytes = c.sel_bs * esz;
  a.turns = (const double*)c.turns;
  return a;
}
int with_slots(SplitArgs* a, const SplitCall& c, int n_slot) {
  const int64_t rows = (int64_t)c.batch * c.l_c * c.h;
  if (!c.ws || c.ws_bytes < slots_bytes(rows, n_slot, c.d)) ESA_FAIL(ESA_EWORKSPACE, "attend_split: workspace too small");
  a->n_slot = n_slot;
  a->part_o = (float*)c.ws;
  a->part_ml = (float*)((char*)c.ws + ml_offset(rows, n_slot, c.d));
  return ESA_OK;
}

// Whether each row of keys and values is fetched by one workgroup and they are together more than the last-level cache keeps from
// one layer's step to the next beside what else passes through it.  One token, 16 x 4225 keys of 8 KV heads (277 MB), us, three inputs in turn:
// 54.7 -> 50.2 (55.2 -> 50.4 on long documents); 8 sequences (138 MB) 31.1 -> 28.9, 4 (69 MB) 19.3 -> 18.3.  Less is often there still:
// 3 sequences (52 MB) 14.6 / 14.7, five tokens of 2 (35 MB) 14.4 -> 15.3.  (One input again and again: 8 sequences 26.6 -> 29.1.)  Row tiles that share
// keys want them kept (fp32, sixteen row tiles: a step 52.2 -> 53.9); so do gathered rows, which have just been written (8 re-encoded sequences 34.5 -> 35.4),
// and sequences that share one cache (16 of them 28.9 / 30.6).
bool streams(const SplitCall& c, const SplitArgs& a, int64_t n_keys) {
  const KeyView& v = a.view[0];
  if (c.batch > 1 && (v.k_bs_bytes == 0 || v.v_bs_bytes == 0)) return false;
  return c.dtype == ESA_BF16 && a.n_rt == 1 && !c.turns && !c.k_sel && 2 * n_keys * c.h_kv * c.batch * c.d * 2 >= ((int64_t)64 << 20);
}
template <typename T, int D>
void run(const SplitCall& c, const SplitArgs& args, int waves, bool stream, hipStream_t st) {
  SplitArgs a = args;
  auto kernel = attend_split<T, D, kWavesOfTwo>;
  if constexpr (sizeof(T) == 2) {
    if (stream) kernel = attend_split<T, D, kWavesOfTwo, false, true>;
    else if (waves == kWavesOfOne) kernel = a.turns ? attend_split<T, D, kWavesOfOne, true> : attend_split<T, D, kWavesOfOne>;
    else if (a.turns) kernel = attend_split<T, D, kWavesOfTwo, true>;
  }
  for_pair_grids((int64_t)c.batch * c.h_kv, a.n_rt, a.view[0].n_split + a.view[1].n_split, [&](dim3 grid, PairGrid placed) {
    a.grid = placed;
    kernel<<<grid, 64 * waves, 0, st>>>(a);
  });
}
template <typename T, int D>
void merge(const SplitCall& c, const SplitArgs& a, int splits, hipStream_t st) {
  const int64_t per_batch = (int64_t)c.l_c * c.h, rows = per_batch * c.batch;
  // many slices of few rows: eight waves share a row's partial outputs, so that they are all requested at once
  if (splits > 16)
    attend_split_merge<T, D, 8><<<dim3((unsigned)rows), 512, 0, st>>>(a.part_o, a.part_ml, splits, a.n_slot, rows, per_batch, (T*)c.out, c.out_bs, c.lse);
  else
    attend_split_merge<T, D, 1><<<dim3((unsigned)((rows + 3) / 4)), 256, 0, st>>>(a.part_o, a.part_ml, splits, a.n_slot, rows, per_batch, (T*)c.out, c.out_bs, c.lse);
}
// what: (call, args) -> void for the storage type and head size of the call
template <typename F>
void dispatch(const SplitCall& c, F&& f) {
  if (c.dtype == ESA_F32) {
    if (c.d == 32) f.template operator()<float, 32>();
    else if (c.d == 64) f.template operator()<float, 64>();
    else f.template operator()<float, 128>();
  } else {
    if (c.d == 64) f.template operator()<bf16_t, 64>();
    else f.template operator()<bf16_t, 128>();
  }
}
struct RunIt {
  const SplitCall& c;
  const SplitArgs& a;
  hipStream_t st;
  int waves = kWavesOfTwo;
  bool stream = false;
  template <typename T, int D> void operator()() { run<T, D>(c, a, waves, stream, st); }
};
struct MergeIt {
  const SplitCall& c;
  const SplitArgs& a;
  int splits;
  hipStream_t st;
  template <typename T, int D> void operator()() { merge<T, D>(c, a, splits, st); }
};

int64_t keys_of(const KeyView& v, int l_c) { return (int64_t)v.n_fixed + (v.with_chunk ? l_c : 0); }

}  // namespace

// The launch grid has one workgroup per (batch entry, KV head, row tile, slice).
bool attend_split_supported(int l_c, int h, int h_kv, int d, int dtype, int batch) {
  if (h % h_kv != 0) return false;
  if (dtype == ESA_BF16 ? (l_c >= 16 || (d != 64 && d != 128)) : (d != 32 && d != 64 && d != 128)) return false;
  return (int64_t)l_c * (h / h_kv) < (1 << 30) &&
         (int64_t)row_tiles(l_c, h, h_kv) * h_kv * batch * 2 * split_limit(l_c, h, h_kv, batch) < ((int64_t)1 << 31);
}

// Turning costs a call 1.5 us and more, a copy its bytes.  Copied / turned, us, by batch entries x KV heads x local keys, one token and four:
// 1 x 4096 12.8 / 13.8, 13.9 / 14.9; 2 x 2048 13.3 / 14.2, 16.1 / 16.9; 2 x 4096 13.9 / 14.1, 17.7 / 17.0; 4 x 2048 14.8 / 14.2, 17.9 / 17.2;
// 16 x 512 14.1 / 13.7, 15.6 / 14.9; 8 x 4096 21.7 / 17.4, 22.7 / 19.7; 64 x 2048 40.0 / 34.3, 41.6 / 34.9; head size 64: 2 x 2048 11.3 / 11.8,
// 2 x 4096 11.7 / 11.8, 4 x 2048 11.95 / 11.8, 64 x 2048 26.8 / 23.2.
bool attend_split_turns_keys(int l_c, int h, int h_kv, int d, int dtype, int batch, int64_t n_keys) {
  return dtype == ESA_BF16 && attend_split_supported(l_c, h, h_kv, d, dtype, batch) && row_tiles(l_c, h, h_kv) == 1 && n_keys * h_kv * batch >= 8192;
}

size_t attend_split_workspace_bytes(int l_c, int h, int h_kv, int d, int dtype, int batch) {
  (void)dtype;
  return slots_bytes((int64_t)batch * l_c * h, 2 * split_limit(l_c, h, h_kv, batch), d);
}

int launch_attend_split(const SplitCall& c, KeyView v0, const KeyView* v1, hipStream_t st) {
  SplitArgs a = make_args(c);
  const int limit = split_limit(c.l_c, c.h, c.h_kv, c.batch);
  const int64_t k0 = keys_of(v0, c.l_c), k1 = v1 ? keys_of(*v1, c.l_c) : 0;
  const int waves = c.dtype == ESA_BF16 ? waves_of((int64_t)a.n_rt * c.h_kv * c.batch, k0, k1) : kWavesOfTwo;
  int n0 = limit, n1 = 0;
  if (waves == kWavesOfOne) {
    n1 = k1 > 0 ? split_count(limit, k1, waves) : 0;
  } else if (k1 > 0) {            // the slices are shared out in proportion to the two parts' lengths, at least one each
    n1 = (int)((limit * k1 + (k0 + k1) / 2) / (k0 + k1));
    n1 = n1 < 1 ? 1 : n1;
    n0 = limit - n1 < 1 ? 1 : limit - n1;
    n1 = split_count(n1, k1);
  }
  n0 = split_count(n0, k0, waves);
  a.view[0] = v0;
  set_splits(&a.view[0], n0, 0);
  a.view[1] = k1 > 0 ? *v1 : v0;
  set_splits(&a.view[1], n1, n0);
  if (n0 + n1 > 1) {
    const int rc = with_slots(&a, c, n0 + n1);
    if (rc != ESA_OK) return rc;
  }
  dispatch(c, RunIt{c, a, st, waves, waves == kWavesOfTwo && streams(c, a, k0 + k1)});
  if (n0 + n1 > 1) dispatch(c, MergeIt{c, a, n0 + n1, st});
  ESA_LAUNCH_CHECK("attend_split");
  return ESA_OK;
}

int launch_attend_split_early(const SplitCall& c, KeyView early, int64_t early_keys, hipStream_t st) {
  SplitArgs a = make_args(c);
  const int limit = split_limit(c.l_c, c.h, c.h_kv, c.batch);
  const int rc = with_slots(&a, c, 2 * limit);
  if (rc != ESA_OK) return rc;
  a.to_slots = 1;
  a.view[0] = early;
  set_splits(&a.view[0], split_count(limit, early_keys), 0);
  a.view[1] = early;
  set_splits(&a.view[1], 0, 0);
  dispatch(c, RunIt{c, a, st});
  ESA_LAUNCH_CHECK("attend_split (early part)");
  return ESA_OK;
}

int launch_attend_split_late(const SplitCall& c, KeyView late, int64_t late_keys, int64_t early_keys, hipStream_t st) {
  SplitArgs a = make_args(c);
  const int limit = split_limit(c.l_c, c.h, c.h_kv, c.batch), n_early = split_count(limit, early_keys);
  const int rc = with_slots(&a, c, 2 * limit);
  if (rc != ESA_OK) return rc;
  a.to_slots = 1;
  a.view[0] = late;
  set_splits(&a.view[0], late_keys > 0 ? split_count(limit, late_keys) : 0, n_early);
  a.view[1] = late;
  set_splits(&a.view[1], 0, 0);
  if (late_keys > 0) dispatch(c, RunIt{c, a, st});
  dispatch(c, MergeIt{c, a, n_early + a.view[0].n_split, st});
  ESA_LAUNCH_CHECK("attend_split (late part)");
  return ESA_OK;
}

}  // namespace esa

// Importance of every middle token (Eq. 6 inside Eq. 4):
//   S[c,m] = q'_c . k'_m,  mu[c] = max_m S[c,m],  F[m] = max_c (S[c,m] - mu[c]),
// optionally with the proximity max-pool of Eq. 8: narrow windows in the kernel that writes the scores, wider ones (and those whose lap
// would take the sweeps another round of workgroups) behind it.
//
// F needs every row maximum before any column maximum.  A chunk of more than a few queries sweeps K' twice and
// recomputes S instead of storing it (S would be l_C x N fp32; K' is only N x d_c storage elements).  Both sweeps compute
// S[c,m] with the same instruction sequence, so the second one reproduces the first bit for bit: the row arg-max token
// gets F = 0 exactly and F <= 0 everywhere.  With up to sixteen queries a row of S is a fraction of a row of K' (4 bytes
// per query against 128 or 256 per token), and a small problem's S is small whatever its shape: there S is stored by one
// sweep, with per-workgroup row maxima beside it, and score_finish subtracts and takes the column maximum.
//
// This file is compiled with the IEEE mode bit off and NaNs declared absent (see build.py): with the bit
// on, every fmaxf() on a matrix-core result costs three instructions, because the compiler first
// "canonicalises" each operand it cannot prove free of signalling NaNs (a max of the value with
// itself).  No NaN occurs here (inputs are finite by contract; -inf is only ever compared).
#include "esa_common.h"
#include <type_traits>
#include "radix_hist.h"
#include "score_shares.h"

namespace esa {
namespace {

// Work-item and workgroup numbers are taken from the hardware builtins in this file: with the IEEE mode bit
// off (see build.py) the device library's accessors behind threadIdx / blockIdx / gridDim are not inlined (their
// floating-point mode attributes differ from the kernels'), and every use would be a function call.

// Workspace: the row maxima (uint32 keys or fp32; eight copies of them and the shares' marks for the matrix-core sweeps, or
// [batch][blocks][l_c] fp32 partial maxima of the kernels that store S), then (windows that no score kernel pools)
// [batch][n] fp32 unpooled scores, then S where it is stored.
__host__ __device__ inline size_t mu_bytes(int l_c, int batch) {      // rows padded to whole groups of 64
  return align_up((size_t)((l_c + 63) / 64 * 64) * batch * 4, 256);
}

__global__ void fill_u32(uint32_t* p, int64_t n, uint32_t v) {
  const int64_t i = (int64_t)__builtin_amdgcn_workgroup_id_x() * 256 + __builtin_amdgcn_workitem_id_x();   // one thread per word
  if (i < n) p[i] = v;
}

// ------------------------------------------------------------------------------------------ generic
constexpr int kGTok = 64;      // middle tokens per block (one per lane)

// One fixed-order dot product in fp32, shared by both sweeps.  Of fp32 rows, in the order of the matrix instructions of score_store_f32, so that a token's
// score does not depend on the call: two chains, of every other eight dimensions, each taking dimensions 0, 4, 1, 5, 2, 6, 3, 7 of its eight.  (One ascending chain:
// scores 1.83e-7 from the 64-bit result at d_c 32, so 1.35e-7; 3.99e-7 and 2.29e-7 at 128.)  d_c is a multiple of 16.
template <typename T>
__device__ __forceinline__ float dot_fixed(const T* __restrict__ q, const float* __restrict__ krow, int d_c) {
  if constexpr (sizeof(T) == 4) {
    float even = 0.f, odd = 0.f;
    for (int i = 0; i < d_c; i += 16)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int at = i + e / 2 + e % 2 * 4;
        even = __fmaf_rn(q[at], krow[at], even);
        odd = __fmaf_rn(q[at + 8], krow[at + 8], odd);
      }
    return even + odd;
  } else {
    float s = 0.f;
    for (int i = 0; i < d_c; ++i) s = __fmaf_rn(load_f32(q + i), krow[i], s);
    return s;
  }
}

// SWEEP 0: row maxima into mu_keys.  SWEEP 1: F into score.
template <typename T, int SWEEP>
__global__ __launch_bounds__(256) void score_fma(const T* __restrict__ qc, int l_c, const T* __restrict__ kc,
                                                 int64_t m_lo, int64_t n, int d_c, uint32_t* __restrict__ mu_keys,
                                                 float* __restrict__ score, int64_t q_bs, int64_t kc_bs,
                                                 int64_t score_bs) {
  extern __shared__ float smem[];                 // kt[kGTok][d_c+1], then red[4][kGTok]
  const int ldk = d_c + 1;
  float* kt = smem;
  float* red = smem + kGTok * ldk;
  const int b = __builtin_amdgcn_workgroup_id_y();
  const T* q = qc + (int64_t)b * q_bs;
  const T* k = kc + (int64_t)b * kc_bs + m_lo * (int64_t)d_c;
  uint32_t* mu = mu_keys + (int64_t)b * l_c;
  const int64_t m0 = (int64_t)__builtin_amdgcn_workgroup_id_x() * kGTok;
  for (int e = __builtin_amdgcn_workitem_id_x(); e < kGTok * d_c; e += 256) {
    const int t = e / d_c, i = e % d_c;
    kt[t * ldk + i] = (m0 + t < n) ? load_f32(k + (m0 + t) * (int64_t)d_c + i) : 0.f;
  }
  __syncthreads();
  const int lane = __builtin_amdgcn_workitem_id_x() & 63, wave = __builtin_amdgcn_workitem_id_x() >> 6;
  const bool valid = (m0 + lane) < n;
  float best = -INFINITY;
  for (int c = wave; c < l_c; c += 4) {
    float s = dot_fixed(q + (int64_t)c * d_c, kt + lane * ldk, d_c);
    if (!valid) s = -INFINITY;
    if (SWEEP == 0) {
      const float mx = wave_max(s);
      if (lane == 0) atomicMax(&mu[c], ordered_key(mx));
    } else {
      best = fmaxf(best, s - ordered_key_to_f32(mu[c]));
    }
  }
  if (SWEEP == 1) {
    red[wave * kGTok + lane] = best;
    __syncthreads();
    if (wave == 0 && valid) {
      const float f = fmaxf(fmaxf(red[lane], red[kGTok + lane]), fmaxf(red[2 * kGTok + lane], red[3 * kGTok + lane]));
      score[(int64_t)b * score_bs + m0 + lane] = f;
    }
  }
}


// ------------------------------------------------------------------------------------------ MFMA (bf16, d_c = 128 or 64)
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// v_mfma_f32_32x32x16_bf16 computes D[32x32] += A[32x16] B[16x32].  Lane l supplies eight
// consecutive reduction elements of A row l%32 and of B column l%32 (which eight depends only on
// l/32, identically for A and B), and owns D[8*(v/4) + 4*(l/32) + v%4][l%32] in register v.
//
// Here A rows are current tokens (queries), B columns are middle tokens.  A workgroup of eight
// waves (two per SIMD) owns up to 512 consecutive middle tokens.  Its whole share of K' (at most
// 128 KB) goes from memory straight into LDS, without passing through registers: sixteen (d_c = 64:
// eight) global_load_lds_dwordx4 per thread, issued back to back at the start of the kernel, each wave
// instruction bringing four 256-byte (eight 128-byte) rows.  Which 16 bytes of its row a lane fetches is
// chosen such that the rows land XOR-swizzled (piece p of row R in slot p ^ R%16; d_c = 64, where two rows
// share the 256 bytes that the banks cover: p ^ (R/2)%8), which makes the fragment
// reads free of bank conflicts without padding.  Loads complete in order, so tile t (32 tokens,
// instruction t, or t/2, of every wave) is usable once every wave has waited for its own instruction and
// a barrier has passed; the tiles are consumed as they land, two per barrier.  Queries are the
// register-resident operand (64 per wave as A fragments for the whole d_c; chunks longer than
// 512 loop over query blocks against the same LDS tile).  Share and queries stay where they are for the second sweep, so K' is read
// from memory once, or, where the shares are more than a round of workgroups, once and again all but the last share of each.
// Up to 256 queries do not give every wave 64 of its own: where it pays, the waves that hold the same ones share out the tiles (query_waves_log2).
//
// Inside a wave the tiles are software-pipelined: right after the matrix instructions of reduction
// step ks of tile t have issued, fragment ks of tile t+1 is read from LDS into the registers they
// have just released, and the maximum / subtract work on tile t-1's accumulators (a second
// accumulator set) sits between the matrix instructions, so that one wave alone keeps the matrix
// pipe fed.  With a token per lane, the column maximum of Eq. 4 is an in-lane reduction over the
// accumulator registers plus one exchange between the two half-waves, folded across waves with an
// LDS integer maximum on order-preserving keys; the row maximum is kept per register across all
// tiles and reduced across lanes once.
//
// While the share is landing, every LDS access of the tile loop is written as an instruction of its
// own with its own counter waits: an LDS access the compiler generates is preceded by a wait for ALL
// outstanding loads into LDS (it cannot tell which rows they fill), which would turn the stream into
// one round trip followed by the arithmetic.  LDS operations complete in order, which the waits
// below rely on: "at most 7 (d_c = 64: 3) outstanding" before the use of fragment ks means that fragment
// has arrived, because exactly so many fragment reads were issued after it (the rest of this tile's and the
// first ks of the next tile's).  Operations the compiler adds on the same counter are newer still
// and only make these waits stricter.
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) unsigned char lds_byte;
typedef __attribute__((address_space(1))) const void global_void;
constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kMT = 2;                   // 32-query tiles per wave
constexpr int kQPerWave = 32 * kMT;
constexpr int kQPerBlock = kWaves * kQPerWave;

// eps > 0: the second sweep pools over +-eps (Eq. 8, at most kTailMaxEps).  Shares then lap over their neighbours' by eps tokens
// on either side, so that a workgroup has the scores of every window it writes; the first sweep's are the same ones.  With a pooling kernel of its own, which read the scores back and built the selection's histogram (4.9 us), a re-encoded step
// took 63.3 us instead of 61.0 (40 tokens at 50 thousand), 80.1 / 77.0 (128 at 100), 62.4 / 59.9 (60 at 12), 77.6 / 75.8 (256 at 30) and the same
// 134 (512 at 130).
// (score_shares.h: how long a share is, and when.)
// Waves of a workgroup that hold different queries (64 each), a power of two; the others take other tiles for the same ones, which takes all tiles in LDS and a
// barrier more for the row maxima.  A share of up to four tiles, or of d_c = 128 and more than 128 queries (whose waves are on all SIMDs as they are), is quicker
// without: eight.  Score, us, shared out / eight waves: 48 queries over 8 thousand tokens (two tiles) 12.2 / 11.0, 17 over 15 12.6 / 11.2 (two launches of all
// eight waves 11.4), 128 over 30 (four) 12.8 / 12.8, 45 (six) 13.4 / 14.4; 129 over 45 15.6 / 14.4, 200 39.3 / 36.4, 256 over 60 17.1 / 16.3, over 8 rows of 50 92.0 /
// 81.2; d_c = 64, 256 queries, 60 thousand 12.5 / 12.9, 12 rows of 120 161 / 170.
__host__ inline int query_waves_log2(int l_c, int per, int d_c) {
  if (per <= 4 || (d_c == 128 && l_c > 128)) return 3;
  return l_c > 256 ? 3 : l_c > 128 ? 2 : l_c > 64 ? 1 : 0;
}
__host__ inline int query_waves(int l_c, int per, int d_c) { return 1 << query_waves_log2(l_c, per, d_c); }
// The first block of queries comes in through LDS behind the share's first tiles, in the place of those that are requested when it
// is in registers: as many as leave room, or, where all eight waves hold queries and consume the tiles as they land, four.
__host__ inline int tiles_before_queries(int per, int d_c, int l_c) {
  const int waves = query_waves(l_c, per, d_c), room = (160 * 1024) / (64 * d_c) - 2 * waves, first = waves == kWaves ? 4 : room;
  return per < first ? per : first;
}
// The share and behind it the second sweep's column maxima, digit histogram and row maxima.
__host__ inline size_t second_sweep_lds_bytes(int per, int d_c) {
  return (size_t)per * 32 * d_c * sizeof(bf16_t) + (size_t)(per + 1) * 32 * sizeof(uint32_t) + (size_t)kRadixBins * sizeof(uint32_t) + (size_t)(kQPerBlock + 4) * sizeof(float);
}
// Later blocks of a chunk of more than 512 queries come in through LDS too, behind all of that, while the block before is at work: whole (1), where there is
// no room for it half of each wave's queries at a time (2); or, where a block is few queries or there is no room, straight from memory (0).  d_c = 128, score,
// us, from memory / so: shares of two tiles (whole): 600 queries over 8 thousand tokens 17.4 / 15.7, 1024 21.4 / 17.7, 2048 36.5 / 28.7, 4096 67.4 / 49.0 (61.3 as two
// launches), 8192 129.1 / 91.2 (109.0); of four (halves): 600 over 30 20.3 / 19.5, 1000 25.7 / 23.9, 4096 85.0 / 77.0; of eight: 600 over 60 26.6 / 27.7, 832
// 33.5 / 33.4, 1000 35.6 / 34.0, 4096 126.3 / 117.7; of ten: 900 over 80 41.7 / 41.4, 1000 42.7 / 41.3.
__host__ inline int later_queries_parts(int per, int d_c, int l_c) {
  const size_t at = align_up(second_sweep_lds_bytes(per, d_c), 1024), block = (size_t)kQPerBlock * d_c * sizeof(bf16_t);
  if (l_c <= kQPerBlock) return 0;
  if (at + block <= 160 * 1024) return 1;
  return at + block / 2 <= 160 * 1024 && (per <= 4 || l_c >= 896) ? 2 : 0;
}
__host__ inline int later_queries_at(int per, int d_c) { return (int)align_up(second_sweep_lds_bytes(per, d_c), 1024); }
__host__ inline size_t sweeps_lds_bytes(int per, int d_c, int l_c) {
  const size_t tile = 32 * d_c * sizeof(bf16_t), staged = (tiles_before_queries(per, d_c, l_c) + 2 * query_waves(l_c, per, d_c)) * tile;
  const int parts = later_queries_parts(per, d_c, l_c);
  const size_t second = parts ? later_queries_at(per, d_c) + (size_t)kQPerBlock * d_c * sizeof(bf16_t) / parts : second_sweep_lds_bytes(per, d_c);
  return staged > second ? staged : second;
}
// Marks of the shares that are done: sixteen to a word, a word to 256 bytes, and kMuCopies copies of them all, one for the readers on each XCD:
// whatever reaches one cache line from several XCDs is served one at a time (250 workgroups behind the last one's mark: 7 us with all
// words in one line, 3.2 with 64 bytes for each, 2.2 with 256).
constexpr int kMuCopies = 8, kMarksPerWord = 16, kMarkStride = 64;
__host__ __device__ constexpr int64_t mark_words(int64_t shares) { return (shares + kMarksPerWord - 1) / kMarksPerWord * kMarkStride; }   // of a copy
// Row maxima of the matrix-core path: one row of mfma_mu_stride(l_c) floats per batch entry, so that groups
// of four are 16-byte aligned and in bounds for every query tile that holds a query.
__host__ __device__ inline int mfma_mu_stride(int l_c) { return (l_c + 63) / 64 * 64; }

// Wait until at most LEFT vector-memory loads of this wave are outstanding, then the workgroup barrier.  It waits for no LDS operation: fragment reads
// in flight stay in flight across it, and what the waves write to LDS for one another takes a __syncthreads.
template <int LEFT>
__device__ __forceinline__ void wait_loads_then_barrier() {
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(LEFT) : "memory");
}

// The kernel.  Workgroup g owns shares g, g + grid, ... of all rows together (one, where a round of workgroups takes them all).  It
// finds its shares' row maxima, folds them into mu_keys with atomic maxima, marks the share as done, waits until every share is
// done, and computes the scores of its shares, the last one of which is still in LDS and its queries still in registers.
// What bounds it: the matrix instructions of the two tile loops where queries are many (in-kernel stamps, 512 queries over 128 thousand tokens: 3.9 us until
// the first, 11 + 10.7 of tile loops, 1.5 of waiting for the slowest workgroup's mark, 0.9 for the row maxima, 1.2 of epilogue); the round trips in
// front of, between and behind them where they are few (77 over 48 thousand: 11.7 in all, 3.3 until the first instruction).
// As two launches with a kernel between them that reduced partial row maxima, a call paid for that kernel, a second start of all
// workgroups, a second fetch of the share and of the queries: 20.7 + 4.9 + 19.2 us against 4.9 + 35.5 with score_sweeps_clear (512 queries, 128 thousand
// tokens), 7.4 + 2.3 + 7.6 against 2.1 + 13.7 (77, 48).  Steps: 101.3 -> 97.2 us, 49.6 -> 46.7; 1024 at 256k 417 -> 407, re-encoded 512 140.5 -> 133.6.
//
// The wait needs no other workgroup to be resident: it is bounded by the time the workgroup has been running itself plus kPatience, and a
// workgroup that has waited so long does the missing shares' row maxima itself, one after the other (the maxima are
// idempotent; whoever finishes a share marks it), so that every workgroup gets to its end whatever else holds the other compute units.
// What a waiting workgroup holds meanwhile another stream's kernels do not get, and the other way round: a step of 512 tokens at 128 thousand whose local attention
// starts on a second stream in front of the sweeps takes 148.5 us where the two launches took 137.5 (behind them 126.4 and 132.3; on one stream 104 and 109.5).
//
// What crosses workgroups inside the launch goes through device-scope atomics only (maxima, marks, and the loads that read them), each
// wave's maxima complete (vmcnt) before its workgroup's marks: no fence, which would write back an L2 (5 to 10 us).  One copy of
// the maxima per XCD: maxima on one address are served one at a time, 17 to 30 ns each.
// What a workgroup waits beyond the time it has been running: those of a short call start up to 2 us apart, and redoing a share costs more than that.
constexpr uint64_t kPatience = 500;              // 5 us in ticks of 10 ns (s_memrealtime)

// LATER: how the blocks of queries behind the first come in (see later_queries_parts).
template <int DC, int LATER>
__global__ __launch_bounds__(kThreads) void score_sweeps_bf16(const bf16_t* __restrict__ qc, const bf16_t* __restrict__ kc, int n, int l_c_arg,
                                                              int tiles_per_block, int before_queries, int member_bits, int n_row,
                                                              int n_shares, int n_wg, int eps, uint32_t row_inverse, uint32_t* mu_keys, uint32_t* marks,
                                                              float* __restrict__ score, int64_t q_bs, int64_t kc_bs, int64_t score_bs,
                                                              uint32_t* __restrict__ first_hist, int64_t first_hist_bs,
                                                              uint32_t patience, int later_at) {     // kc: the first middle token's row
  static_assert(DC == 64 || DC == 128, "swizzle and load pattern");
  constexpr int kDc = DC;
  constexpr int kKSteps = kDc / 16;        // MFMA reduction steps per tile
  constexpr int kTileBytes = 32 * kDc * 2; // one tile of K' in LDS
  constexpr int kPieces = kDc / 8;         // 16-byte pieces of a row
  constexpr int kTilesPerLoad = kWaves * 1024 / kTileBytes;           // tiles that one load instruction per wave brings
  constexpr int kLoads = kMaxTilesPerBlock / kTilesPerLoad;           // load instructions of a full share
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
  const uint64_t started = __builtin_amdgcn_s_memrealtime();
  int tpb = tiles_per_block, l_c = l_c_arg;
  const int span = tpb * 32;                                           // tokens of a share
  uint32_t* colmax = (uint32_t*)(lds_raw + (size_t)tpb * kTileBytes);  // second sweep: [32 spare + span] keys
  uint32_t* digit_hist = colmax + 32 + span;                           // [kRadixBins]
  float* mu_rows = (float*)(digit_hist + kRadixBins);                  // [kWaves][kQPerWave]
  int* todo = (int*)(mu_rows + kQPerBlock);                            // the share that nobody has done, or -1
  int wave = __builtin_amdgcn_readfirstlane(__builtin_amdgcn_workitem_id_x() >> 6);      // uniform: lives in a scalar register
  int n_groups = kWaves >> member_bits, member = wave & ((1 << member_bits) - 1), group = wave >> member_bits;
  const int wg = __builtin_amdgcn_workgroup_id_x();
  // The lane's number, taken afresh wherever it is needed outside the tile loop, whose registers are all spoken for: what is
  // computed from a value that the compiler knows to stay the same it would keep (or spill) through the loop.
  auto lane_now = [&]() -> int {
    uint32_t l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return (int)l;
  };
  // The same for the scalars that most addresses and conditions follow from: new values, as far as the compiler knows, once per share
  // (it put 200 instructions in front of the first request).
  auto scalars_afresh = [&]() { asm volatile("" : "+s"(tpb), "+s"(l_c), "+s"(wave), "+s"(n_groups), "+s"(member), "+s"(group)); };
  const uint32_t lds_tiles = (uint32_t)(uintptr_t)(lds_byte*)lds_raw;  // LDS byte address of the share
  const uint32_t lds_colmax = lds_tiles + (uint32_t)tpb * kTileBytes;

  // the share at hand.  Its row: a product with row_inverse (see inverse_of).  Counted down row by row, 1024 rows of 1500 tokens took 332 us, not 184,
  // and 4096 of 1200 3507, not 632; a division, set up in front of the first request, costs one row 0.15 us (the product: none; two rows 0.1).
  int b = 0, blk = 0;
  int tok_base = 0;
  const char* kshare = nullptr;
  uint32_t first_row = 0, last_row = 0;                           // rows outside the middle segment repeat its first or last token
  auto set_share = [&](int s) {
    b = 0;
    if (s >= n_row) {
      b = (int)(((uint64_t)(uint32_t)s * row_inverse) >> 32);
      s -= b * n_row;
      if (s >= n_row) {
        s -= n_row;
        ++b;
      }
    }
    blk = s;
    tok_base = s * (span - 2 * eps) - eps;
    kshare = (const char*)(kc + (int64_t)tok_base * kDc);
    if (b > 0) kshare += (int64_t)b * kc_bs * (int64_t)sizeof(bf16_t);
    first_row = tok_base < 0 ? (uint32_t)-tok_base : 0u;
    last_row = (uint32_t)(n - 1) - (uint32_t)tok_base;            // below 2^31 + 16
    last_row = last_row < (uint32_t)(span - 1) ? last_row : (uint32_t)(span - 1);
  };

  bf16x8 a[kMT][kKSteps];
  float aux[kMT][16];                    // first sweep: running row maxima.  Second: mu of the lane's rows.
  // Rows past the chunk repeat its last query: a repeated row changes no maximum, and its own results
  // are never written (first sweep) or are pushed to -inf by mu = +inf (second).  Register v of tile mt
  // belongs to row 8*(v/4) + 4*hi + v%4 of the tile.
  // Later blocks of a chunk of more than 512 queries, straight from memory (LATER == 0).  Requests and wait are one block of instructions, whose
  // registers are complete behind it; a load of the compiler's would put its wait into the tile loop, which the first block
  // runs with the share still landing.
  auto wave_has_queries = [&](int qb) { return qb * kQPerBlock + member * kQPerWave < l_c; };
  auto load_query_block = [&](int qb) {
    if (!wave_has_queries(qb)) return;    // a wave without queries only takes part in the share's loads and the barriers
    const bf16_t* q = qc + (int64_t)b * q_bs;
    const int lane = lane_now(), r = lane & 31, hi = lane >> 5;
    const bf16_t* p[kMT];
#pragma unroll
    for (int mt = 0; mt < kMT; ++mt) {
      int row = qb * kQPerBlock + member * kQPerWave + 32 * mt + r;
      row = row < l_c ? row : l_c - 1;
      p[mt] = q + (int64_t)row * kDc + hi * 8;
    }
#define ESA_LOAD4(r0, r1, r2, r3, p, at)                                                                                   \
  "global_load_dwordx4 %" r0 ", %" p ", off offset:" at "\n\tglobal_load_dwordx4 %" r1 ", %" p ", off offset:" at "+32\n\t" \
  "global_load_dwordx4 %" r2 ", %" p ", off offset:" at "+64\n\tglobal_load_dwordx4 %" r3 ", %" p ", off offset:" at "+96\n\t"
#define ESA_REGS4(mt, ks) "=&v"(a[mt][ks]), "=&v"(a[mt][(ks) + 1]), "=&v"(a[mt][(ks) + 2]), "=&v"(a[mt][(ks) + 3])
    if constexpr (kKSteps == 8)
      asm volatile(ESA_LOAD4("0", "1", "2", "3", "16", "0") ESA_LOAD4("4", "5", "6", "7", "16", "128")
                   ESA_LOAD4("8", "9", "10", "11", "17", "0") ESA_LOAD4("12", "13", "14", "15", "17", "128") "s_waitcnt vmcnt(0)"
                   : ESA_REGS4(0, 0), ESA_REGS4(0, kKSteps - 4), ESA_REGS4(1, 0), ESA_REGS4(1, kKSteps - 4)
                   : "v"(p[0]), "v"(p[1])
                   : "memory");
    else
      asm volatile(ESA_LOAD4("0", "1", "2", "3", "8", "0") ESA_LOAD4("4", "5", "6", "7", "9", "0") "s_waitcnt vmcnt(0)"
                   : ESA_REGS4(0, 0), ESA_REGS4(1, 0)
                   : "v"(p[0]), "v"(p[1])
                   : "memory");
#undef ESA_LOAD4
#undef ESA_REGS4
  };
  // Tiles 0 and 1 are in LDS once at most so many of the share's requests are outstanding.
  constexpr int kLeftFirst = kLoads - 2 / kTilesPerLoad;

  // ---- the pipeline over a share's tiles
  bf16x8 bfr[kKSteps];
  f32x16 acc0[kMT], acc1[kMT];
  // LDS byte address of this lane's fragment ks of tile nt: row r, slot (2 ks + hi) ^ swizzle(r).  The share
  // starts at a multiple of 256 bytes, so the slot's ks bits can be XORed into the address of fragment 0.
  auto swizzle = [](uint32_t row) { return kDc == 128 ? row & 15 : (row >> 1) & 7; };
  const uint32_t first_lane = __builtin_amdgcn_workitem_id_x() & 63, frag_row = first_lane & 31;
  const uint32_t frag0_at = lds_tiles + frag_row * (kDc * 2) + ((first_lane >> 5) ^ swizzle(frag_row)) * 16;
  const uint32_t colmax_at = lds_colmax + frag_row * 4;
  // A request only: its registers are the compiler's to use again from here on, as far as it knows, until a wait names them.  So every
  // request is followed, on every path, by a wait with its fragment as an operand; those of the last step by fragments_arrived.
  auto read_fragment = [&](int nt, int ks) {
    asm volatile("ds_read_b128 %0, %1" : "=v"(bfr[ks]) : "v"((frag0_at ^ (uint32_t)(ks * 32)) + (uint32_t)nt * kTileBytes));
  };
  auto fragments_arrived = [&]() {
    if constexpr (kKSteps == 8)
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(bfr[0]), "+v"(bfr[1]), "+v"(bfr[2]), "+v"(bfr[3]), "+v"(bfr[kKSteps - 4]), "+v"(bfr[kKSteps - 3]),
                   "+v"(bfr[kKSteps - 2]), "+v"(bfr[kKSteps - 1]) : : "memory");
    else
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(bfr[0]), "+v"(bfr[1]), "+v"(bfr[2]), "+v"(bfr[3]) : : "memory");
  };
  float best = -INFINITY;
  // One reduction step's share of the maximum / subtract work on a finished tile's accumulators.
  auto epilogue_part = [&](auto sweep, f32x16 (&P)[kMT], int part) {
    constexpr int kShare = 16 * kMT / kKSteps;
#pragma unroll
    for (int e = kShare * part; e < kShare * (part + 1); ++e) {
      const int mt = e / 16, v = e % 16;
      if (decltype(sweep)::value == 0) aux[mt][v] = fmaxf(aux[mt][v], P[mt][v]);
      else best = fmaxf(best, P[mt][v] - aux[mt][v]);
    }
  };
  auto epilogue_end = [&](auto sweep, int nt) {
    if (decltype(sweep)::value == 1) {
      // The other half-wave's maximum for the same token: a lane swap in the vector unit (an LDS-routed
      // shuffle would put a wait for every outstanding fragment read into each tile).  Both halves then hold
      // the column maximum and both fold it into LDS: an integer maximum, exact and order-free.
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(best), __float_as_uint(best), false, false);
      best = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
      asm volatile("ds_max_u32 %0, %1" ::"v"(colmax_at + (uint32_t)(nt + 1) * 128), "v"(ordered_key(best)) : "memory");
      best = -INFINITY;
    }
  };
  // The tile whose fragments have been read into C; meanwhile the fragments of tile `next` are fetched and the epilogue of tile
  // `prev`, held in P, is done.  The first tile's "previous tile" is a set of -inf (its column maxima go to the spare slots in
  // front of colmax); behind the last tile it is fetched again and nothing uses it: every step is the same code.
  auto step = [&](auto sweep, int next, int prev, f32x16 (&C)[kMT], f32x16 (&P)[kMT]) {
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < kKSteps; ++ks) {
      asm volatile("s_waitcnt lgkmcnt(%c1)" : "+v"(bfr[ks]) : "n"(kKSteps - 1));
#pragma unroll
      for (int mt = 0; mt < kMT; ++mt)
        C[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[mt][ks], bfr[ks], ks == 0 ? zero : C[mt], 0, 0, 0);
      read_fragment(next, ks);
      epilogue_part(sweep, P, ks);
    }
    epilogue_end(sweep, prev);
    __builtin_amdgcn_sched_barrier(0);                       // a tile's work stays inside its step
  };
  // streaming: the share is still landing.  Tiles become usable in growing groups: 0-1 behind the barrier in
  // front of the loop, then 2-3, 4-7 and 8-15, each behind a barrier in front of the odd step that fetches
  // the group's first fragments.  Early on this follows the arrival of the data; later, when the data is
  // ahead of the arithmetic, the waves run free of each other (a barrier per pair of tiles costs more than
  // it hides: of the two waves of a SIMD one gets ahead, waits, and the other cannot fill the matrix pipe
  // alone).  The number of tiles is even.
  auto next_group = [&](int nt) {                            // the wait and barrier behind step nt (0, 2 or 6)
    if (nt == 0) wait_loads_then_barrier<kLoads - 4 / kTilesPerLoad>();
    else if (nt == 2) wait_loads_then_barrier<kLoads - 8 / kTilesPerLoad>();
    else wait_loads_then_barrier<0>();
  };
  auto run_tiles = [&](auto sweep, bool streaming, bool active) {
    if (!active) {
      if (streaming)
        for (int nt = 0; nt + 2 < tpb && nt <= 6; nt += nt + 2) next_group(nt);
      return;
    }
    // Group g takes tiles g, g + n_groups, ..., an even number of them, where need be the last tile again (no maximum changes).
    const int last = tpb - 1, steps = (((tpb + n_groups - 1) >> (3 - member_bits)) + 1) & ~1;
    auto tile_of = [&](int i) { return group + i * n_groups < last ? group + i * n_groups : last; };
    const int first = tile_of(0);
#pragma unroll
    for (int ks = 0; ks < kKSteps; ++ks) read_fragment(first, ks);
#pragma unroll
    for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc1[mt][v] = -INFINITY;
    __builtin_amdgcn_s_waitcnt(0xC07F);                      // lgkmcnt(0), where the compiler sees it: not inside the loop
    int prev = -1, even = first;
    for (int nt = 0; nt < steps; nt += 2) {
      const int odd = tile_of(nt + 1);
      step(sweep, odd, prev, acc0, acc1);
      if (streaming && nt + 2 < tpb && (nt == 0 || nt == 2 || nt == 6))
        next_group(nt);
      const int next = tile_of(nt + 2);
      step(sweep, next, even, acc1, acc0);
      prev = odd;
      even = next;
    }
#pragma unroll
    for (int ks = 0; ks < kKSteps; ++ks) epilogue_part(sweep, acc1, ks);
    fragments_arrived();
    epilogue_end(sweep, prev);
  };

  // First sweep: 32 running maxima per lane, each to be reduced over the 32 lanes of a half-wave: a butterfly
  // that halves the number of values per step (31 exchanges instead of 160).  Every exchange is a vector-unit
  // move: the two 16-lane rows of the half-wave swap (v_permlane16_swap hands both directions over at once),
  // then inside a row lane i pairs with i ^ 8 (row rotation by 8), with 7 - i inside its group of eight
  // (half-row mirror), with i ^ 1 and with i ^ 2 (quad permutations).  The side a lane keeps is decided by its
  // bits 4, 3, 2, 0, 1 in that order, so lane r ends up with value (r & 28) | (r & 1) << 1 | (r >> 1) & 1.
  // A wave without queries only takes part in the barrier.
  auto flush_row_maxima = [&](int q0, bool active) {
    const int lane = lane_now(), r = lane & 31, hi = lane >> 5;
    float red[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) red[i] = aux[i / 16][i % 16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {     // rows: an even row keeps values 0..15, the odd row 16..31
      const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(red[i]), __float_as_uint(red[i + 16]), false, false);
      red[i] = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    }
#define ESA_EXCHANGE_STEP(cnt, bit, ctrl)                                                                          \
    {                                                                                                              \
      const bool upper = (r & (bit)) != 0;                                                                         \
      _Pragma("unroll") for (int i = 0; i < (cnt) / 2; ++i) {                                                      \
        const float lo_v = red[i], hi_v = red[i + (cnt) / 2];                                                      \
        const float keep = upper ? hi_v : lo_v, send = upper ? lo_v : hi_v;                                        \
        red[i] = fmaxf(keep, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(send), (ctrl), 0xF, 0xF, true))); \
      }                                                                                                            \
    }
    ESA_EXCHANGE_STEP(16, 8, 0x128)    // row_ror:8
    ESA_EXCHANGE_STEP(8, 4, 0x141)     // row_half_mirror
    ESA_EXCHANGE_STEP(4, 1, 0xB1)      // quad_perm [1,0,3,2]
    ESA_EXCHANGE_STEP(2, 2, 0x4E)      // quad_perm [2,3,0,1]
#undef ESA_EXCHANGE_STEP
    const int held = (r & 28) | ((r & 1) << 1) | ((r >> 1) & 1);
    const int mt = held / 16, v = held % 16;
    const int in_wave = 32 * mt + 8 * (v / 4) + 4 * hi + (v % 4), qrow = q0 + in_wave;
    uint32_t key = ordered_key(red[0]);
    if (n_groups > 1) {                // the groups' maxima meet in LDS: one operation per row and workgroup
      uint32_t* rows = (uint32_t*)mu_rows + member * kQPerWave + in_wave;
      rows[group * (kQPerWave << member_bits)] = key;
      __syncthreads();
      if (group > 0) return;
      for (int g = 1; g < n_groups; ++g) {
        const uint32_t other = rows[g * (kQPerWave << member_bits)];
        key = key > other ? key : other;
      }
    }
    if (!active) return;
    if (qrow < l_c)
      __hip_atomic_fetch_max(&mu_keys[((int64_t)b * kMuCopies + wg % kMuCopies) * mfma_mu_stride(l_c) + qrow], key, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
  };

  // ---- requests, in the order their results are needed (loads complete in order): query fragments, then the
  // K' share.  Instruction i of wave w fills row group 8*i + w (four or eight rows, 1 KB of
  // LDS); a lane fetches, for its slot of its row of the group, the piece that undoes the swizzle.
  // Rows past an end of the middle segment repeat its last (first) token (no maximum changes, nothing of theirs
  // is stored); shares shorter than sixteen tiles repeat their last instruction, identical data to an
  // identical place, so that the count of outstanding loads means the same in every workgroup.
  auto request_share = [&](int from, int to) {
    const int lane = lane_now();
    const uint32_t row_in_load = (64 / kPieces) * wave + lane / kPieces;
    const uint32_t piece = (lane % kPieces) ^ swizzle(row_in_load);
    const int n_loads = tpb / kTilesPerLoad;                 // tpb is even
#pragma unroll 1
    for (int i = from; i < to; ++i) {
      const int t = i < n_loads ? i : n_loads - 1;
      uint32_t row = 32 * kTilesPerLoad * t + row_in_load;
      row = row < last_row ? row : last_row;
      row = row > first_row ? row : first_row;
      __builtin_amdgcn_global_load_lds((global_void*)(kshare + (row * (uint32_t)(kDc * sizeof(bf16_t)) + piece * 16)),
                                       (lds_void*)(lds_raw + (size_t)(8 * t + wave) * 1024), 16, 0, 0);
    }
  };
  // Queries come through LDS, whole rows of 256 (128) bytes, four (eight) to an instruction, into a place of each wave's own: read as fragments, 16 bytes
  // of 32 rows to an instruction, 512 of them held the address unit for 2 us before the share's first request got through.
  constexpr int kRowsPerLoad = 64 / kPieces, kRowLoads = kQPerWave / kRowsPerLoad;
  auto request_queries = [&](int qb, uint32_t stage, int from, int to) {          // loads [from, to) of the wave's
    const int lane = lane_now();
    const char* q = (const char*)(qc + (int64_t)b * q_bs);
#pragma unroll 1
    for (int i = from; i < to; i += n_groups) {
      const uint32_t mine = kRowsPerLoad * i + lane / kPieces;
      uint32_t row = qb * kQPerBlock + member * kQPerWave + mine;
      row = row < (uint32_t)l_c ? row : (uint32_t)l_c - 1;
      __builtin_amdgcn_global_load_lds((global_void*)(q + (row * (uint32_t)(kDc * sizeof(bf16_t)) + ((lane % kPieces) ^ swizzle(mine)) * 16)),
                                       (lds_void*)(lds_raw + stage + 1024 * i), 16, 0, 0);
    }
  };
  auto read_tile = [&](bf16x8 (&f)[kKSteps], uint32_t at) {    // requests and wait in one block: the registers are complete behind it
    at += frag0_at;
    if constexpr (kKSteps == 8)
      asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %11\n\t"
                   "ds_read_b128 %4, %12\n\tds_read_b128 %5, %13\n\tds_read_b128 %6, %14\n\tds_read_b128 %7, %15\n\ts_waitcnt lgkmcnt(0)"
                   : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[kKSteps - 4]),
                     "=&v"(f[kKSteps - 3]), "=&v"(f[kKSteps - 2]), "=&v"(f[kKSteps - 1])
                   : "v"(at), "v"(at ^ 32u), "v"(at ^ 64u), "v"(at ^ 96u), "v"(at ^ 128u), "v"(at ^ 160u), "v"(at ^ 192u), "v"(at ^ 224u)
                   : "memory");
    else
      asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\ts_waitcnt lgkmcnt(0)"
                   : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3])
                   : "v"(at), "v"(at ^ 32u), "v"(at ^ 64u), "v"(at ^ 96u)
                   : "memory");
  };
  static_assert(kMT == 2, "two tiles of queries");
  auto read_queries = [&](uint32_t stage) {
    asm volatile("" : "+s"(stage));                            // (its sixteen addresses would be kept from block to block)
    read_tile(a[0], stage);
    read_tile(a[1], stage + kTileBytes);
  };
  // A block of queries behind the first: requested (by halves the first one) while the block before is at work, and taken in.
  auto later_stage = [&]() { return (uint32_t)(later_at + member * (kMT * kTileBytes / (LATER == 0 ? 1 : LATER))); };
  auto request_later = [&](int qb) { request_queries(qb, later_stage(), 0, kRowLoads / (LATER == 0 ? 1 : LATER)); };
  auto take_later = [&](int qb) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // a wave reads what it has requested itself
    if constexpr (LATER == 1) {
      read_queries(later_stage());
    } else {
      uint32_t stage = later_stage();
      asm volatile("" : "+s"(stage));
      read_tile(a[0], stage);
      request_queries(qb, stage - 1024 * (kRowLoads / 2), kRowLoads / 2, kRowLoads);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      read_tile(a[1], stage);
    }
  };
  // Brings in the share at hand and, where `queries`, the first block of them.  When it returns the queries are in registers and, with one
  // group, tiles 0 and 1 in LDS; with several all tiles.
  auto begin = [&](bool queries) {
    const int before = queries ? before_queries : kMaxTilesPerBlock;
    const uint32_t stage = (uint32_t)((before + member * kMT) * kTileBytes);
    if (queries) request_queries(0, stage, group, kRowLoads);
    const int first_loads = queries && before < tpb ? before / kTilesPerLoad : kLoads;
    request_share(0, first_loads);
    if (queries) {
      if (n_groups == 1) {                                     // a wave reads what it has requested itself
        if (first_loads == kLoads) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kLoads) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 / kTilesPerLoad) : "memory");
      } else {
        wait_loads_then_barrier<0>();
      }
      read_queries(stage);
    }
    if (first_loads < kLoads) {
      wait_loads_then_barrier<2 / kTilesPerLoad>();            // tiles 0 and 1 of four; every wave has its queries
      request_share(first_loads, kLoads);
      if (n_groups > 1) wait_loads_then_barrier<0>();
    } else if (n_groups == 1) {
      wait_loads_then_barrier<kLeftFirst>();                   // tiles 0 and 1
    } else {
      wait_loads_then_barrier<0>();                            // all tiles; every wave has its queries
    }
  };

  int in_regs = 0, in_regs_row = -1;     // the query block in registers, and whose
  // One sweep over the share at hand, all query blocks (chunks longer than 512 tokens have several): first the one in registers.
  auto sweep_share = [&](auto sweep, bool streaming) {
    const int n_blocks = (l_c + kQPerBlock - 1) / kQPerBlock;
    auto next_block = [&]() { return in_regs + 1 < n_blocks ? in_regs + 1 : 0; };
    for (int i = 0; i < n_blocks; ++i) {
      if (i > 0) {
        in_regs = next_block();
        if constexpr (LATER == 0) load_query_block(in_regs);
        else if (wave_has_queries(in_regs)) take_later(in_regs);
      }
      // (behind a landing share: its waits count loads, and would wait for the share's last ones as well)
      const bool landing = streaming && i == 0, more = LATER != 0 && i + 1 < n_blocks && wave_has_queries(next_block());
      if (more && !landing) request_later(next_block());
      const bool active = wave_has_queries(in_regs);
      if (decltype(sweep)::value == 0) {
#pragma unroll
        for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
          for (int v = 0; v < 16; ++v) aux[mt][v] = -INFINITY;
      } else if (active) {
        const int lane = lane_now(), hi = lane >> 5, row = in_regs * kQPerBlock + member * kQPerWave + lane;      // < mu_stride
        const int mu_stride = mfma_mu_stride(l_c);
        uint32_t* p = mu_keys + (int64_t)b * kMuCopies * mu_stride + row;
        uint32_t key[kMuCopies];
#pragma unroll
        for (int c = 0; c < kMuCopies; ++c) key[c] = __hip_atomic_load(p + c * mu_stride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int c = 1; c < kMuCopies; ++c) key[0] = key[0] > key[c] ? key[0] : key[c];
        float* mine = mu_rows + wave * kQPerWave;
        mine[lane] = row < l_c ? ordered_key_to_f32(key[0]) : INFINITY;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int mt = 0; mt < kMT; ++mt)
#pragma unroll
          for (int g4 = 0; g4 < 4; ++g4) {
            const f32x4 m4 = *(const f32x4*)(mine + 32 * mt + 8 * g4 + 4 * hi);
#pragma unroll
            for (int e = 0; e < 4; ++e) aux[mt][4 * g4 + e] = m4[e];
          }
      }
      run_tiles(sweep, landing && n_groups == 1, active);
      if (more && landing) request_later(next_block());
      if (decltype(sweep)::value == 0 && (active || n_groups > 1)) flush_row_maxima(in_regs * kQPerBlock + member * kQPerWave, active);
    }
  };

  // ---- first sweep, and the wait
  int share = wg, own = wg, at_hand;
  bool waiting = false;
  uint64_t give_up = 0;
  for (;;) {
    scalars_afresh();
    set_share(share);
    at_hand = share;
    const bool queries = in_regs_row != b;
    begin(queries);
    if (queries) in_regs = 0;
    in_regs_row = b;
    sweep_share(std::integral_constant<int, 0>(), true);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // this wave's maxima are in mu_keys
    __syncthreads();
    const int lane = lane_now(), tid = 64 * wave + lane;
    uint32_t* my_marks = marks + wg % kMuCopies * mark_words(n_shares);
    if (tid < kMuCopies)
      __hip_atomic_fetch_or(&marks[tid * mark_words(n_shares) + share / kMarksPerWord * kMarkStride], 1u << (share % kMarksPerWord), __ATOMIC_RELAXED,
                            __HIP_MEMORY_SCOPE_AGENT);
    if (!waiting && share + n_wg < n_shares) {
      own = share += n_wg;
      continue;
    }
    for (int i = tid; i < span + 32; i += kThreads) colmax[i] = kOrderedKeyOfMinusInf;
    for (int i = tid; i < kRadixBins; i += kThreads) digit_hist[i] = 0u;
    if (wave == 0) {
      if (!waiting) {
        const uint64_t now = __builtin_amdgcn_s_memrealtime();     // 10 ns
        give_up = now + (patience ? patience - 1 : (now - started) + kPatience);
      }
      int missing = -1;
      auto marks_from = [&](int c) {                              // the lane's word: the bits of shares
        const int here = n_shares - c - lane * kMarksPerWord;
        return here >= kMarksPerWord ? (1u << kMarksPerWord) - 1u : here > 0 ? (1u << here) - 1u : 0u;
      };
      uint32_t open = marks_from(0);
      for (int c = 0; c < n_shares;) {                            // 64 words of marks at a time; a word that is complete is not read again
        const int of = c + lane * kMarksPerWord;
        if (open != 0u) open &= ~__hip_atomic_load(&my_marks[of / kMarksPerWord * kMarkStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t lanes = __ballot(open != 0u);
        if (lanes == 0) {
          c += 64 * kMarksPerWord;
          open = marks_from(c);
        } else if (__builtin_amdgcn_s_memrealtime() >= give_up) {
          // lanes in turn from one of the workgroup's own: those that give up together take different shares
          const int turn = (wg * 29) & 63;
          const uint64_t turned = (lanes >> turn) | (turn ? lanes << (64 - turn) : 0);
          const int l = (__ffsll((long long)turned) - 1 + turn) & 63;
          missing = __builtin_amdgcn_readlane(of + __ffs((int)open) - 1, l);
          break;
        } else {
          __builtin_amdgcn_s_sleep(1);
        }
      }
      if (lane == 0) *todo = missing;
    }
    __syncthreads();
    const int missing = __builtin_amdgcn_readfirstlane(*todo);
    if (missing < 0) break;
    waiting = true;
    share = missing;
    __syncthreads();                                              // *todo is read
  }

  // ---- second sweep: own shares, the last one first
  for (;; own -= n_wg) {
    scalars_afresh();
    if (own != at_hand) {
      set_share(own);
      const bool queries = in_regs_row != b;
      begin(queries);
      if (queries) in_regs = 0;
      in_regs_row = b;
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      const int tid = 64 * wave + lane_now();
      for (int i = tid; i < span + 32; i += kThreads) colmax[i] = kOrderedKeyOfMinusInf;
      for (int i = tid; i < kRadixBins; i += kThreads) digit_hist[i] = 0u;
      __syncthreads();
    }
    sweep_share(std::integral_constant<int, 1>(), false);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // this wave's column maxima are in LDS
    __syncthreads();
    const int tid = 64 * wave + lane_now();
    for (int i0 = 0; i0 < span; i0 += kThreads) {          // whole waves stay in step for hist_add
      const int i = i0 + tid;
      const int64_t m = (int64_t)tok_base + i;
      const bool ok = i >= eps && i < span - eps && m < n;
      uint32_t key = ok ? colmax[32 + i] : 0u;
      if (ok)                              // (a repeated token only meets windows that hold it)
        for (int d = 1; d <= eps; ++d) {
          const uint32_t left = colmax[32 + i - d], right = colmax[32 + i + d];
          key = key > left ? key : left;
          key = key > right ? key : right;
        }
      if (ok) score[(int64_t)b * score_bs + m] = ordered_key_to_f32(key);
      if (first_hist) hist_add(digit_hist, ok, score_digit(key));
    }
    if (first_hist) {
      __syncthreads();
      hist_flush(first_hist + (int64_t)b * first_hist_bs, digit_hist, blk, tid, kThreads);
    }
    if (own < n_wg) break;
    at_hand = -1;
    __syncthreads();                                       // the LDS is free for the next share
  }
}

// In front of the sweeps: mu_keys and the marks, and the selection's histograms, cleared.  (A kernel of its own, 2 us for 77 tokens, 4 to 5 for 512 and 1024: nothing
// that a call finds in its workspace says whether another workgroup has cleared it already.)
__global__ __launch_bounds__(256) void score_sweeps_clear(uint4* __restrict__ own, int64_t n_own, uint32_t* __restrict__ hists,
                                                          int64_t hists_bs, int batch) {
  const int64_t i = (int64_t)__builtin_amdgcn_workgroup_id_x() * 256 + __builtin_amdgcn_workitem_id_x();
  const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
  if (i < n_own) {
    own[i] = zero;
    return;
  }
  constexpr int kRow = kHistWords / 4;
  const int64_t j = i - n_own;
  if (hists && j < (int64_t)kRow * batch) *(uint4*)(hists + j / kRow * hists_bs + j % kRow * 4) = zero;
}

// ------------------------------------------------------------------------------------------ decode (l_c = 1)
// One current token: S is a matrix-vector product over the whole compressed-key cache, pure HBM
// streaming.  LPR lanes share a K' row (16 bytes each), so a wave reads 64*16 contiguous bytes per
// step; a workgroup covers 64 or 512 rows.  Writes S and the workgroup's maximum of it (no atomics: thousands of
// workgroups folding into one word serialise in L2); score_finish then reduces those maxima to mu,
// every workgroup for itself, and forms F = S - mu.
// What bounds it is HBM.  Workgroups of 512 rows, eight requests a lane in flight, non-temporal (see streams), each row whole cache lines of one
// instruction; the scores leave by way of LDS, 256 bytes a wave and non-temporally too (four lanes' words at a time cost 18 of 172 us, 10
// now).  Sixteen rows of 260 thousand (1.07 GB) 201.5 -> 169.6 us, 6.3 TB/s (with the loads behind their bounds checks and stores as they came
// 256 rows a workgroup had 5.3); one row out of HBM 17.9 -> 13.1, of 180 thousand 15.4 -> 10.2.
// Few rows in all give a compute unit too few requests that way, and the last-level cache often has them still: 64 rows a workgroup, ordinary
// loads.  512 for one row of more than 196608, whose list of partial maxima each of score_finish's workgroups goes through (4.6 us with 64-row
// workgroups, 4.2), and for more rows than that in all from 72 MB on, where at most an eighth of the work is padding.  64 / 512 rows, us:
//                           score and selection, one input again and again, three in turn, twelve      the step, attention between two scores
//    1 x 165 thousand, d' 128   42 MB   22.1 / 22.9   22.3 / 24.2   23.4 / 24.0
//    1 x 262           d'  64   34 MB   20.9 / 20.6   22.2 / 21.1   23.5 / 22.0
//    1 x 262           d' 128   67 MB   26.2 / 25.8   26.2 / 25.8   28.2 / 26.9
//    1 x 262           d' 256  134 MB   36.0 / 36.8   39.5 / 38.0   39.8 / 38.9
//    8 x  30           d' 128   61 MB   25.3 / 25.9   24.8 / 26.5   27.3 / 27.1                           58.4 / 60.7
//   16 x  32           d'  64   66 MB   27.3 / 29.0   27.4 / 29.7   29.2 / 29.7                           62.3 / 65.2
//    4 x 150           d'  64   77 MB                                                                     48.4 / 47.1
//    2 x 190           d' 128   97 MB                                                                     51.3 / 49.0
//    8 x  60           d' 128  123 MB   35.2 / 37.4   38.7 / 38.2   39.3 / 38.8                           73.6 / 71.8
//    2 x 150           d' 256  154 MB                                                                     60.8 / 62.7
//   12 x 100           d' 128  307 MB                                                                    121.6 / 115.5
// (A single layer whose K' a cache keeps from one call to the next would rather have 64 up to 270 MB: 16 x 60 thousand 54.5 / 61.7, 1 x 290 of d' 256, 148 MB, score
// and selection 38.5 / 43.6; the same with eight inputs in turn 50.8 / 45.1.)
// Sequences that share one K' read it from a cache all but once: 8 x 130 thousand 22.0 / 46.5, five queries each of 4 x 130 27.4 / 30.9.
__host__ inline bool shared_keys(int batch, int64_t kc_bs) { return batch > 1 && kc_bs == 0; }
__host__ inline bool gemv_streams(int64_t n, int batch, int d_c, int64_t kc_bs) {
  const int64_t rows = n * batch;
  if (shared_keys(batch, kc_bs)) return false;
  return n > 196608 || (rows > 196608 && rows * d_c * (int64_t)sizeof(bf16_t) >= ((int64_t)72 << 20) && (n + 511) / 512 * 512 * 8 <= n * 9);
}
// grids of the passes over the scores (host and device agree on them; the kernels do not ask the dispatch packet)
__host__ __device__ inline int maxpool_blocks(int64_t n) { return (int)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096); }

// Sum over groups of LPR consecutive lanes (LPR = 8, 16, 32) with DPP moves; every lane gets the total.
template <int LPR>
__device__ __forceinline__ float lanes_sum(float v) {
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true));    // quad_perm [1,0,3,2]
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, true));    // quad_perm [2,3,0,1]
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xF, 0xF, true));   // row_half_mirror
  if (LPR >= 16) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xF, 0xF, true));   // row_mirror
  if (LPR >= 32) v += __shfl_xor(v, 16, 64);
  return v;
}

// Maximum over the 16 lanes of a DPP row; every lane receives it.
__device__ __forceinline__ float lanes_max16(float v) {
  v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, true)));
  v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, true)));
  v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xF, 0xF, true)));
  return fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xF, 0xF, true)));
}

// THREADS, and STEPS rows to each LPR of them.
template <int LPR, int THREADS, int STEPS>
__global__ __launch_bounds__(THREADS) void score_gemv_bf16(const bf16_t* __restrict__ qc, const bf16_t* __restrict__ kc,
                                                           int64_t m_lo, int64_t n, float* __restrict__ part,
                                                           float* __restrict__ raw, int64_t q_bs, int64_t kc_bs,
                                                           int64_t raw_bs, uint32_t* __restrict__ hists, int64_t hists_bs) {
  constexpr int kDcv = LPR * 8;
  constexpr int kRowsPerStep = THREADS / LPR;
  constexpr int kRows = kRowsPerStep * STEPS;
  constexpr int kAhead = STEPS < 8 ? STEPS : 8;            // rows of a lane in flight
  constexpr bool kStream = THREADS == 512;
  const int n_wg = (int)((n + kRows - 1) / kRows);         // workgroups per batch entry
  if ((int)__builtin_amdgcn_workgroup_id_x() >= n_wg) return;      // (the launch's grid is rounded up for shared_keys)
  __shared__ float red[THREADS / 64];
  __shared__ float staged[kRows];
  const int b = __builtin_amdgcn_workgroup_id_y(), tid = __builtin_amdgcn_workitem_id_x();
  if (hists)       // the selection's histograms, zeroed here for the pass that follows
    for (int i = __builtin_amdgcn_workgroup_id_x() * THREADS + tid; i < kHistWords; i += n_wg * THREADS)
      hists[(int64_t)b * hists_bs + i] = 0u;
  const bf16_t* kmid = kc + (int64_t)b * kc_bs + m_lo * (int64_t)kDcv;
  const int sub = tid % LPR, grp = tid / LPR;
  float qv[8];
  {
    const uint4 u = *(const uint4*)(qc + (int64_t)b * q_bs + sub * 8);
    qv[0] = __uint_as_float(u.x << 16); qv[1] = __uint_as_float(u.x & 0xFFFF0000u);
    qv[2] = __uint_as_float(u.y << 16); qv[3] = __uint_as_float(u.y & 0xFFFF0000u);
    qv[4] = __uint_as_float(u.z << 16); qv[5] = __uint_as_float(u.z & 0xFFFF0000u);
    qv[6] = __uint_as_float(u.w << 16); qv[7] = __uint_as_float(u.w & 0xFFFF0000u);
  }
  float best = -INFINITY;
  const int64_t row0 = (int64_t)__builtin_amdgcn_workgroup_id_x() * kRows;
#pragma unroll
  for (int it0 = 0; it0 < STEPS; it0 += kAhead) {
    uint4 u[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {                     // rows past the end repeat the last one: no maximum changes
      const int64_t row = row0 + (it0 + i) * kRowsPerStep + grp;
      u[i] = load16<kStream>(kmid + (row < n ? row : n - 1) * kDcv + sub * 8);
    }
#pragma unroll
    for (int i = 0; i < kAhead; ++i) {
      float s = qv[0] * __uint_as_float(u[i].x << 16);
      s = __fmaf_rn(qv[1], __uint_as_float(u[i].x & 0xFFFF0000u), s);
      s = __fmaf_rn(qv[2], __uint_as_float(u[i].y << 16), s);
      s = __fmaf_rn(qv[3], __uint_as_float(u[i].y & 0xFFFF0000u), s);
      s = __fmaf_rn(qv[4], __uint_as_float(u[i].z << 16), s);
      s = __fmaf_rn(qv[5], __uint_as_float(u[i].z & 0xFFFF0000u), s);
      s = __fmaf_rn(qv[6], __uint_as_float(u[i].w << 16), s);
      s = __fmaf_rn(qv[7], __uint_as_float(u[i].w & 0xFFFF0000u), s);
      s = lanes_sum<LPR>(s);
      if (sub == 0) staged[(it0 + i) * kRowsPerStep + grp] = s;
      best = fmaxf(best, s);
    }
  }
  best = wave_max(best);
  if ((tid & 63) == 0) red[tid >> 6] = best;
  __syncthreads();
  for (int i = tid; i < kRows; i += THREADS)
    if (row0 + i < n) {
      float* to = &raw[(int64_t)b * raw_bs + row0 + i];
      if (kStream) __builtin_nontemporal_store(staged[i], to);
      else *to = staged[i];
    }
  if (tid == 0) {
#pragma unroll
    for (int w = 1; w < THREADS / 64; ++w) best = fmaxf(best, red[w]);
    part[(int64_t)b * n_wg + __builtin_amdgcn_workgroup_id_x()] = best;
  }
}

// Two to sixteen current tokens: one pass over K' on the matrix cores, S stored.  v_mfma_f32_16x16x32_bf16, A rows are
// tokens, B columns queries (rows past the chunk repeat its last one): a lane owns four consecutive tokens of one query,
// a 16-byte store.  K' is the stream to keep moving, in whole cache lines: a wave requests its 64 tokens' rows at once, a lane 16 bytes of
// each, and passes them through 4 KB of LDS of its own, sixteen rows at a time, into fragments.  Read as fragments, half a line to an instruction, the rows could
// not be fetched non-temporally (17.8 -> 24.9 us).  From kFewStreamBytes on they are: four sequences of 100k tokens (102 MB), five queries,
// out of HBM 22.2 -> 21.0 us; less is often still in the last-level cache (eight of 30k, 61 MB, ordinary loads 12.0 / 14.4, non-temporal 14.7 / 14.0 with three inputs
// in turn / eight; two of 60k 7.7 / 8.5, 8.1 / 8.1).  Each of the two sweeps took 35 us for the 102 MB.
constexpr int kFewQueries = 16;
constexpr int kFewTok = 256;             // tokens per workgroup
constexpr int64_t kFewStreamBytes = (int64_t)64 << 20;
template <int DC, bool STREAM>
__global__ __launch_bounds__(256) void score_few_bf16(const bf16_t* __restrict__ qc, int l_c, const bf16_t* __restrict__ kc,
                                                      int64_t m_lo, int64_t n, float* __restrict__ part, float* __restrict__ S,
                                                      int64_t s_ld, int64_t s_bs, int64_t q_bs, int64_t kc_bs, int n_wg,
                                                      uint32_t* __restrict__ hists, int64_t hists_bs) {
  constexpr int kKS = DC / 32, kTiles = kFewTok / 64;
  constexpr int kPieces = DC / 8, kLoadRows = 64 / kPieces;                  // 16-byte pieces of a row, rows of a load instruction
  constexpr int kTileLoads = 16 / kLoadRows;
  __shared__ __attribute__((aligned(256))) unsigned char staged[4][16 * DC * 2];
  __shared__ float red[4][kFewQueries];
  const int b = __builtin_amdgcn_workgroup_id_y(), blk = __builtin_amdgcn_workgroup_id_x(), tid = __builtin_amdgcn_workitem_id_x();
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), r = lane & 15, q4 = lane >> 4;
  const bf16_t* k = kc + (int64_t)b * kc_bs + m_lo * (int64_t)DC + lane % kPieces * 8;
  const bf16_t* qp = qc + (int64_t)b * q_bs + (int64_t)(r < l_c ? r : l_c - 1) * DC + q4 * 8;
  bf16x8 qf[kKS];
#pragma unroll
  for (int ks = 0; ks < kKS; ++ks) qf[ks] = *(const bf16x8*)(qp + 32 * ks);
  const int64_t tok0 = (int64_t)blk * kFewTok + wave * (16 * kTiles);
  uint4 kv[kTiles][kTileLoads];
#pragma unroll
  for (int t = 0; t < kTiles; ++t)
#pragma unroll
    for (int i = 0; i < kTileLoads; ++i) {
      const int64_t tok = tok0 + 16 * t + kLoadRows * i + lane / kPieces;
      kv[t][i] = load16<STREAM>(k + (tok < n ? tok : n - 1) * DC);                // repeats the last token: no maximum changes
    }
  if (hists)       // the selection's histograms, zeroed here for the pass that follows
    for (int i = blk * 256 + tid; i < kHistWords; i += n_wg * 256) hists[(int64_t)b * hists_bs + i] = 0u;
  // rows land in LDS with their pieces swizzled, so that neither the writes nor the fragment reads meet in a bank
  auto slot = [&](uint32_t row, uint32_t piece) { return staged[wave] + row * (DC * 2) + ((piece ^ (DC == 128 ? row & 15 : (row >> 1) & 7)) << 4); };
  float best = -INFINITY;
  f32x4 acc[kTiles];
#pragma unroll
  for (int t = 0; t < kTiles; ++t) {
#pragma unroll
    for (int i = 0; i < kTileLoads; ++i) *(uint4*)slot(kLoadRows * i + lane / kPieces, lane % kPieces) = kv[t][i];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");                   // (a wave's LDS operations complete in order)
    bf16x8 kf[kKS];
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) kf[ks] = *(const bf16x8*)slot(r, 4 * ks + q4);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    acc[t] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks], qf[ks], acc[t], 0, 0, 0);
    best = fmaxf(fmaxf(best, acc[t][0]), fmaxf(fmaxf(acc[t][1], acc[t][2]), acc[t][3]));
  }
#pragma unroll
  for (int t = 0; t < kTiles; ++t) {
    const int64_t tok = tok0 + 16 * t + 4 * q4;
    if (r < l_c && tok < s_ld) *(f32x4*)(S + (int64_t)b * s_bs + (int64_t)r * s_ld + tok) = acc[t];      // s_ld: n rounded up to whole tiles
  }
  best = fmaxf(best, __shfl_xor(best, 16, 64));
  best = fmaxf(best, __shfl_xor(best, 32, 64));
  if (lane < kFewQueries) red[wave][lane] = best;
  __syncthreads();
  if (tid < l_c) part[((int64_t)b * n_wg + blk) * l_c + tid] = fmaxf(fmaxf(red[0][tid], red[1][tid]), fmaxf(red[2][tid], red[3][tid]));
}

// The same for every storage type, d_c and alignment: a workgroup computes S for 64 tokens (one per lane) and 32 queries (eight per
// wave), both in LDS as fp32 rows (the queries' reads are broadcasts), fp32 FMAs in ascending order (of fp32 rows in dot_fixed's).
constexpr int kStoreQ = 32;
constexpr int kTileQ = 64;
__host__ __device__ inline int store_ld(int d_c) { return d_c + 4; }       // d_c is a multiple of 16: rows 16-byte aligned, spread over the banks
template <typename T>
__global__ __launch_bounds__(256) void score_store_fma(const T* __restrict__ qc, int l_c, const T* __restrict__ kc, int64_t m_lo,
                                                       int64_t n, int d_c, float* __restrict__ part, float* __restrict__ S,
                                                       int64_t s_ld, int64_t s_bs, int64_t q_bs, int64_t kc_bs, int n_wg,
                                                       uint32_t* __restrict__ hists, int64_t hists_bs) {
  extern __shared__ __attribute__((aligned(16))) float smem[];               // [kGTok][ld] tokens, [kStoreQ][ld] queries
  const int ld = store_ld(d_c);
  float* qs = smem + kGTok * ld;
  const int b = __builtin_amdgcn_workgroup_id_z(), blk = __builtin_amdgcn_workgroup_id_x(), tid = __builtin_amdgcn_workitem_id_x();
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t m0 = (int64_t)blk * kGTok;
  const int cg0 = (int)__builtin_amdgcn_workgroup_id_y() * kStoreQ, c0 = cg0 + wave * (kStoreQ / 4);
  const T* k = kc + (int64_t)b * kc_bs + m_lo * (int64_t)d_c;
  const T* q = qc + (int64_t)b * q_bs;
  constexpr int kAtOnce = 12;                          // loads in flight per thread: all of them at d_c = 32
  for (int e0 = tid; e0 < (kGTok + kStoreQ) * d_c; e0 += 256 * kAtOnce) {
    float v[kAtOnce];
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u) {
      const int e = e0 + 256 * u, t = e / d_c, i = e % d_c;
      // past the end: the last token, the last query again
      const T* from = t < kGTok ? k + (m0 + t < n ? m0 + t : n - 1) * (int64_t)d_c
                                : q + (int64_t)(cg0 + t - kGTok < l_c ? cg0 + t - kGTok : l_c - 1) * d_c;
      v[u] = load_f32(from + i);
    }
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u) {
      const int e = e0 + 256 * u;
      if (e < (kGTok + kStoreQ) * d_c) smem[e / d_c * ld + e % d_c] = v[u];
    }
  }
  if (hists && __builtin_amdgcn_workgroup_id_y() == 0)
    for (int i = blk * 256 + tid; i < kHistWords; i += n_wg * 256) hists[(int64_t)b * hists_bs + i] = 0u;
  __syncthreads();
  float acc[kStoreQ / 4] = {};
  const float* qrow = qs + wave * (kStoreQ / 4) * ld;
  if constexpr (sizeof(T) == 4) {                      // the order of dot_fixed
    float odd[kStoreQ / 4] = {};
    for (int i = 0; i < d_c; i += 16) {
      float4 kv[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) kv[p] = *(const float4*)&smem[lane * ld + i + 4 * p];
      auto eight = [](const float4& q0, const float4& q1, const float4& k0, const float4& k1, float s) {
        s = __fmaf_rn(q1.x, k1.x, __fmaf_rn(q0.x, k0.x, s));
        s = __fmaf_rn(q1.y, k1.y, __fmaf_rn(q0.y, k0.y, s));
        s = __fmaf_rn(q1.z, k1.z, __fmaf_rn(q0.z, k0.z, s));
        return __fmaf_rn(q1.w, k1.w, __fmaf_rn(q0.w, k0.w, s));
      };
#pragma unroll
      for (int j = 0; j < kStoreQ / 4; ++j) {
        const float4* qv = (const float4*)&qrow[j * ld + i];
        acc[j] = eight(qv[0], qv[1], kv[0], kv[1], acc[j]);
        odd[j] = eight(qv[2], qv[3], kv[2], kv[3], odd[j]);
      }
    }
#pragma unroll
    for (int j = 0; j < kStoreQ / 4; ++j) acc[j] += odd[j];
  } else {
    for (int i = 0; i < d_c; i += 4) {
      const float4 kv = *(const float4*)&smem[lane * ld + i];
#pragma unroll
      for (int j = 0; j < kStoreQ / 4; ++j) {
        const float4 qv = *(const float4*)&qrow[j * ld + i];
        acc[j] = __fmaf_rn(qv.x, kv.x, acc[j]);
        acc[j] = __fmaf_rn(qv.y, kv.y, acc[j]);
        acc[j] = __fmaf_rn(qv.z, kv.z, acc[j]);
        acc[j] = __fmaf_rn(qv.w, kv.w, acc[j]);
      }
    }
  }
#pragma unroll
  for (int j = 0; j < kStoreQ / 4; ++j) {
    if (c0 + j >= l_c) break;
    if (m0 + lane < s_ld) S[(int64_t)b * s_bs + (int64_t)(c0 + j) * s_ld + m0 + lane] = acc[j];
    const float mx = wave_max(acc[j]);
    if (lane == 0) part[((int64_t)b * n_wg + blk) * l_c + c0 + j] = mx;
  }
}

// The same for fp32 rows that are 16-byte aligned, on the matrix cores: v_mfma_f32_32x32x2_f32, exact products and fp32 sums, A rows are
// tokens, B columns queries; a lane's sixteen bytes of a row feed four instructions (lanes 32 apart hold neighbouring pieces).  A wave owns
// 32 tokens x 32 queries and takes its fragments straight from memory: a small layer's call is round trips, and staging through LDS with
// its index arithmetic, 72 LDS reads a wave and a butterfly per query made it 6.8 us for 128 queries over 1632 tokens of d_c 32, 4.2 now (five
// queries over 940: 6.4 -> 3.8).  dot_fixed's order.
__global__ __launch_bounds__(256) void score_store_f32(const float* __restrict__ qc, int l_c, const float* __restrict__ kc, int64_t m_lo,
                                                       int64_t n, int d_c, float* __restrict__ part, float* __restrict__ S,
                                                       int64_t s_ld, int64_t s_bs, int64_t q_bs, int64_t kc_bs, int n_wg,
                                                       uint32_t* __restrict__ hists, int64_t hists_bs) {
  __shared__ float red[2][kTileQ];
  const int b = __builtin_amdgcn_workgroup_id_z(), blk = __builtin_amdgcn_workgroup_id_x(), tid = __builtin_amdgcn_workitem_id_x();
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), r = lane & 31, hi = lane >> 5;
  const int64_t tok0 = (int64_t)blk * kGTok + (wave & 1) * 32;
  const int c0 = (int)__builtin_amdgcn_workgroup_id_y() * kTileQ + (wave >> 1) * 32, c = c0 + r;
  // past the end: the last token, the last query again
  const float* kp = kc + (int64_t)b * kc_bs + (m_lo + (tok0 + r < n ? tok0 + r : n - 1)) * (int64_t)d_c + 4 * hi;
  const float* qp = qc + (int64_t)b * q_bs + (int64_t)(c < l_c ? c : l_c - 1) * d_c + 4 * hi;
  f32x16 even, odd;                                        // two chains, each of half the sum
#pragma unroll
  for (int v = 0; v < 16; ++v) even[v] = odd[v] = 0.f;
  constexpr int kAhead = 4;                                // steps of eight dimensions in flight: all of them at d_c = 32
  const int steps = d_c / 8;                               // even
  for (int j0 = 0; j0 < steps; j0 += kAhead) {
    f32x4 k4[kAhead], q4[kAhead];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const int at = 8 * (j0 + j < steps ? j0 + j : j0);
      k4[j] = *(const f32x4*)(kp + at);
      q4[j] = *(const f32x4*)(qp + at);
    }
#pragma unroll
    for (int j = 0; j < kAhead; j += 2) {
      if (j0 + j >= steps) break;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        even = __builtin_amdgcn_mfma_f32_32x32x2f32(k4[j][e], q4[j][e], even, 0, 0, 0);
        odd = __builtin_amdgcn_mfma_f32_32x32x2f32(k4[j + 1][e], q4[j + 1][e], odd, 0, 0, 0);
      }
    }
  }
  if (hists && __builtin_amdgcn_workgroup_id_y() == 0)
    for (int i = blk * 256 + tid; i < kHistWords; i += n_wg * 256) hists[(int64_t)b * hists_bs + i] = 0u;
  even += odd;
  float best = -INFINITY;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const f32x4 s4 = {even[4 * g], even[4 * g + 1], even[4 * g + 2], even[4 * g + 3]};
    best = fmaxf(best, fmaxf(fmaxf(s4[0], s4[1]), fmaxf(s4[2], s4[3])));
    if (c < l_c) *(f32x4*)(S + (int64_t)b * s_bs + (int64_t)c * s_ld + tok0 + 8 * g + 4 * hi) = s4;      // s_ld: whole blocks of 64 tokens
  }
  const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(best), __float_as_uint(best), false, false);
  best = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
  if (hi == 0) red[wave & 1][(wave >> 1) * 32 + r] = best;
  __syncthreads();
  const int cc = (int)__builtin_amdgcn_workgroup_id_y() * kTileQ + tid;
  if (tid < kTileQ && cc < l_c) part[((int64_t)b * n_wg + blk) * l_c + cc] = fmaxf(red[0][tid], red[1][tid]);
}

// F[m] = max_c (S[c][m] - mu_c), mu_c = the largest of the n_part partial maxima of query c ([n_part][l_c]), found by
// every workgroup for itself; pooled over +-eps (<= kTailMaxEps) when asked; with first_hist given also the histogram
// of the results' first digits.  SPLIT = 1 (up to sixteen queries): a workgroup owns `sub` tiles of 1024 tokens, four per
// thread, the ones that the selection's workgroup of the same number reads next (written and read on the same XCD; with
// many rows several tiles, so that fewer workgroups reduce the partial maxima and flush a histogram).
// SPLIT = 4: 64 tokens (pooled ones at the ends only feed their neighbours), the queries shared out over the waves.
constexpr int kFinishMaxQueries = 4096;
template <int SPLIT, bool POOL, bool ONE = false>
__global__ __launch_bounds__(256) void score_finish(const float* __restrict__ S, int64_t s_ld, int64_t s_bs, int64_t n,
                                                    const float* __restrict__ part, int n_part, int l_c, int eps_arg, int sub,
                                                    float* __restrict__ score, int64_t score_bs,
                                                    uint32_t* __restrict__ first_hist, int64_t first_hist_bs) {
  const int eps = POOL ? eps_arg : 0;
  constexpr int kPer = POOL ? 5 : 4;                        // SPLIT = 1: tokens of a thread, the last one of the pooling margin
  constexpr int kAhead = ONE ? 1 : 4;                       // queries whose scores are in flight together
  constexpr int kTok = SPLIT == 1 ? 1024 : 64;
  __shared__ float mu[SPLIT == 1 ? kFewQueries : kFinishMaxQueries];
  __shared__ float red[256];
  __shared__ float tile[SPLIT == 1 ? kTok + 2 * kTailMaxEps : kTok];
  __shared__ __attribute__((aligned(16))) uint32_t digit_hist[(SPLIT == 1 ? kLaneCopies : 1) * kRadixBins];
  const int b = __builtin_amdgcn_workgroup_id_y(), blk = __builtin_amdgcn_workgroup_id_x(), tid = __builtin_amdgcn_workitem_id_x();
  const int lane = tid & 63, wave = tid >> 6;
  const float* s = S + (int64_t)b * s_bs;
  const float* pt = part + (int64_t)b * n_part * l_c;
  int64_t first = SPLIT == 1 ? (int64_t)blk * sub * kTok - eps : (int64_t)blk * (kTok - 2 * eps) - eps;   // of the tokens read
  auto clamped = [&](int64_t m) { return m < 0 ? (int64_t)0 : (m < n ? m : n - 1); };
  // SPLIT = 1: the first queries' scores are requested in front of the partial maxima (one round trip together)
  float x[kAhead][kPer];
  auto request = [&](int64_t from, int c0) {
    int64_t mine_at[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) mine_at[u] = clamped(from + 256 * u + tid);
#pragma unroll
    for (int a = 0; a < kAhead; ++a)
#pragma unroll
      for (int u = 0; u < kPer; ++u)
        if ((a == 0 || (!ONE && c0 + a < l_c)) && (u < 4 || tid < 2 * eps)) x[a][u] = s[(int64_t)(c0 + a) * s_ld + mine_at[u]];
  };
  if (SPLIT == 1) request(first, 0);
  // The 256 threads are shared out over lc2 >= l_c queries (a power of two): thread t reduces every (256 / lc2)-th partial
  // maximum of one of them.
  float mu_one = 0.f;
  if (ONE) {
    float m = -INFINITY;
    for (int j0 = tid; j0 < n_part; j0 += 4 * 256) {
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = pt[j0 + u * 256 < n_part ? j0 + u * 256 : j0];
      m = fmaxf(fmaxf(m, v[0]), fmaxf(fmaxf(v[1], v[2]), v[3]));
    }
    if (first_hist) lane_copies_clear(digit_hist, tid, 256);
    m = wave_max(m);
    if (lane == 0) red[wave] = m;
    __syncthreads();
    mu_one = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  } else if (SPLIT == 1) {
    int lc2 = 1;
    while (lc2 < l_c) lc2 *= 2;                             // at most sixteen: whole 16-lane rows per query
    const int per = 256 / lc2, c = tid / per < l_c ? tid / per : l_c - 1;
    float m = -INFINITY;
    for (int j0 = tid % per; j0 < n_part; j0 += 4 * per) {
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = pt[(int64_t)(j0 + u * per < n_part ? j0 + u * per : j0) * l_c + c];
      m = fmaxf(fmaxf(m, v[0]), fmaxf(fmaxf(v[1], v[2]), v[3]));
    }
    m = lanes_max16(m);
    if ((tid & 15) == 0) red[tid >> 4] = m;
    if (first_hist) lane_copies_clear(digit_hist, tid, 256);
    __syncthreads();
    if (tid < l_c) {
      const int rows = 16 / lc2;
      m = red[tid * rows];
      for (int i = 1; i < rows; ++i) m = fmaxf(m, red[tid * rows + i]);
      mu[tid] = m;
    }
    __syncthreads();
  } else {
    if (first_hist)
      for (int i = tid; i < kRadixBins; i += 256) digit_hist[i] = 0u;
    int lc2 = 1;
    while (lc2 < l_c && lc2 < 256) lc2 *= 2;
    const int groups = 256 / lc2, jg = tid / lc2;
    for (int c0 = 0; c0 < l_c; c0 += lc2) {
      const int c = c0 + tid % lc2 < l_c ? c0 + tid % lc2 : l_c - 1;
      float m = -INFINITY;
      for (int j0 = jg; j0 < n_part; j0 += 8 * groups) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = pt[(int64_t)(j0 + u * groups < n_part ? j0 + u * groups : j0) * l_c + c];
#pragma unroll
        for (int u = 0; u < 8; ++u) m = fmaxf(m, v[u]);
      }
      red[tid] = m;
      __syncthreads();
      if (tid < lc2 && c0 + tid < l_c) {
        for (int g = 1; g < groups; ++g) m = fmaxf(m, red[g * lc2 + tid]);
        mu[c0 + tid] = m;
      }
      __syncthreads();
    }
  }
  auto pooled = [&](int64_t at_token, int at, float f) {    // tile[at] is token at_token
    for (int d = -eps; d <= eps; ++d)
      if (at_token + d >= 0 && at_token + d < n) f = fmaxf(f, tile[at + d]);
    return f;
  };
  if (SPLIT == 1) {
    for (int st = 0; st < sub && first + eps < n; ++st, first += kTok) {
      float f[kPer];
#pragma unroll
      for (int u = 0; u < kPer; ++u) f[u] = ONE ? x[0][u] - mu_one : -INFINITY;
      for (int c0 = 0; !ONE && c0 < l_c; c0 += kAhead) {
        if (c0 > 0) request(first, c0);
#pragma unroll
        for (int a = 0; a < kAhead; ++a) {
          if (c0 + a < l_c) {
            const float muc = mu[c0 + a];
#pragma unroll
            for (int u = 0; u < kPer; ++u) f[u] = fmaxf(f[u], x[a][u] - muc);
          }
        }
      }
      if (st + 1 < sub) request(first + kTok, 0);           // the next tile's, during this one's histogram
      if (POOL) {
        if (st > 0) __syncthreads();
#pragma unroll
        for (int u = 0; u < kPer; ++u)
          if (u < 4 || tid < 2 * eps) tile[256 * u + tid] = f[u];
        __syncthreads();
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t m = first + eps + 256 * u + tid;
        float v = f[u];
        if (POOL) v = m < n ? pooled(m, 256 * u + tid + eps, tile[256 * u + tid + eps]) : 0.f;
        if (m < n) score[(int64_t)b * score_bs + m] = v;
        if (first_hist) lane_copies_add(digit_hist, m < n, score_digit(ordered_key(v)), lane);
      }
    }
  } else {
    const int64_t m = first + lane;
    const float* col = s + clamped(m);
    float f = -INFINITY;
#pragma unroll 8
    for (int c = wave; c < l_c; c += 4) f = fmaxf(f, col[(int64_t)c * s_ld] - mu[c]);
    red[tid] = f;
    __syncthreads();
    if (wave == 0) {
      f = fmaxf(fmaxf(red[lane], red[64 + lane]), fmaxf(red[128 + lane], red[192 + lane]));
      tile[lane] = f;
    }
    __syncthreads();
    if (wave == 0) {
      const bool mine = m >= 0 && m < n && lane >= eps && lane < kTok - eps;
      if (POOL && mine) f = pooled(m, lane, f);
      if (mine) score[(int64_t)b * score_bs + m] = f;
      if (first_hist) hist_add(digit_hist, mine, score_digit(ordered_key(f)));
    }
  }
  if (first_hist) {
    __syncthreads();
    uint32_t* gh = first_hist + (int64_t)b * first_hist_bs;
    if (SPLIT == 1)
      lane_copies_flush(gh, digit_hist, blk, tid, 256);
    else
      hist_flush(gh, digit_hist, blk, tid, 256);
  }
}

// Eq. 8: out[j] = max(in[max(j-eps,0) .. min(j+eps,n-1)]).  With first_hist given, also the histogram of the
// pooled scores' first digits (this is the kernel that writes the scores the selection reads).
__global__ __launch_bounds__(256) void proximity_maxpool(const float* __restrict__ in, float* __restrict__ out, int64_t n,
                                                         int eps, int64_t in_bs, int64_t out_bs,
                                                         uint32_t* __restrict__ first_hist, int64_t first_hist_bs) {
  __shared__ uint32_t digit_hist[kRadixBins];
  const int n_wg = maxpool_blocks(n);                         // workgroups per batch entry (the launch's grid)
  if (first_hist)
    for (int i = __builtin_amdgcn_workitem_id_x(); i < kRadixBins; i += 256) digit_hist[i] = 0u;
  __syncthreads();
  const float* src = in + (int64_t)__builtin_amdgcn_workgroup_id_y() * in_bs;
  float* dst = out + (int64_t)__builtin_amdgcn_workgroup_id_y() * out_bs;
  // whole waves stay in the loop together (hist_add is a wave-wide operation)
  for (int64_t j0 = (int64_t)__builtin_amdgcn_workgroup_id_x() * 256 + (__builtin_amdgcn_workitem_id_x() & ~63); j0 < n; j0 += (int64_t)n_wg * 256) {
    const int64_t j = j0 + (__builtin_amdgcn_workitem_id_x() & 63);
    float m = 0.f;
    if (j < n) {
      const int64_t lo = j - eps > 0 ? j - eps : 0, hi = j + eps < n - 1 ? j + eps : n - 1;
      m = src[lo];
      for (int64_t w = lo + 1; w <= hi; ++w) m = fmaxf(m, src[w]);
      dst[j] = m;
    }
    if (first_hist) hist_add(digit_hist, j < n, score_digit(ordered_key(m)));
  }
  if (first_hist) {
    __syncthreads();
    uint32_t* gh = first_hist + (int64_t)__builtin_amdgcn_workgroup_id_y() * first_hist_bs;
    hist_flush(gh, digit_hist, __builtin_amdgcn_workgroup_id_x(), __builtin_amdgcn_workitem_id_x(), 256);
  }
}

}  // namespace

// S is stored (one pass over K') instead of recomputed: few queries, or a small S.
__host__ inline bool stores_scores(int l_c, int64_t n, int batch) {
  return l_c <= kFewQueries || (l_c <= kFinishMaxQueries && (int64_t)l_c * n * batch * 4 <= ((int64_t)16 << 20));
}
__host__ inline int64_t stored_ld(int64_t n) { return (n + 63) / 64 * 64; }
// One current token: S is kept where F goes.  (The workspace is asked for without type and d_c: it holds the S of fp32 queries, which
// bf16 ones with d_c 64 or 128, swept twice, leave unused.)
__host__ inline size_t stored_bytes(int l_c, int64_t n, int batch) {
  return l_c > 1 && stores_scores(l_c, n, batch) ? (size_t)l_c * stored_ld(n) * 4 * batch : 0;
}

// partial row maxima of the kernels that store S: one per query and workgroup of at least 64 tokens
__host__ inline size_t part_bytes(int l_c, int64_t n_mid, int batch) {
  return stores_scores(l_c, n_mid, batch) ? align_up((size_t)((n_mid + kGTok - 1) / kGTok) * l_c * batch * 4, 256) : 0;
}
// what the sweeps need cleared: the copies of the row maxima, a mark for every share
__host__ inline size_t mu_copies_bytes(int l_c, int batch) { return mu_bytes(l_c, batch) * kMuCopies; }
__host__ inline size_t sweeps_bytes(int l_c, int64_t n_mid, int eps, int batch) {
  return mu_copies_bytes(l_c, batch) + (size_t)mark_words(most_shares(n_mid, eps <= kTailMaxEps ? eps : 0, batch)) * kMuCopies * 4;
}

// The two sweeps of the matrix-core path.  patience: 0, or 1 + how long (10 ns) a workgroup waits for the others.
template <int DC>
int launch_sweeps(const bf16_t* qc, int l_c, const bf16_t* kc, int64_t m_lo, int64_t n, void* ws, float* score, int batch, int64_t q_bs,
                  int64_t kc_bs, int64_t score_bs, uint32_t* hists, bool fill_first, int64_t hists_bs, int eps, uint32_t patience, hipStream_t st) {
  const int per = (int)share_tiles(n, eps, batch), n_row = (int)share_count(n, eps, batch);
  const int64_t n_shares = (int64_t)n_row * batch;
  const int n_wg = (int)(n_shares < kComputeUnits ? n_shares : kComputeUnits);
  static OncePerDevice raised;
  constexpr int kHalves = DC == 128 ? 2 : 1;               // d_c = 64: there is always room for whole blocks
  const int rc = raise_lds_limit(raised, {(const void*)score_sweeps_bf16<DC, 0>, (const void*)score_sweeps_bf16<DC, 1>, (const void*)score_sweeps_bf16<DC, kHalves>},
                                 160 * 1024, "score_sweeps_bf16");
  if (rc != ESA_OK) return rc;
  uint32_t* mu_keys = (uint32_t*)ws;
  uint32_t* marks = (uint32_t*)((char*)ws + mu_copies_bytes(l_c, batch));
  const int64_t n_own = (int64_t)(mu_copies_bytes(l_c, batch) + mark_words(n_shares) * kMuCopies * 4) / 16;
  const int parts = later_queries_parts(per, DC, l_c);
  const auto sweeps = parts == 0 ? score_sweeps_bf16<DC, 0> : parts == 1 ? score_sweeps_bf16<DC, 1> : score_sweeps_bf16<DC, kHalves>;
  const int64_t n_clear = n_own + (hists ? (int64_t)batch * (kHistWords / 4) : 0);
  score_sweeps_clear<<<(unsigned)((n_clear + 255) / 256), 256, 0, st>>>((uint4*)ws, n_own, hists, hists_bs, batch);
  sweeps<<<n_wg, kThreads, sweeps_lds_bytes(per, DC, l_c), st>>>(
      qc, kc + m_lo * DC, (int)n, l_c, per, tiles_before_queries(per, DC, l_c), query_waves_log2(l_c, per, DC), n_row, (int)n_shares, n_wg, eps, inverse_of((uint32_t)n_row),
      mu_keys, marks, score, q_bs, kc_bs, score_bs, fill_first ? hists : nullptr, hists_bs, patience, later_queries_at(per, DC));
  return ESA_OK;
}

// What lies in front of the partial maxima: the sweeps', or the row maxima alone.
__host__ inline size_t front_bytes(int l_c, int64_t n_mid, int eps, int batch) {
  return l_c > kFewQueries ? sweeps_bytes(l_c, n_mid, eps, batch) : mu_bytes(l_c, batch);
}

// Callers size one workspace by their chunks and use it for the few tokens behind them, too, which store S and so need more than a chunk does.
// A chunk's size is therefore not what the sweeps need but 4 bytes a query and share and 256 bytes a query (whole blocks): it covers any shorter
// chunk that is swept, one token and, as far as it goes, up to sixteen (512 tokens over 20000: eight).
size_t score_workspace_bytes(int l_c, int64_t n_mid, int eps, int batch) {
  if (l_c <= 0 || batch <= 0 || n_mid < 0) return 256;
  size_t b = front_bytes(l_c, n_mid, eps, batch) + part_bytes(l_c, n_mid, batch);
  if (l_c > kFewQueries) {
    const size_t shares = (size_t)most_shares(n_mid, eps <= kTailMaxEps ? eps : 0, batch), blocks = (l_c + kQPerBlock - 1) / kQPerBlock;
    size_t rows = align_up(shares * l_c * 4, 256);
    rows = rows > part_bytes(l_c, n_mid, batch) ? rows : part_bytes(l_c, n_mid, batch);
    const size_t chunk = mu_bytes(l_c, batch) + rows + blocks * kQPerBlock * 256 * batch;
    b = b > chunk ? b : chunk;
  }
  if (eps > 0) b += align_up((size_t)n_mid * 4, 256) * (size_t)batch;
  b += stored_bytes(l_c, n_mid, batch);
  return b;
}

int launch_score(const void* qc, int l_c, const void* kc_cache, int64_t m_lo, int64_t m_hi, int d_c, int eps,
                 float* score, int dtype, int batch, int64_t q_bs, int64_t kc_bs, int64_t score_bs, void* ws,
                 size_t ws_bytes, hipStream_t st, uint32_t* first_hist, int64_t first_hist_bs, bool* first_hist_done,
                 ScoreTail* tail, uint32_t patience) {
  const int64_t n = m_hi - m_lo;
  // eps > 0: windows of up to kTailMaxEps on either side are pooled by whatever finishes the scores (score_finish, the second
  // sweep where sweep_pools, or the selection through *tail); the unpooled scores of the other cases go to `raw` and proximity_maxpool reads them.
  const bool narrow = eps <= kTailMaxEps;
  bool zeroed = false;                  // the selection's histograms have been zeroed ...
  if (first_hist_done) *first_hist_done = false;        // ... and the first one filled
  float* part = (float*)((char*)ws + front_bytes(l_c, n, eps, batch));
  char* at = (char*)part + part_bytes(l_c, n, batch);
  float* raw = score;
  int64_t raw_bs = score_bs;
  if (eps > 0) {
    raw = (float*)at;
    raw_bs = (int64_t)(align_up((size_t)n * 4, 256) / 4);
    at += align_up((size_t)n * 4, 256) * (size_t)batch;
  }
  if (tail) *tail = ScoreTail{score, score_bs, nullptr, 0, 0};
  bool pool_left = eps > 0;
  const bool vec_ok = dtype == ESA_BF16 && (((uintptr_t)qc | (uintptr_t)kc_cache) % 16 == 0) && q_bs % 8 == 0 &&
                      kc_bs % 8 == 0;
  // S of one current token: where F goes (pooling reads neighbours: the unpooled buffer); of several: in the workspace
  float* S = l_c == 1 ? raw : (float*)at;
  const int64_t s_ld = l_c == 1 ? n : stored_ld(n), s_bs = l_c == 1 ? raw_bs : (int64_t)l_c * s_ld;
  auto finish = [&](int n_part) {
    float* out = narrow ? score : raw;
    const int64_t out_bs = narrow ? score_bs : raw_bs;
    const int e = narrow ? eps : 0;
    uint32_t* hist = narrow ? first_hist : nullptr;
    const bool few = l_c <= kFewQueries;
    const auto kernel = l_c == 1 ? (e > 0 ? score_finish<1, true, true> : score_finish<1, false, true>)
                        : few    ? (e > 0 ? score_finish<1, true> : score_finish<1, false>)
                                 : (e > 0 ? score_finish<4, true> : score_finish<4, false>);
    const int sub = topk_tiles_per_wg(n, batch);
    const unsigned wgs = few ? (unsigned)((n + 1024 * (int64_t)sub - 1) / (1024 * (int64_t)sub)) : (unsigned)((n + 63 - 2 * e) / (64 - 2 * e));
    kernel<<<dim3(wgs, batch), 256, 0, st>>>(S, s_ld, s_bs, n, part, n_part, l_c, e, sub, out, out_bs, hist, first_hist_bs);
    if (hist && first_hist_done) *first_hist_done = true;
    zeroed = first_hist != nullptr;
    pool_left = eps > 0 && !narrow;
  };
  if (vec_ok && l_c == 1 && (d_c == 64 || d_c == 128 || d_c == 256)) {
    const bool stream = gemv_streams(n, batch, d_c, kc_bs);
    const int rows = stream ? 512 : 64, threads = stream ? 512 : 256, nblk = (int)((n + rows - 1) / rows);
    const auto gemv = stream ? (d_c == 64 ? score_gemv_bf16<8, 512, 8> : d_c == 128 ? score_gemv_bf16<16, 512, 16> : score_gemv_bf16<32, 512, 32>)
                             : (d_c == 64 ? score_gemv_bf16<8, 256, 2> : d_c == 128 ? score_gemv_bf16<16, 256, 4> : score_gemv_bf16<32, 256, 8>);
    // workgroup w runs on XCD w % 8: in rows of a multiple of eight, all sequences that share a part of K' fetch it into one L2
    const unsigned grid = shared_keys(batch, kc_bs) ? (unsigned)((nblk + 7) / 8 * 8) : (unsigned)nblk;
    gemv<<<dim3(grid, batch), threads, 0, st>>>((const bf16_t*)qc, (const bf16_t*)kc_cache, m_lo, n, part, raw, q_bs, kc_bs, raw_bs,
                                                      first_hist, first_hist_bs);
    if (tail && narrow) {
      *tail = ScoreTail{raw, raw_bs, part, nblk, eps};
      pool_left = false;
    } else {
      finish(nblk);
    }
  } else if (vec_ok && l_c <= kFewQueries && (d_c == 128 || d_c == 64)) {
    const int nblk = (int)((n + kFewTok - 1) / kFewTok);
    const bool stream = !shared_keys(batch, kc_bs) && n * batch * d_c * (int64_t)sizeof(bf16_t) >= kFewStreamBytes;
    const auto few = d_c == 128 ? (stream ? score_few_bf16<128, true> : score_few_bf16<128, false>)
                                : (stream ? score_few_bf16<64, true> : score_few_bf16<64, false>);
    few<<<dim3((unsigned)nblk, batch), 256, 0, st>>>((const bf16_t*)qc, l_c, (const bf16_t*)kc_cache, m_lo, n, part, S, s_ld, s_bs, q_bs,
                                                     kc_bs, nblk, first_hist, first_hist_bs);
    finish(nblk);
  } else if (vec_ok && (d_c == 128 || d_c == 64)) {
    const auto sweeps = d_c == 128 ? launch_sweeps<128> : launch_sweeps<64>;
    const bool pools = sweep_pools(n, eps, batch, kTailMaxEps);
    const int rc = sweeps((const bf16_t*)qc, l_c, (const bf16_t*)kc_cache, m_lo, n, ws, pools ? score : raw, batch, q_bs, kc_bs,
                          pools ? score_bs : raw_bs, first_hist, pools, first_hist_bs, pools ? eps : 0, patience, st);
    if (rc != ESA_OK) return rc;
    zeroed = first_hist != nullptr;
    if (first_hist && pools && first_hist_done) *first_hist_done = true;
    if (pools) pool_left = false;
  } else if (stores_scores(l_c, n, batch)) {
    const int nblk = (int)((n + kGTok - 1) / kGTok);
    const dim3 grid((unsigned)nblk, (unsigned)((l_c + kStoreQ - 1) / kStoreQ), batch);
    const size_t smem = (size_t)(kGTok + kStoreQ) * store_ld(d_c) * sizeof(float);
    const auto go = [&](auto kernel, auto* q, auto* k) -> int {
      if (smem > 65536) {
        const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return hip_failed(e, "hipFuncSetAttribute(score_store_fma)");
      }
      kernel<<<grid, 256, smem, st>>>(q, l_c, k, m_lo, n, d_c, part, S, s_ld, s_bs, q_bs, kc_bs, nblk, first_hist, first_hist_bs);
      return ESA_OK;
    };
    // (one query's S lies where F goes, in rows of any length)
    if (dtype == ESA_F32 && l_c > 1 && (((uintptr_t)qc | (uintptr_t)kc_cache) % 16 == 0) && q_bs % 4 == 0 && kc_bs % 4 == 0) {
      score_store_f32<<<dim3((unsigned)nblk, (unsigned)((l_c + kTileQ - 1) / kTileQ), batch), 256, 0, st>>>(
          (const float*)qc, l_c, (const float*)kc_cache, m_lo, n, d_c, part, S, s_ld, s_bs, q_bs, kc_bs, nblk, first_hist, first_hist_bs);
    } else {
      const int rc = dtype == ESA_BF16 ? go(score_store_fma<bf16_t>, (const bf16_t*)qc, (const bf16_t*)kc_cache)
                                       : go(score_store_fma<float>, (const float*)qc, (const float*)kc_cache);
      if (rc != ESA_OK) return rc;
    }
    finish(nblk);
  } else {
    uint32_t* mu = (uint32_t*)ws;
    fill_u32<<<(l_c * batch + 255) / 256, 256, 0, st>>>(mu, (int64_t)l_c * batch, kOrderedKeyOfMinusInf);
    const dim3 grid((unsigned)((n + kGTok - 1) / kGTok), batch);
    const size_t smem = (size_t)(kGTok * (d_c + 1) + 4 * kGTok) * sizeof(float);
    if (smem > 65536) {   // d_c > 240: raise the dynamic LDS limit of the four instantiations
      const void* fns[] = {(const void*)score_fma<bf16_t, 0>, (const void*)score_fma<bf16_t, 1>,
                           (const void*)score_fma<float, 0>, (const void*)score_fma<float, 1>};
      for (const void* f : fns) {
        hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return hip_failed(e, "hipFuncSetAttribute(score_fma)");
      }
    }
    if (dtype == ESA_BF16) {
      score_fma<bf16_t, 0><<<grid, 256, smem, st>>>((const bf16_t*)qc, l_c, (const bf16_t*)kc_cache, m_lo, n, d_c, mu,
                                                    raw, q_bs, kc_bs, raw_bs);
      score_fma<bf16_t, 1><<<grid, 256, smem, st>>>((const bf16_t*)qc, l_c, (const bf16_t*)kc_cache, m_lo, n, d_c, mu,
                                                    raw, q_bs, kc_bs, raw_bs);
    } else {
      score_fma<float, 0><<<grid, 256, smem, st>>>((const float*)qc, l_c, (const float*)kc_cache, m_lo, n, d_c, mu,
                                                   raw, q_bs, kc_bs, raw_bs);
      score_fma<float, 1><<<grid, 256, smem, st>>>((const float*)qc, l_c, (const float*)kc_cache, m_lo, n, d_c, mu,
                                                   raw, q_bs, kc_bs, raw_bs);
    }
  }
  if (pool_left) {
    uint32_t* ph = zeroed ? first_hist : nullptr;      // only behind kernels that have zeroed the histograms
    proximity_maxpool<<<dim3(maxpool_blocks(n), batch), 256, 0, st>>>(raw, score, n, eps, raw_bs, score_bs, ph, first_hist_bs);
    if (ph && first_hist_done) *first_hist_done = true;
  }
  ESA_LAUNCH_CHECK("score");
  return ESA_OK;
}

}  // namespace esa

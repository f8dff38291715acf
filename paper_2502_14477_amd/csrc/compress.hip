// Query/key compression (Eq. 5): out[n, :] = x[n, :] . W (+ bias), one linear layer on the
// head-concatenated vector, fp32 accumulation, result rounded to the storage type.
//
// Kernels:
//   * compress_mfma_packed_bf16 — bf16 storage, weights in the packed (output-major) layout written by
//     esa_pack_weights.  Both MFMA operands then have their reduction elements contiguous in memory
//     and reach LDS in whole cache lines without passing through registers.  A workgroup owns 16 or 32
//     token rows x 16 outputs; its eight waves share d_in and the partial tiles are added in a fixed
//     order (deterministic, no atomics).
//   * compress_few_packed_bf16 — the same inputs for one to four tokens (a decode step): one workgroup per
//     output, a dot product per token.
//   * compress_mfma_bf16 — bf16 storage, weights as given ([d_in, d_c]); W is transposed through LDS.
//   * compress_fma — any storage type, shape and weight layout, plain fp32 FMAs.
//   * pack_weights — the one-time transposition [d_in, d_c] -> [d_c, d_in].
#include "esa_common.h"

namespace esa {
namespace {

// One launch serves up to two inputs ("jobs") that share the token count, d_c and the batch: the chunk's
// queries and keys are compressed side by side (Eq. 5 has both).  The job is the slow index of the grid
// (blockIdx.y = job * col_tiles + column tile), so that all workgroups of job 0 are dispatched before
// those of job 1 and a compute unit gets one of each rather than two of the long ones.
template <typename T>
struct CompressJob {
  const T* x;
  const T* Wt;
  const T* bias;
  T* out;
  int64_t d_in, ldx, ldo, x_bs, out_bs;
};
// field-wise select: every kernel argument is fetched in the first round trip
template <typename T>
__device__ __forceinline__ CompressJob<T> pick_job(const CompressJob<T>& j0, const CompressJob<T>& j1, bool second) {
  CompressJob<T> j;
  j.x = second ? j1.x : j0.x;
  j.Wt = second ? j1.Wt : j0.Wt;
  j.bias = second ? j1.bias : j0.bias;
  j.out = second ? j1.out : j0.out;
  j.d_in = second ? j1.d_in : j0.d_in;
  j.ldx = second ? j1.ldx : j0.ldx;
  j.ldo = second ? j1.ldo : j0.ldo;
  j.x_bs = second ? j1.x_bs : j0.x_bs;
  j.out_bs = second ? j1.out_bs : j0.out_bs;
  return j;
}

// ------------------------------------------------------------------------------------------ generic
// A workgroup owns 16 tokens x 16 outputs, one per thread of 256; four groups of 256 threads take a quarter of every
// 256 staged reduction elements each, and their sums are added in a fixed order.  What bounds a small layer is the
// number of round trips (a chunk of 128 tokens of an fp32 layer with d_in = 256: one; 28 us per input for one workgroup
// per 16 tokens that walked the reduction 64 elements at a time).
constexpr int kTok = 16;
constexpr int kCols = 16;
constexpr int kStage = 256;    // reduction elements staged per step

template <typename T, bool PACKED>
__global__ __launch_bounds__(1024) void compress_fma(CompressJob<T> j0, CompressJob<T> j1, int64_t n_tok, int d_c, int col_tiles) {
  constexpr int kLd = kStage + 4;                // rows 16 bytes apart in the banks
  __shared__ __attribute__((aligned(16))) float xs[kTok][kLd], ws[kCols][kLd];
  __shared__ float red[4][kTok * kCols];
  const bool second = (int)blockIdx.y >= col_tiles;
  const CompressJob<T> j = pick_job(j0, j1, second);
  const T* xb = j.x + (int64_t)blockIdx.z * j.x_bs;
  const int tid = threadIdx.x, kg = tid >> 8, o = tid & 255, t = o >> 4, c = o & 15;
  const int64_t tok0 = (int64_t)blockIdx.x * kTok;
  const int col0 = ((int)blockIdx.y - (second ? col_tiles : 0)) * kCols;      // d_c is a multiple of 16
  float acc = 0.f;
  for (int64_t i0 = 0; i0 < j.d_in; i0 += kStage) {
    float xv[4], wv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = tid + 1024 * u, row = e >> 8;
      const int64_t i = i0 + (e & 255), tok = tok0 + row;
      xv[u] = i < j.d_in && tok < n_tok ? load_f32(xb + tok * j.ldx + i) : 0.f;
      if (PACKED) {
        wv[u] = i < j.d_in ? load_f32(j.Wt + (int64_t)(col0 + row) * j.d_in + i) : 0.f;
      } else {
        const int64_t iw = i0 + (e >> 4);
        wv[u] = iw < j.d_in ? load_f32(j.Wt + iw * (int64_t)d_c + col0 + (e & 15)) : 0.f;
      }
    }
    __syncthreads();                             // the previous step's reads are done
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = tid + 1024 * u;
      xs[e >> 8][e & 255] = xv[u];
      if (PACKED) ws[e >> 8][e & 255] = wv[u];
      else ws[e & 15][e >> 4] = wv[u];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kStage / 4; k += 4) {
      const float4 a = *(const float4*)&xs[t][kg * (kStage / 4) + k], b = *(const float4*)&ws[c][kg * (kStage / 4) + k];
      acc = __fmaf_rn(a.x, b.x, acc);
      acc = __fmaf_rn(a.y, b.y, acc);
      acc = __fmaf_rn(a.z, b.z, acc);
      acc = __fmaf_rn(a.w, b.w, acc);
    }
  }
  red[kg][o] = acc;
  __syncthreads();
  if (kg == 0 && tok0 + t < n_tok) {
    float v = (red[0][o] + red[1][o]) + (red[2][o] + red[3][o]);
    if (j.bias) v += load_f32(j.bias + col0 + c);
    store_f32(j.out + (int64_t)blockIdx.z * j.out_bs + (tok0 + t) * j.ldo + col0 + c, v);
  }
}

// ------------------------------------------------------------------------------------------ MFMA
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// Tile: 16 tokens x 64 outputs per workgroup (4 waves, one 16x16 output tile each), the whole
// reduction dimension walked in steps of 128.  v_mfma_f32_16x16x32_bf16: lane l supplies
// A[l%16][8*(l/16) .. +7] and B[8*(l/16) .. +7][l%16], and owns C[4*(l/16) .. +3][l%16].
// x rows are read straight from global memory (16 bytes per lane); W is staged transposed in LDS
// so that a lane's eight reduction elements of one output column are contiguous.
constexpr int kMTok = 16;
constexpr int kMCols = 64;
constexpr int kMStep = 128;

__global__ __launch_bounds__(256) void compress_mfma_bf16(const bf16_t* __restrict__ x, int64_t n_tok, int64_t d_in,
                                                          int64_t ldx, const bf16_t* __restrict__ W,
                                                          const bf16_t* __restrict__ bias, int d_c,
                                                          bf16_t* __restrict__ out, int64_t ldo, int64_t x_bs,
                                                          int64_t out_bs) {
  // wt[col][k]: 64 columns x 128 reduction elements, row padded by 8 elements (16 bytes).
  __shared__ __attribute__((aligned(16))) bf16_t wt[kMCols][kMStep + 8];
  const bf16_t* xb = x + (int64_t)blockIdx.z * x_bs;
  bf16_t* ob = out + (int64_t)blockIdx.z * out_bs;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t tok0 = (int64_t)blockIdx.x * kMTok;
  const int col0 = blockIdx.y * kMCols;
  const int r = lane & 15, q = lane >> 4;
  int64_t tok = tok0 + r;
  const bool tok_ok = tok < n_tok;
  if (!tok_ok) tok = n_tok - 1;                      // keep the address valid; result discarded
  const bf16_t* xrow = xb + tok * ldx;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};

  for (int64_t i0 = 0; i0 < d_in; i0 += kMStep) {
    __syncthreads();
    // Stage W[i0 .. i0+128, col0 .. col0+64) transposed: thread handles 2 rows x 16 columns... simple 2-byte scatter.
    for (int e = threadIdx.x; e < kMStep * (kMCols / 8); e += 256) {
      const int kk = e / (kMCols / 8), c8 = (e % (kMCols / 8)) * 8;
      const uint4 v = *(const uint4*)(W + (i0 + kk) * (int64_t)d_c + col0 + c8);
      const bf16_t* pv = (const bf16_t*)&v;
#pragma unroll
      for (int j = 0; j < 8; ++j) wt[c8 + j][kk] = pv[j];
    }
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < kMStep / 32; ++ks) {
      const bf16x8 a = *(const bf16x8*)(xrow + i0 + ks * 32 + q * 8);
      const bf16x8 b = *(const bf16x8*)(&wt[wave * 16 + r][ks * 32 + q * 8]);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
    }
  }
  // C[4q+v][r]: token tok0+4q+v, column col0 + wave*16 + r.
  const int col = col0 + wave * 16 + r;
  const float bv = bias ? bf16_to_f32(bias[col]) : 0.f;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int64_t t = tok0 + q * 4 + v;
    if (t < n_tok) ob[t * ldo + col] = f32_to_bf16(acc[v] + bv);
  }
}


// ------------------------------------------------------------------------------------------ MFMA, packed weights
// v_mfma_f32_16x16x32_bf16: lane l supplies A[l%16][8*(l/16) .. +7] and B[8*(l/16) .. +7][l%16] and owns
// C[4*(l/16) .. +3][l%16].  A rows are tokens (of all batch entries, numbered through), B columns are outputs.
//
// A workgroup owns TT x 16 rows x 16 outputs of both inputs, its eight waves take every eighth piece of 64 reduction
// elements.  What bounds it is the rate at which the L2s hand rows out (512 tokens: 80 MB in the 3.4 us of the loop, 24 TB/s of some 31): each reads (16 TT + 16)
// rows of d_in.  Read as fragments, sixteen half cache lines per instruction, a line's second half had left the first-
// level cache before it was asked for and the 80 MB of a chunk of 512 tokens became 160 MB of L2 traffic: 11.1 us
// (7.0 now; 1024 tokens 22.4 -> 10.9, 77 tokens 9.8 -> 6.0).  So whole lines go to LDS without passing through registers, eight 128-byte rows per instruction, two
// pieces at a time in a ring of the wave's own: no barrier until the waves' sums meet, in a fixed order (deterministic).  (More pieces in flight are
// no quicker: 512 tokens with two, three, four, five 7.0, 7.4, 7.4, 8.0 us; 16 rows 5.6, 6.0, 6.2, 6.4.)
// 16-byte slots of a row are swizzled by row / 2 (two rows share the 256 bytes that the banks cover), which keeps the
// fragment reads free of conflicts.
constexpr int kPWaves = 8;
constexpr int kPiece = 64;                       // reduction elements of a piece: a cache line per row
constexpr int kPieceRows = 16 * kPiece * 2;      // bytes of sixteen rows of a piece
constexpr int kRing = 2;                         // pieces of a wave in LDS
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) const void global_void;

template <int TT>
constexpr int packed_lds_bytes() { return kPWaves * kRing * (TT + 1) * kPieceRows; }

// Every load but the LEFT newest of this wave is in LDS.
template <int LEFT>
__device__ __forceinline__ void loads_but() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LEFT) : "memory"); }

// split_jobs: a workgroup takes one of the two inputs (column tiles numbered job by job) instead of both.
template <int TT>
__global__ __launch_bounds__(64 * kPWaves) void compress_mfma_packed_bf16(CompressJob<bf16_t> j0, CompressJob<bf16_t> j1, int n_jobs,
                                                                          int split_jobs, uint32_t n_tok, uint32_t n_rows,
                                                                          int row_tiles, int col_tiles) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char ring_lds[];
  constexpr int kLoads = 2 * TT + 2;             // load instructions of a piece
  constexpr int kBytes = (TT + 1) * kPieceRows;  // a piece in LDS: the token rows, then the weight rows
  // Column tiles of one row tile on one XCD where there are enough row tiles (workgroup w runs on XCD w % 8): its rows
  // are then fetched into one L2.  Fewer row tiles spread over the XCDs.
  const int n_col = split_jobs ? n_jobs * col_tiles : col_tiles;
  int rt, ct;
  if (row_tiles >= 8) {
    const int k = blockIdx.x >> 3;
    rt = (blockIdx.x & 7) + 8 * (k / n_col);
    ct = k % n_col;
    if (rt >= row_tiles) return;
  } else {
    rt = blockIdx.x / n_col;
    ct = blockIdx.x % n_col;
  }
  const int only = split_jobs && ct >= col_tiles ? 1 : 0;
  const int job_first = only, job_last = split_jobs ? only : n_jobs - 1;
  const int col0 = (ct - only * col_tiles) * 16;
  const uint32_t row0 = (uint32_t)rt * (16 * TT);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, q = lane >> 4;

  // ---- pieces of this wave, input after input: wave, wave + 8, ... of each
  const int n0 = (int)(j0.d_in / kPiece), n1 = (int)(j1.d_in / kPiece);
  const int c0 = job_first == 0 ? (n0 - wave + kPWaves - 1) / kPWaves : 0;        // of job 0 (never negative: n0 >= 1)
  const int c1 = job_last == 1 ? (n1 - wave + kPWaves - 1) / kPWaves : 0;
  const int count = c0 + c1;

  // ---- loads: a lane brings 16 bytes of row lane / 8 of every group of eight rows
  const uint32_t lr = lane >> 3, slot = lane & 7;
  uint32_t xb[2 * TT], xt[2 * TT];               // batch entry and token of this lane's rows
#pragma unroll
  for (int i = 0; i < 2 * TT; ++i) {
    uint32_t row = row0 + 8 * i + lr;
    row = row < n_rows ? row : n_rows - 1;       // keep the address valid; the row is discarded
    xb[i] = n_rows == n_tok ? 0u : row / n_tok;
    xt[i] = row - xb[i] * n_tok;
  }
  const char *px[2 * TT], *pw[2];
  auto point_at = [&](bool second) {
    const CompressJob<bf16_t> j = pick_job(j0, j1, second);
#pragma unroll
    for (int i = 0; i < 2 * TT; ++i)
      px[i] = (const char*)(j.x + (int64_t)xb[i] * j.x_bs + (int64_t)xt[i] * j.ldx + wave * kPiece + (slot ^ (((8 * i + lr) >> 1) & 7)) * 8);
#pragma unroll
    for (int i = 0; i < 2; ++i)
      pw[i] = (const char*)(j.Wt + (int64_t)(col0 + 8 * i + lr) * j.d_in + wave * kPiece + (slot ^ (((8 * i + lr) >> 1) & 7)) * 8);
  };
  unsigned char* mine = ring_lds + wave * (kRing * kBytes);
  int issued = 0, in_slot = 0;
  auto issue = [&]() {                           // the next piece into the next slot of the ring
    if (issued == 0 || issued == c0) point_at(issued >= c0);
    unsigned char* dst = mine + in_slot * kBytes;
#pragma unroll
    for (int i = 0; i < 2 * TT; ++i) {
      __builtin_amdgcn_global_load_lds((global_void*)px[i], (lds_void*)(dst + 1024 * i), 16, 0, 0);
      px[i] += kPWaves * kPiece * 2;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      __builtin_amdgcn_global_load_lds((global_void*)pw[i], (lds_void*)(dst + TT * kPieceRows + 1024 * i), 16, 0, 0);
      pw[i] += kPWaves * kPiece * 2;
    }
    ++issued;
    in_slot = in_slot ^ 1;
  };
#pragma unroll
  for (int i = 0; i < kRing; ++i)
    if (i < count) issue();

  // Two chains per tile (even and odd halves of the pieces) for each input.
  f32x4 acc[2][TT][2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h) acc[j][t][h] = f32x4{0.f, 0.f, 0.f, 0.f};
  const uint32_t frag = (uint32_t)(uintptr_t)(lds_void*)mine + r * 128 + ((q ^ ((r >> 1) & 7)) << 4);
  int out_slot = 0;
  for (int i = 0; i < count; ++i) {
    if (issued - i == kRing) loads_but<kLoads>();  // a piece has been requested after this one
    else loads_but<0>();
    // The fragment reads and their wait are one block: reads that the compiler sees would wait for every load in flight.
    const uint32_t at0 = frag + (uint32_t)(out_slot * kBytes), at1 = at0 ^ 64u;
    bf16x8 x0[TT], x1[TT], w0, w1;
    if constexpr (TT == 1) {
      asm volatile(
          "ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %4 offset:2048\n\tds_read_b128 %3, %5 offset:2048\n\t"
          "s_waitcnt lgkmcnt(0)"
          : "=&v"(x0[0]), "=&v"(x1[0]), "=&v"(w0), "=&v"(w1)
          : "v"(at0), "v"(at1)
          : "memory");
    } else {
      asm volatile(
          "ds_read_b128 %0, %6\n\tds_read_b128 %1, %7\n\tds_read_b128 %4, %6 offset:4096\n\tds_read_b128 %5, %7 offset:4096\n\t"
          "ds_read_b128 %2, %6 offset:2048\n\tds_read_b128 %3, %7 offset:2048\n\ts_waitcnt lgkmcnt(0)"
          : "=&v"(x0[0]), "=&v"(x1[0]), "=&v"(x0[TT - 1]), "=&v"(x1[TT - 1]), "=&v"(w0), "=&v"(w1)
          : "v"(at0), "v"(at1)
          : "memory");
    }
    if (issued < count) issue();                 // the slot is free: its fragments are in registers
    out_slot = out_slot ^ 1;
    auto multiply = [&](f32x4 (&c)[TT][2]) {
#pragma unroll
      for (int t = 0; t < TT; ++t) {
        c[t][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x0[t], w0, c[t][0], 0, 0, 0);
        c[t][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x1[t], w1, c[t][1], 0, 0, 0);
      }
    };
    if (i < c0) multiply(acc[0]);
    else multiply(acc[1]);
  }

  // ---- the waves' sums meet in LDS: red[input][wave][row][output]
  __syncthreads();
  float* red = (float*)ring_lds;
  constexpr int kTile = TT * 256;
  static_assert(2 * kPWaves * kTile * 4 <= packed_lds_bytes<TT>(), "the sums of both inputs fit the ring");
#pragma unroll
  for (int j = 0; j < 2; ++j)
    if (j >= job_first && j <= job_last)
#pragma unroll
      for (int t = 0; t < TT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[(j * kPWaves + wave) * kTile + (16 * t + 4 * q + v) * 16 + r] = acc[j][t][0][v] + acc[j][t][1][v];
  __syncthreads();
  for (int e = tid + job_first * kTile; e < (job_last + 1) * kTile; e += 64 * kPWaves) {
    const int job = e / kTile, at = e % kTile;
    const uint32_t row = row0 + (at >> 4);
    const int col = col0 + (at & 15);
    if (row >= n_rows) continue;
    const CompressJob<bf16_t> j = pick_job(j0, j1, job == 1);
    float v = red[job * kPWaves * kTile + at];
#pragma unroll
    for (int w = 1; w < kPWaves; ++w) v += red[(job * kPWaves + w) * kTile + at];
    if (j.bias) v += bf16_to_f32(j.bias[col]);
    const uint32_t b = n_rows == n_tok ? 0u : row / n_tok, t = row - b * n_tok;
    j.out[(int64_t)b * j.out_bs + (int64_t)t * j.ldo + col] = f32_to_bf16(v);
  }
}

// Up to four tokens (a decode step): the matrix-core kernel above would occupy d_c / 16 workgroups per input and
// leave the chip idle while sixteen compute units pull the weights through; here every output is a workgroup of
// its own (d_c per input, two inputs per launch), which streams its weight row once, 16 bytes per lane and step,
// against the one to four token rows, and adds up in a fixed order (in-lane, wave butterfly, four waves through
// LDS): deterministic, no atomics.  blockIdx.x = output, blockIdx.y = input (job), blockIdx.z = batch entry.
constexpr int kFewTok = 4;
constexpr int kFewBatch = 4;     // larger batches re-read the weights once per entry here: the matrix-core kernel wins
__global__ __launch_bounds__(256) void compress_few_packed_bf16(CompressJob<bf16_t> j0, CompressJob<bf16_t> j1, int n_tok) {
  __shared__ float red[4][kFewTok];
  const bool second = blockIdx.y != 0;
  const CompressJob<bf16_t> jb = pick_job(j0, j1, second);
  const bf16_t *x = jb.x, *Wt = jb.Wt, *bias = jb.bias;
  bf16_t* out = jb.out;
  const int64_t d_in = jb.d_in, ldx = jb.ldx, ldo = jb.ldo, x_bs = jb.x_bs, out_bs = jb.out_bs;
  const bf16_t* xb = x + (int64_t)blockIdx.z * x_bs;
  const int col = blockIdx.x;
  const bf16_t* wrow = Wt + (int64_t)col * d_in;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float acc[kFewTok] = {0.f, 0.f, 0.f, 0.f};
  // Two steps of the reduction per trip, every load of the trip requested before the first is used and none of
  // them behind a branch (a step past the end re-reads the trip's first, a token past the last re-reads token 0;
  // neither is added): the kernel is a handful of round trips long, and loads that wait for each other are
  // most of them.
  constexpr int kAhead = 2;
  for (int64_t i0 = (int64_t)tid * 8; i0 < d_in; i0 += 256 * 8 * kAhead) {
    bf16x8 w[kAhead], v[kAhead][kFewTok];
#pragma unroll
    for (int a = 0; a < kAhead; ++a) {
      const int64_t i = i0 + a * 256 * 8, ic = i < d_in ? i : i0;
      w[a] = *(const bf16x8*)(wrow + ic);
#pragma unroll
      for (int t = 0; t < kFewTok; ++t) v[a][t] = *(const bf16x8*)(xb + (int64_t)(t < n_tok ? t : 0) * ldx + ic);
    }
#pragma unroll
    for (int a = 0; a < kAhead; ++a) {
      if (i0 + a * 256 * 8 < d_in) {
#pragma unroll
        for (int t = 0; t < kFewTok; ++t) {
          if (t < n_tok) {
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[t] = __fmaf_rn((float)v[a][t][e], (float)w[a][e], acc[t]);
          }
        }
      }
    }
  }
#pragma unroll
  for (int t = 0; t < kFewTok; ++t) {
    if (t >= n_tok) break;
    acc[t] = wave_sum(acc[t]);
    if (lane == 0) red[wave][t] = acc[t];
  }
  __syncthreads();
  if (tid < n_tok) {
    float v = ((red[0][tid] + red[1][tid]) + red[2][tid]) + red[3][tid];
    if (bias) v += bf16_to_f32(bias[col]);
    out[(int64_t)blockIdx.z * out_bs + (int64_t)tid * ldo + col] = f32_to_bf16(v);
  }
}

// W [d_in, d_c] -> Wt [d_c, d_in], through a padded LDS tile so both sides are coalesced.
template <typename T>
__global__ __launch_bounds__(256) void pack_weights(const T* __restrict__ W, int64_t d_in, int d_c, T* __restrict__ Wt) {
  __shared__ T tile[32][33];
  const int64_t i0 = (int64_t)blockIdx.x * 32;
  const int j0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;     // 32 x 8
  for (int yy = ty; yy < 32; yy += 8)
    if (i0 + yy < d_in && j0 + tx < d_c) tile[yy][tx] = W[(i0 + yy) * d_c + j0 + tx];
  __syncthreads();
  for (int yy = ty; yy < 32; yy += 8)
    if (j0 + yy < d_c && i0 + tx < d_in) Wt[(int64_t)(j0 + yy) * d_in + i0 + tx] = tile[tx][yy];
}

}  // namespace

int launch_pack_weights(const void* W, int64_t d_in, int d_c, int dtype, void* Wt, hipStream_t st) {
  const dim3 grid((unsigned)((d_in + 31) / 32), (unsigned)((d_c + 31) / 32));
  if (dtype == ESA_BF16) pack_weights<bf16_t><<<grid, 256, 0, st>>>((const bf16_t*)W, d_in, d_c, (bf16_t*)Wt);
  else pack_weights<float><<<grid, 256, 0, st>>>((const float*)W, d_in, d_c, (float*)Wt);
  ESA_LAUNCH_CHECK("pack_weights");
  return ESA_OK;
}

namespace {

// Inputs that the packed kernels read 16 bytes at a time.
bool packed_ok(const void* x, int64_t d_in, int64_t ldx, const void* W, int64_t x_bs) {
  return d_in % kPiece == 0 && ldx % 8 == 0 && x_bs % 8 == 0 && (((uintptr_t)x | (uintptr_t)W) % 16 == 0);
}

template <int TT>
int run_packed_tiles(const CompressJob<bf16_t>& j0, const CompressJob<bf16_t>& j1, int n_jobs, int split_jobs, uint32_t n_tok,
                     uint32_t n_rows, int d_c, hipStream_t st) {
  constexpr int kLds = packed_lds_bytes<TT>();
  static OncePerDevice raised;
  const int rc = raise_lds_limit(raised, {(const void*)compress_mfma_packed_bf16<TT>}, kLds, "esa_compress");
  if (rc != ESA_OK) return rc;
  const int row_tiles = (int)((n_rows + 16 * TT - 1) / (16 * TT)), col_tiles = d_c / 16;
  const int64_t padded = row_tiles >= 8 ? (row_tiles + 7) / 8 * 8 : row_tiles;
  const int64_t n_wg = padded * col_tiles * (split_jobs ? n_jobs : 1);
  compress_mfma_packed_bf16<TT><<<dim3((unsigned)n_wg), 64 * kPWaves, kLds, st>>>(j0, j1, n_jobs, split_jobs, n_tok, n_rows,
                                                                                      row_tiles, col_tiles);
  ESA_LAUNCH_CHECK("compress");
  return ESA_OK;
}

// bf16 with packed weights, one input or two.
int run_packed(const CompressJob<bf16_t>& j0, const CompressJob<bf16_t>& j1, int n_jobs, int64_t n_tok, int d_c, int batch, hipStream_t st) {
  if (n_tok <= kFewTok && batch <= kFewBatch) {
    compress_few_packed_bf16<<<dim3(d_c, n_jobs, batch), 256, 0, st>>>(j0, j1, (int)n_tok);
    ESA_LAUNCH_CHECK("compress");
    return ESA_OK;
  }
  const uint32_t n_rows = (uint32_t)(n_tok * batch);
  const int64_t tiles = ((int64_t)n_rows + 15) / 16 * (d_c / 16);
  // Sixteen rows per workgroup while those fit the chip at one workgroup per compute unit (each brings 32 rows of d_in
  // in); beyond, thirty-two rows (48 rows for twice the work).  Both inputs in one workgroup, unless compute units
  // would stay idle.
  if (tiles > 256) return run_packed_tiles<2>(j0, j1, n_jobs, 0, (uint32_t)n_tok, n_rows, d_c, st);
  return run_packed_tiles<1>(j0, j1, n_jobs, n_jobs == 2 && 2 * tiles <= 256, (uint32_t)n_tok, n_rows, d_c, st);
}

// The kernel for every storage type, shape and alignment; job 1 may repeat job 0 (n_jobs = 1).
template <typename T>
void run_compress_fma(const CompressJob<T>& j0, const CompressJob<T>& j1, int n_jobs, int64_t n_tok, int d_c, bool packed, int batch,
                      hipStream_t st) {
  const dim3 grid((unsigned)((n_tok + kTok - 1) / kTok), n_jobs * (d_c / kCols), batch);
  if (packed) compress_fma<T, true><<<grid, 1024, 0, st>>>(j0, j1, n_tok, d_c, d_c / kCols);
  else compress_fma<T, false><<<grid, 1024, 0, st>>>(j0, j1, n_tok, d_c, d_c / kCols);
}

}  // namespace

int launch_compress(const void* x, int64_t n_tok, int64_t d_in, int64_t ldx, const void* W, int w_layout,
                    const void* bias, int d_c, void* out, int64_t ldo, int dtype, int batch, int64_t x_bs,
                    int64_t out_bs, hipStream_t st) {
  const bool packed = (w_layout == ESA_W_PACKED);
  if (dtype == ESA_BF16) {
    const bool vec_ok = (ldx % 8 == 0) && (x_bs % 8 == 0) && (((uintptr_t)x | (uintptr_t)W) % 16 == 0);
    const CompressJob<bf16_t> job{(const bf16_t*)x, (const bf16_t*)W, (const bf16_t*)bias, (bf16_t*)out, d_in, ldx, ldo, x_bs, out_bs};
    if (packed && d_c % 16 == 0 && packed_ok(x, d_in, ldx, W, x_bs) && n_tok * batch < ((int64_t)1 << 31)) {
      return run_packed(job, job, 1, n_tok, d_c, batch, st);
    } else if (!packed && vec_ok && (d_c % kMCols == 0) && (d_in % kMStep == 0)) {
      compress_mfma_bf16<<<dim3((unsigned)((n_tok + kMTok - 1) / kMTok), d_c / kMCols, batch), 256, 0, st>>>(
          (const bf16_t*)x, n_tok, d_in, ldx, (const bf16_t*)W, (const bf16_t*)bias, d_c, (bf16_t*)out, ldo, x_bs,
          out_bs);
    } else {
      run_compress_fma<bf16_t>(job, job, 1, n_tok, d_c, packed, batch, st);
    }
  } else {
    const CompressJob<float> job{(const float*)x, (const float*)W, (const float*)bias, (float*)out, d_in, ldx, ldo, x_bs, out_bs};
    run_compress_fma<float>(job, job, 1, n_tok, d_c, packed, batch, st);
  }
  ESA_LAUNCH_CHECK("compress");
  return ESA_OK;
}

// Two inputs in one launch when both take the same kernel (packed bf16, or fp32); otherwise one launch each.
int launch_compress_pair(const void* x0, int64_t d_in0, int64_t ldx0, const void* W0, const void* bias0, void* out0,
                         int64_t ldo0, int64_t x0_bs, int64_t out0_bs, const void* x1, int64_t d_in1, int64_t ldx1,
                         const void* W1, const void* bias1, void* out1, int64_t ldo1, int64_t x1_bs, int64_t out1_bs,
                         int64_t n_tok, int d_c, int w_layout, int dtype, int batch, hipStream_t st) {
  if (dtype == ESA_BF16 && w_layout == ESA_W_PACKED && d_c % 16 == 0 && n_tok * batch < ((int64_t)1 << 31) &&
      packed_ok(x0, d_in0, ldx0, W0, x0_bs) && packed_ok(x1, d_in1, ldx1, W1, x1_bs)) {
    const CompressJob<bf16_t> j0{(const bf16_t*)x0, (const bf16_t*)W0, (const bf16_t*)bias0, (bf16_t*)out0, d_in0, ldx0, ldo0, x0_bs, out0_bs};
    const CompressJob<bf16_t> j1{(const bf16_t*)x1, (const bf16_t*)W1, (const bf16_t*)bias1, (bf16_t*)out1, d_in1, ldx1, ldo1, x1_bs, out1_bs};
    return run_packed(j0, j1, 2, n_tok, d_c, batch, st);
  }
  if (dtype == ESA_F32) {
    const CompressJob<float> j0{(const float*)x0, (const float*)W0, (const float*)bias0, (float*)out0, d_in0, ldx0, ldo0, x0_bs, out0_bs};
    const CompressJob<float> j1{(const float*)x1, (const float*)W1, (const float*)bias1, (float*)out1, d_in1, ldx1, ldo1, x1_bs, out1_bs};
    run_compress_fma<float>(j0, j1, 2, n_tok, d_c, w_layout == ESA_W_PACKED, batch, st);
    ESA_LAUNCH_CHECK("compress (fp32 pair)");
    return ESA_OK;
  }
  const int rc = launch_compress(x0, n_tok, d_in0, ldx0, W0, w_layout, bias0, d_c, out0, ldo0, dtype, batch, x0_bs, out0_bs, st);
  if (rc != ESA_OK) return rc;
  return launch_compress(x1, n_tok, d_in1, ldx1, W1, w_layout, bias1, d_c, out1, ldo1, dtype, batch, x1_bs, out1_bs, st);
}

}  // namespace esa

// Rotary position encoding of query / key rows (Section 3.2 re-encodes positions per step: local
// keys and queries in order, global queries at one fixed position, initial and selected keys at
// position 0, which is the identity).  Rotate-half pairing: element i of a head's first half and
// element i of its second half turn by the angle pos * base^(-2i/d).
//
// The arithmetic is fp64 end to end and rounds once into the storage type, so a row encoded here
// equals the fp64 definition rounded to storage.  What bounds it is that arithmetic as much as the memory traffic
// (re-encoded decode, batch 8: 16392 key rows of 2 KB, 67 MB): with a power, a sine and a cosine per row and frequency,
// their table read again for every head, and a rounding from fp64 to bf16 in 64-bit integer steps it took 31.5 us.  Now
// the frequencies and the turn from one row to the next come from the host (fp64 too, kept per thread for a base and
// head size), a thread evaluates sine and cosine for the first of its few consecutive rows and turns the others by complex
// multiplication (a handful of errors of 2^-53), and the heads of a row share the pairs held in registers.
// fp32 products of the same angles take 9.2 us (512 queries twice and 4608 keys, 31 MB; fp64 12.4), but put an element of every
// hundredth row on the other side of a rounding.  Checked against their error bound and done again in fp64 where it leaves the rounding
// open (one element in a thousand, so two instructions of a wave in three), they take what fp64 takes.
#include <cmath>

#include "esa_common.h"

namespace esa {
namespace {

typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

constexpr int kMaxHalf = 128;
// Angle per position of every frequency, and its cosine and sine for one turn of `step` positions.
struct Turns {
  double freq[kMaxHalf], c[kMaxHalf], s[kMaxHalf];
};
struct RopeJobs {
  RopeJob j[kMaxRopeJobs];
};

template <typename T> __device__ __forceinline__ double load_f64(T v);
template <> __device__ __forceinline__ double load_f64<float>(float v) { return (double)v; }
template <> __device__ __forceinline__ double load_f64<bf16_t>(bf16_t v) { return (double)bf16_to_f32(v); }

// Results rounded into storage.
template <int N> __device__ __forceinline__ void store_f64(float* p, const double (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) p[i] = (float)v[i];
}
template <int N> __device__ __forceinline__ void store_f64(bf16_t* p, const double (&v)[N]) {
  float f[N];
  narrow_for_bf16(v, f);
#pragma unroll
  for (int i = 0; i < N; i += 2) *(uint32_t*)(p + i) = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{f[i], f[i + 1]}), bf16x2));
}

constexpr int kRopeRows = 16;     // most rows of a workgroup
constexpr int kAhead = 4;         // heads whose loads a thread has in flight
// Pairs whose roundings share a branch: with one for every element, 512 queries twice and 4608 keys took 13.5 us; four pairs 12.4, eight 12.6.
constexpr int kTogether = 4;
// Rows of a workgroup, of at most `budget` rows x heads: fewer of the wide ones, so that a thread has one or two rounds
// of kAhead heads to turn (every round is a round trip to memory, and a chunk's queries are few rows of many heads).
__host__ __device__ inline int rows_of(int heads, int budget) {
  int r = kRopeRows;
  while (r > 1 && r * heads > budget) r /= 2;
  return r;
}

// A table of turns instead of rows, cosine and sine for each frequency: of one position, then of every multiple of d / 8.
__device__ __forceinline__ void write_turns(double* out, int64_t row, int i, int half, double freq) {
  const double pos = row == 0 ? 1.0 : (double)((row - 1) * (half / 4));
  double c = 1.0, s = 0.0;
  if (pos != 0.0) sincos(pos * freq, &s, &c);
  out[(row * half + i) * 2] = c;
  out[(row * half + i) * 2 + 1] = s;
}

// grid (groups of rows, jobs, batch); 256 threads.  The rows' angles go through LDS once; then a thread owns VEC
// consecutive pairs of a row (VEC elements = 16 bytes per access when VEC > 1; VEC == 1 serves unaligned rows) for all of
// the row's heads, or for every hs-th of them where there are too few rows to go round.
template <typename T, int VEC>
__global__ __launch_bounds__(256) void rope_rows(RopeJobs jobs, Turns turns, int d, int budget) {
  extern __shared__ double cs[];                       // [kRopeRows][d/2] cosines, then sines
  const RopeJob jb = jobs.j[blockIdx.y];
  const int wg_rows = jb.rotate == kRopeTurns ? 512 / d : rows_of(jb.heads, budget);
  const int64_t row0 = (int64_t)blockIdx.x * wg_rows;
  if (row0 >= jb.n_tok) return;
  const int n_rows = jb.n_tok - row0 < wg_rows ? (int)(jb.n_tok - row0) : wg_rows;
  const int half = d >> 1, tid = threadIdx.x;
  if (jb.rotate == kRopeTurns) {          // one table for all batch entries, a sine and a cosine to a thread
    const int g = tid / half;
    if (blockIdx.z == 0 && g < n_rows) write_turns((double*)jb.out, row0 + g, tid % half, half, turns.freq[tid % half]);
    return;
  }
  const T* x = (const T*)jb.x + (int64_t)blockIdx.z * jb.x_bs + row0 * jb.ldx;
  T* o = (T*)jb.out + (int64_t)blockIdx.z * jb.out_bs + row0 * jb.ldo;
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  if (!jb.rotate) {                       // plain copy of the rows
    const int n = jb.heads * d / VEC;     // d is a multiple of VEC
    for (int e = tid; e < n_rows * n; e += 256)
      *(vec_t*)(o + (int64_t)(e / n) * jb.ldo + e % n * VEC) = *(const vec_t*)(x + (int64_t)(e / n) * jb.ldx + e % n * VEC);
    return;
  }
  double* sn = cs + kRopeRows * half;
  {
    const int groups = 256 / half, i = tid % half, g = tid / half;        // half is a power of two, at most kMaxHalf
    const int per = groups < wg_rows ? wg_rows / groups : 1;              // consecutive rows of a thread
    const int first = g * per;
    if (first < n_rows) {
      const double pos = jb.pos0 + (double)(row0 + first) * jb.pos_step;
      double c = 1.0, s = 0.0;
      if (pos != 0.0) sincos(pos * turns.freq[i], &s, &c);
      const bool turning = jb.pos_step != 0.0;
      const double dc = turning ? turns.c[i] : 1.0, ds = turning ? turns.s[i] : 0.0;
      for (int r = first; r < first + per && r < n_rows; ++r) {
        cs[r * half + i] = c;
        sn[r * half + i] = s;
        const double c2 = c * dc - s * ds;
        s = s * dc + c * ds;
        c = c2;
      }
    }
  }
  __syncthreads();
  const int n_vecs = half / VEC;                       // half is a multiple of VEC
  int hs = 1;
  while (hs < jb.heads && n_rows * n_vecs * hs < 256) hs *= 2;
  for (int e = tid; e < n_rows * n_vecs * hs; e += 256) {
    const int i = e % n_vecs * VEC, r = e / n_vecs % n_rows, h0 = e / (n_vecs * n_rows);
    double c[VEC], s[VEC];
#pragma unroll
    for (int k = 0; k < VEC; ++k) {
      c[k] = cs[r * half + i + k];
      s[k] = sn[r * half + i + k];
    }
    const T* xr = x + (int64_t)r * jb.ldx + i;
    T* orow = o + (int64_t)r * jb.ldo + i;
    for (int hb = h0; hb < jb.heads; hb += hs * kAhead) {
      vec_t a[kAhead], b[kAhead];
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int h = hb + u * hs < jb.heads ? hb + u * hs : hb;
        a[u] = *(const vec_t*)(xr + h * d);
        b[u] = *(const vec_t*)(xr + h * d + half);
      }
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int h = hb + u * hs;
        if (h >= jb.heads) break;
        if constexpr (VEC > 1) {
          vec_t r2[2];                                 // the turned pairs' first and second halves
#pragma unroll
          for (int k = 0; k < VEC; k += kTogether) {
            double v[2 * kTogether];
#pragma unroll
            for (int j = 0; j < kTogether; ++j) {
              const double a0 = load_f64<T>(a[u][k + j]), b0 = load_f64<T>(b[u][k + j]);
              v[j] = a0 * c[k + j] - b0 * s[k + j];
              v[kTogether + j] = b0 * c[k + j] + a0 * s[k + j];
            }
            T out[2 * kTogether] __attribute__((aligned(16)));
            store_f64(out, v);
#pragma unroll
            for (int j = 0; j < kTogether; ++j) {
              r2[0][k + j] = out[j];
              r2[1][k + j] = out[kTogether + j];
            }
          }
          *(vec_t*)(orow + h * d) = r2[0];
          *(vec_t*)(orow + h * d + half) = r2[1];
        } else {
          const double a0 = load_f64<T>(a[u][0]), b0 = load_f64<T>(b[u][0]);
          __attribute__((aligned(8))) T both[2];
          const double v[2] = {a0 * c[0] - b0 * s[0], b0 * c[0] + a0 * s[0]};
          store_f64(both, v);
          orow[h * d] = both[0];
          orow[h * d + half] = both[1];
        }
      }
    }
  }
}

const Turns& turns_for(double base, int d, double step) {
  struct Kept {
    double base = 0.0, step = 0.0;
    int d = 0;
    Turns t;
  };
  static thread_local Kept k;
  if (k.base != base || k.d != d || k.step != step) {
    k.base = base;
    k.d = d;
    k.step = step;
    for (int i = 0; i < d / 2; ++i) {
      k.t.freq[i] = std::pow(base, -2.0 * (double)i / (double)d);
      k.t.c[i] = std::cos(step * k.t.freq[i]);
      k.t.s[i] = std::sin(step * k.t.freq[i]);
    }
  }
  return k.t;
}

}  // namespace

bool rope_head_size_ok(int d) { return d >= 2 && d <= 256 && (d & (d - 1)) == 0; }

int launch_rope_jobs(const RopeJob* jobs, int n_jobs, int d, double base, int dtype, int batch, hipStream_t st) {
  RopeJobs js;
  double step = 0.0;      // the jobs' common step (a job may also stand still)
  int64_t rows = 0;
  for (int k = 0; k < kMaxRopeJobs; ++k) {
    js.j[k] = jobs[k < n_jobs ? k : 0];
    if (k >= n_jobs) js.j[k].n_tok = 0;
    if (js.j[k].n_tok > rows) rows = js.j[k].n_tok;
    if (k < n_jobs && js.j[k].rotate == 1 && js.j[k].pos_step != 0.0) {
      if (step != 0.0 && step != js.j[k].pos_step) ESA_FAIL(ESA_EINVAL, "rope: jobs of one launch share their step");
      step = js.j[k].pos_step;
    }
  }
  if (rows == 0) return ESA_OK;
  const Turns& turns = turns_for(base, d, step);
  // Groups of rows: of the longest job, and of all.
  struct Groups {
    int64_t most, all;
  };
  auto groups_of = [&](int budget) {
    Groups g = {0, 0};
    for (int k = 0; k < n_jobs; ++k) {
      const int r = jobs[k].rotate == kRopeTurns ? 512 / d : rows_of(jobs[k].heads, budget);
      const int64_t n = (jobs[k].n_tok + r - 1) / r;
      g.most = n > g.most ? n : g.most;
      g.all += n;
    }
    return g;
  };
  // Sixteen bf16 rows of eight heads share their sines and cosines best; eight where that would leave compute units without
  // work (batch 8: 18.6 against 20.0 us; a chunk of 512 behind a window of 4096: 14.2 against 12.6 us), four where even
  // those are fewer than two groups per compute unit (64 rows of 32 heads 5.1 -> 4.2, 512 of them 5.8 -> 5.2).  fp32 rows are
  // twice as long: always eight (20000 rows 33.2 -> 26.7).
  int budget = 64;
  if (dtype == ESA_BF16) budget = groups_of(64).all * batch < 512 ? 32 : groups_of(128).most * batch >= 512 ? 128 : 64;
  const int64_t groups = groups_of(budget).most;
  const dim3 grid((unsigned)groups, n_jobs, batch);
  const size_t lds = (size_t)kRopeRows * d * sizeof(double);
  // 16-byte accesses when every row of every job starts on a 16-byte boundary
  const int vec = dtype == ESA_BF16 ? 8 : 4;
  bool wide = (d / 2) % vec == 0;
  for (int k = 0; k < n_jobs; ++k) {
    const RopeJob& j = jobs[k];
    if (j.rotate == kRopeTurns) continue;
    wide = wide && ((uintptr_t)j.x % 16 == 0) && ((uintptr_t)j.out % 16 == 0) && j.ldx % vec == 0 && j.ldo % vec == 0 &&
           j.x_bs % vec == 0 && j.out_bs % vec == 0;
  }
  if (dtype == ESA_BF16) {
    if (wide)
      rope_rows<bf16_t, 8><<<grid, 256, lds, st>>>(js, turns, d, budget);
    else
      rope_rows<bf16_t, 1><<<grid, 256, lds, st>>>(js, turns, d, budget);
  } else {
    if (wide)
      rope_rows<float, 4><<<grid, 256, lds, st>>>(js, turns, d, budget);
    else
      rope_rows<float, 1><<<grid, 256, lds, st>>>(js, turns, d, budget);
  }
  ESA_LAUNCH_CHECK("rope_rows");
  return ESA_OK;
}

}  // namespace esa

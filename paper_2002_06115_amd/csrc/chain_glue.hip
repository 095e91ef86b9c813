// chain_glue.hip -- column-wise operations between the hops of a multi-hop
// chain (Sec. 3.2): softmax over relations, L1 normalisation of entity
// weights, softmax cross-entropy of the last hop, and their backwards.
//
// Every operation reduces over the n rows of each column of an [n][b]
// batch-contiguous array and then writes an [n][b] array.  A workgroup owns
// TW consecutive columns: THREADS / TW row phases of TW lanes, phase p taking
// rows p, p + P, p + 2P, ... of its range in that order, the loads of kDepth
// such rows issued before their values are used.  The phases' partial values
// of a column are combined by shuffles inside each wavefront and through LDS
// across them, in a fixed order.  Sums and maxima are taken in double, so
// results are bitwise reproducible.
//
// Short columns (one launch): the workgroup reduces its columns over all rows
// and writes them.  Bound by latency (dependent passes over a few hundred KB),
// so tiles are 4 columns wide where that gives more workgroups (see launch): 1000
// rows of 256 columns, L1 normalisation 10.2 -> 7.3 us, cross-entropy 27.2 -> 12.1
// (with 16-column tiles, a barrier per tree level and four passes before).
//
// Long columns (two launches, with the caller's scratch): the rows are cut
// into ranges, one workgroup per tile and range; the first launch writes each
// range's partial values, the second combines them (every workgroup for its
// own columns, the same order everywhere) and writes its range.  43,000 rows of
// 128 columns (22 MB), L1 normalisation 317 -> 26 us, its backward 333 -> 26,
// cross-entropy 977 -> 45 (with 8 workgroups of 16 columns over all rows before):
// 1.5 to 1.7 TB/s of the bytes they cannot do without, 4 bytes a lane and four
// rows deep.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "kbchain.h"

namespace {

constexpr int kDepth = 4;          // rows of one thread whose loads are in flight together
constexpr int kLongThreads = 256;  // workgroups of the two-launch path

// The rows and the column a thread works on.
struct Span {
  int64_t begin, end;  // rows begin, begin + step, ... below end
  int64_t step;
  int64_t last;        // the workgroup's last row: where loads past the end go
  int col;             // column (may be >= b: idle, but joins every barrier)
  bool valid;          // col < b, and the workgroup has rows
};

template <int TW, int THREADS>
__device__ __forceinline__ Span span(int64_t r0, int64_t r1, int32_t b, uint32_t tile) {
  Span s;
  const uint32_t col = tile * TW + threadIdx.x % TW;  // below 2^31 + 2^8
  s.col = col < (uint32_t)b ? (int)col : b;
  s.begin = r0 + (int64_t)(threadIdx.x / TW);
  s.end = r1;
  s.step = THREADS / TW;
  s.last = r1 - 1;
  s.valid = s.col < b && r0 < r1;
  return s;
}

// NaN wins, as in every maximum here.
__device__ __forceinline__ double max_nan(double a, double w) {
  return (w > a || w != w) ? w : a;
}

// Sums (MAX: maxima) of K values over the threads of each column, returned to
// all of them: shuffles over the phases of a wavefront, then the wavefronts'
// values in order.
template <int TW, int THREADS, int K, bool MAX>
__device__ __forceinline__ void combine(double (&v)[K], double *lds) {
  static_assert(TW <= 64 && THREADS % 64 == 0, "a wavefront holds whole phases");
  constexpr int kWaves = THREADS / 64;
#pragma unroll
  for (int m = TW; m < 64; m <<= 1)
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const double w = __shfl_xor(v[k], m);
      v[k] = MAX ? max_nan(v[k], w) : v[k] + w;
    }
  if constexpr (kWaves > 1) {
    const int c = threadIdx.x % TW, w = threadIdx.x / 64;
    __syncthreads();  // earlier readers of lds are done
    if (threadIdx.x % 64 < TW)
#pragma unroll
      for (int k = 0; k < K; ++k) lds[(k * kWaves + w) * TW + c] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      double acc = lds[(k * kWaves) * TW + c];
      for (int i = 1; i < kWaves; ++i) {
        const double x = lds[(k * kWaves + i) * TW + c];
        acc = MAX ? max_nan(acc, x) : acc + x;
      }
      v[k] = acc;
    }
  }
}

// f(i, k) for the thread's rows i, in order; `load(i, k)` puts row i's values in
// place k of the kDepth in flight.
template <class L, class F>
__device__ __forceinline__ void each_row(const Span &s, L load, F f) {
  if (!s.valid) return;
  for (int64_t i0 = s.begin; i0 < s.end; i0 += s.step * kDepth) {
#pragma unroll
    for (int k = 0; k < kDepth; ++k) {
      const int64_t i = i0 + k * s.step;
      load(i < s.end ? i : s.last, k);
    }
#pragma unroll
    for (int k = 0; k < kDepth; ++k)
      if (i0 + k * s.step < s.end) f(i0 + k * s.step, k);
  }
}

// -- what each operation reduces -------------------------------------------------

// Sum of a column, or of the products of two.
__device__ __forceinline__ double sum_part(const Span &s, int32_t b, const float *u) {
  float v[kDepth];
  double acc = 0.0;
  each_row(s, [&](int64_t i, int k) { v[k] = u[i * b + s.col]; },
           [&](int64_t, int k) { acc += (double)v[k]; });
  return acc;
}
__device__ __forceinline__ double dot_part(const Span &s, int32_t b, const float *x,
                                           const float *y) {
  float v[kDepth], w[kDepth];
  double acc = 0.0;
  each_row(
      s,
      [&](int64_t i, int k) {
        v[k] = x[i * b + s.col];
        w[k] = y[i * b + s.col];
      },
      [&](int64_t, int k) { acc += (double)w[k] * (double)v[k]; });
  return acc;
}

// The statistics of a softmax over part of a column, in one pass: the maximum
// m, s = sum of exp(z - m) and, for the cross-entropy, the sum ts of the targets
// and td = sum of t (z - m).  Where m rises, s and td move to the new m.  (An
// m of -inf has seen no finite value: s stays 0, td takes z itself.)
struct Stats {
  double m, s, ts, td;
};
__device__ __forceinline__ void rebase(Stats &a, double m) {
  if (a.m == m) return;
  if (a.m != -INFINITY) {
    a.s *= exp(a.m - m);
    a.td += (a.m - m) * a.ts;
  }
  a.m = m;
}
template <bool XENT>
__device__ __forceinline__ Stats stats_part(const Span &s, int32_t b, const float *z,
                                            const float *t) {
  Stats a = {-INFINITY, 0.0, 0.0, 0.0};
  if (!s.valid) return a;
  for (int64_t i0 = s.begin; i0 < s.end; i0 += s.step * kDepth) {
    float v[kDepth], w[kDepth];
    double m = a.m;
#pragma unroll
    for (int k = 0; k < kDepth; ++k) {
      const int64_t i = i0 + k * s.step, r = i < s.end ? i : s.last;
      v[k] = z[r * b + s.col];
      if constexpr (XENT) w[k] = t[r * b + s.col];
    }
#pragma unroll
    for (int k = 0; k < kDepth; ++k)
      if (i0 + k * s.step < s.end) m = max_nan(m, (double)v[k]);
    rebase(a, m);
#pragma unroll
    for (int k = 0; k < kDepth; ++k)
      if (i0 + k * s.step < s.end) {
        const double d = m == -INFINITY ? (double)v[k] : (double)v[k] - m;
        if (m != -INFINITY) a.s += exp(d);
        if constexpr (XENT) {
          a.ts += (double)w[k];
          a.td += (double)w[k] * d;
        }
      }
  }
  return a;
}
// The statistics of whole columns from the threads' parts.
template <int TW, int THREADS, bool XENT>
__device__ __forceinline__ Stats stats_combine(Stats a, double *lds) {
  double m[1] = {a.m};
  combine<TW, THREADS, 1, true>(m, lds);
  rebase(a, m[0]);
  if constexpr (XENT) {
    double v[3] = {a.s, a.ts, a.td};
    combine<TW, THREADS, 3, false>(v, lds);
    return {m[0], v[0], v[1], v[2]};
  } else {
    double v[1] = {a.s};
    combine<TW, THREADS, 1, false>(v, lds);
    return {m[0], v[0], 0.0, 0.0};
  }
}

// -- the operations ----------------------------------------------------------------

enum Op { kSoftmax, kSoftmaxBackward, kL1, kL1Backward, kXent };

struct Args {
  int64_t n;
  int32_t b;
  const float *x, *y;    // inputs: z | p, dp | u | x, dx | z, t
  double *col;           // sums (written by kL1, read by kL1Backward) | col_loss
  float *out;
  double *part;          // two launches: [value][range][b]
  int64_t rows_per;      // two launches: rows of one range
  int32_t ranges;
};

template <int OP>
constexpr int kValues = OP == kXent ? 4 : OP == kSoftmax ? 2 : 1;

// The thread's share of what OP reduces.
template <int OP>
__device__ __forceinline__ Stats reduce_part(const Args &a, const Span &s) {
  if constexpr (OP == kSoftmax || OP == kXent)
    return stats_part<OP == kXent>(s, a.b, a.x, a.y);
  else if constexpr (OP == kL1)
    return {0.0, sum_part(s, a.b, a.x), 0.0, 0.0};
  else
    return {0.0, dot_part(s, a.b, a.x, a.y), 0.0, 0.0};
}

template <int OP, int TW, int THREADS>
__device__ __forceinline__ Stats reduce_combine(const Stats &p, double *lds) {
  if constexpr (OP == kSoftmax || OP == kXent) {
    return stats_combine<TW, THREADS, OP == kXent>(p, lds);
  } else {
    double v[1] = {p.s};
    combine<TW, THREADS, 1, false>(v, lds);
    return {0.0, v[0], 0.0, 0.0};
  }
}

// Writes the thread's rows of the output (and, by one thread per column, the
// column's own value) from the column's reduced values.
template <int OP>
__device__ __forceinline__ void apply(const Args &a, const Span &s, const Stats &r, bool first) {
  const int32_t b = a.b;
  const int col = s.col;
  float v[kDepth], w[kDepth];
  auto load1 = [&](int64_t i, int k) { v[k] = a.x[i * b + col]; };
  auto load2 = [&](int64_t i, int k) {
    v[k] = a.x[i * b + col];
    w[k] = a.y[i * b + col];
  };
  if constexpr (OP == kSoftmax) {
    const double inv = 1.0 / r.s;
    each_row(s, load1,
             [&](int64_t i, int k) { a.out[i * b + col] = (float)(exp((double)v[k] - r.m) * inv); });
  } else if constexpr (OP == kSoftmaxBackward) {
    each_row(s, load2, [&](int64_t i, int k) {
      a.out[i * b + col] = (float)((double)v[k] * ((double)w[k] - r.s));
    });
  } else if constexpr (OP == kL1) {
    if (first) a.col[col] = r.s;
    const double inv = 1.0 / r.s;
    each_row(s, load1, [&](int64_t i, int k) { a.out[i * b + col] = (float)((double)v[k] * inv); });
  } else if constexpr (OP == kL1Backward) {
    if (!s.valid) return;
    const double inv = 1.0 / a.col[col];
    each_row(s, load2, [&](int64_t i, int k) {
      a.out[i * b + col] = (float)(((double)w[k] - r.s) * inv);
    });
  } else {
    if (first) a.col[col] = -(r.td - log(r.s) * r.ts);
    const double inv_b = 1.0 / (double)b, scale = r.ts / r.s;
    each_row(s, load2, [&](int64_t i, int k) {
      a.out[i * b + col] = (float)((exp((double)v[k] - r.m) * scale - (double)w[k]) * inv_b);
    });
  }
}

// One launch: all rows of TW columns.  Tiles that share cache lines are on one
// XCD (workgroup w runs on XCD w mod 8; a grid of more than 8 is a multiple of
// 8): in order,
// every XCD's L2 fetched every line, which cost wide arrays up to 3.5 times the
// time (1000 rows of 2048 columns, 4-column tiles, softmax backward 46 -> 12 us).
constexpr uint32_t kXcds = 8;
template <int OP, int TW, int THREADS>
__global__ __launch_bounds__(THREADS) void column_kernel(Args a) {
  __shared__ double lds[3 * (THREADS / 64) * TW];
  const uint32_t share = (gridDim.x + kXcds - 1) / kXcds;
  const Span s =
      span<TW, THREADS>(0, a.n, a.b, blockIdx.x % kXcds * share + blockIdx.x / kXcds);
  const Stats r = reduce_combine<OP, TW, THREADS>(reduce_part<OP>(a, s), lds);
  apply<OP>(a, s, r, s.valid && threadIdx.x < TW);
}

// Two launches: this range's partial values, then the column's from all ranges
// and this range of the output.
template <int OP, int TW>
__global__ __launch_bounds__(kLongThreads) void range_kernel(Args a) {
  __shared__ double lds[3 * (kLongThreads / 64) * TW];
  const int64_t r0 = (int64_t)blockIdx.y * a.rows_per;
  const Span s = span<TW, kLongThreads>(r0, min(a.n, r0 + a.rows_per), a.b, blockIdx.x);
  const Stats r = reduce_combine<OP, TW, kLongThreads>(reduce_part<OP>(a, s), lds);
  if (!(s.col < a.b) || threadIdx.x >= TW) return;
  double *p = a.part + (int64_t)blockIdx.y * a.b + s.col;
  const int64_t plane = (int64_t)a.ranges * a.b;
  p[0] = r.s;
  if constexpr (kValues<OP> > 1) p[plane] = r.m;
  if constexpr (kValues<OP> > 2) {
    p[2 * plane] = r.ts;
    p[3 * plane] = r.td;
  }
}

template <int OP, int TW>
__global__ __launch_bounds__(kLongThreads) void apply_kernel(Args a) {
  __shared__ double lds[3 * (kLongThreads / 64) * TW];
  const int64_t r0 = (int64_t)blockIdx.y * a.rows_per;
  const Span s = span<TW, kLongThreads>(r0, min(a.n, r0 + a.rows_per), a.b, blockIdx.x);
  constexpr int kPhases = kLongThreads / TW;
  const int64_t plane = (int64_t)a.ranges * a.b;
  Stats p = {OP == kSoftmax || OP == kXent ? -INFINITY : 0.0, 0.0, 0.0, 0.0};
  if (s.col < a.b) {
    const double *q = a.part + s.col;
    if constexpr (kValues<OP> > 1)
      for (int k = (int)(threadIdx.x / TW); k < a.ranges; k += kPhases)
        p.m = max_nan(p.m, q[plane + (int64_t)k * a.b]);
    for (int k = (int)(threadIdx.x / TW); k < a.ranges; k += kPhases) {
      const double *qk = q + (int64_t)k * a.b;
      Stats o = {p.m, qk[0], 0.0, 0.0};
      if constexpr (kValues<OP> > 2) o = {p.m, qk[0], qk[2 * plane], qk[3 * plane]};
      if constexpr (kValues<OP> > 1) {
        o.m = qk[plane];
        rebase(o, p.m);
      }
      p.s += o.s;
      p.ts += o.ts;
      p.td += o.td;
    }
  }
  const Stats r = reduce_combine<OP, TW, kLongThreads>(p, lds);
  apply<OP>(a, s, r, s.valid && threadIdx.x < TW && blockIdx.y == 0);
}

// loss[0] = (col_loss[0] + ... + col_loss[b-1]) / b, added in order.  The
// workgroup stages 1024 values at a time in LDS (one load per thread, all in
// flight together) and thread 0 adds them in index order.
constexpr int kMeanThreads = 1024;

__global__ __launch_bounds__(kMeanThreads) void mean_kernel(int32_t b,
                                                            const double *__restrict__ col_loss,
                                                            double *__restrict__ loss) {
  __shared__ double stage[kMeanThreads];
  double s = 0.0;
  for (int32_t c0 = 0; c0 < b; c0 += kMeanThreads) {
    const int32_t c = c0 + (int32_t)threadIdx.x;
    __syncthreads();  // thread 0 is done with the previous batch
    stage[threadIdx.x] = c < b ? col_loss[c] : 0.0;
    __syncthreads();
    if (threadIdx.x == 0) {
      const int32_t m = b - c0 < kMeanThreads ? b - c0 : kMeanThreads;
      for (int32_t k = 0; k < m; ++k) s += stage[k];
    }
  }
  if (threadIdx.x == 0) loss[0] = s / (double)b;
}

kbc_status launched() { return hipGetLastError() == hipSuccess ? KBC_OK : KBC_EHIP; }

// -- how a call is launched -----------------------------------------------------------

// Rows from which two launches win over one: 2000 rows of 93 columns take the
// one-launch path 6 to 8 us (softmax 11, cross-entropy 15), 4000 rows of 128 10 to
// 27 (17, 35) against 7 (12, 15) in two launches.
constexpr int64_t kLongRows = 2048;
// Ranges of the two-launch path: about two workgroups per CU over all tiles, and
// at least two rounds of kDepth rows per thread.
constexpr int kMaxRanges = 512;

struct LongPlan {
  int tile;         // columns per workgroup: a power of two, at most 32
  int32_t tiles, ranges;
  int64_t rows_per;
};

LongPlan long_plan(int64_t n, int32_t b) {
  LongPlan p;
  p.tile = 1;
  while (p.tile < 32 && p.tile < b) p.tile <<= 1;
  p.tiles = (int32_t)(((int64_t)b + p.tile - 1) / p.tile);
  const int64_t phases = kLongThreads / p.tile;
  int64_t ranges = (512 + p.tiles - 1) / p.tiles;
  const int64_t most = (n + phases * 2 * kDepth - 1) / (phases * 2 * kDepth);
  ranges = ranges < most ? ranges : most;
  ranges = ranges < kMaxRanges ? ranges : kMaxRanges;
  ranges = ranges > 1 ? ranges : 1;
  p.rows_per = (n + ranges - 1) / ranges;
  p.ranges = (int32_t)((n + p.rows_per - 1) / p.rows_per);
  return p;
}

bool is_long(int64_t n, int32_t b) { return n > kLongRows && long_plan(n, b).ranges > 1; }

size_t scratch_bytes(int64_t n, int32_t b) {
  if (n < 1 || b < 1 || !is_long(n, b)) return 0;
  return (size_t)long_plan(n, b).ranges * (size_t)b * 4 * sizeof(double);
}

template <int OP, int TW>
void launch_long(const Args &a, const LongPlan &p, hipStream_t s) {
  const dim3 grid((unsigned)p.tiles, (unsigned)p.ranges);
  hipLaunchKernelGGL((range_kernel<OP, TW>), grid, dim3(kLongThreads), 0, s, a);
  hipLaunchKernelGGL((apply_kernel<OP, TW>), grid, dim3(kLongThreads), 0, s, a);
}

template <int OP>
kbc_status launch(Args a, double *scratch, hipStream_t s) {
  if (scratch && is_long(a.n, a.b)) {
    const LongPlan p = long_plan(a.n, a.b);
    a.part = scratch;
    a.rows_per = p.rows_per;
    a.ranges = p.ranges;
    switch (p.tile) {
      case 1: launch_long<OP, 1>(a, p, s); break;
      case 2: launch_long<OP, 2>(a, p, s); break;
      case 4: launch_long<OP, 4>(a, p, s); break;
      case 8: launch_long<OP, 8>(a, p, s); break;
      case 16: launch_long<OP, 16>(a, p, s); break;
      default: launch_long<OP, 32>(a, p, s); break;
    }
    return launched();
  }
  auto go = [&](auto kernel, int tw, int threads) {
    int64_t tiles = ((int64_t)a.b + tw - 1) / tw;
    if (tiles > kXcds) tiles = (tiles + kXcds - 1) / kXcds * kXcds;
    hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(threads), 0, s, a);
  };
  // Narrow tiles give a narrow array more workgroups, wide ones read more of each
  // line.  The five operations together, us, with 4 / 8 / 16 columns (512, 512
  // and 1024 threads): 1000 rows of 256 columns 33 / 41 / 59, of 768 42 / 47 / 65,
  // of 1024 50 / 50 / 67, of 4000 138 / 112 / 105; 400 rows of 1024 34 / 35 / 45,
  // of 4000 84 / 73 / 74.  Up to 128 rows give 512 threads too little to do (60 rows
  // of 1024 columns, tiles of 8, 27 -> 25 with 256; of 8000, tiles of 16 and 1024
  // threads, 103 -> 87).
  const bool few = a.n <= 128;
  if (a.n > kLongRows || (a.b >= 4096 && !few))
    go(column_kernel<OP, 16, 1024>, 16, 1024);
  else if (a.b >= 4096)
    go(column_kernel<OP, 16, 256>, 16, 256);
  else if (a.b >= 1024 && !few)
    go(column_kernel<OP, 8, 512>, 8, 512);
  else if (a.b >= 1024)
    go(column_kernel<OP, 8, 256>, 8, 256);
  else if (!few)
    go(column_kernel<OP, 4, 512>, 4, 512);
  else
    go(column_kernel<OP, 4, 256>, 4, 256);
  return launched();
}

bool bad_scratch(int64_t n, int32_t b, const void *scratch, size_t bytes) {
  return scratch && (bytes < scratch_bytes(n, b) || reinterpret_cast<uintptr_t>(scratch) % 8 != 0);
}

}  // namespace

extern "C" {

size_t kbc_scratch_size(int64_t n, int32_t b) { return scratch_bytes(n, b); }

kbc_status kbc_softmax_scratch(int64_t n, int32_t b, const float *z, float *p, void *scratch,
                               size_t bytes, void *stream) {
  if (n < 1 || b < 1 || !z || !p || bad_scratch(n, b, scratch, bytes)) return KBC_EINVAL;
  const Args a{n, b, z, nullptr, nullptr, p, nullptr, 0, 0};
  return launch<kSoftmax>(a, static_cast<double *>(scratch), static_cast<hipStream_t>(stream));
}

kbc_status kbc_softmax_backward_scratch(int64_t n, int32_t b, const float *p, const float *dp,
                                        float *dz, void *scratch, size_t bytes, void *stream) {
  if (n < 1 || b < 1 || !p || !dp || !dz || bad_scratch(n, b, scratch, bytes)) return KBC_EINVAL;
  const Args a{n, b, p, dp, nullptr, dz, nullptr, 0, 0};
  return launch<kSoftmaxBackward>(a, static_cast<double *>(scratch),
                                  static_cast<hipStream_t>(stream));
}

kbc_status kbc_l1_normalize_scratch(int64_t n, int32_t b, const float *u, float *x, double *sums,
                                    void *scratch, size_t bytes, void *stream) {
  if (n < 1 || b < 1 || !u || !x || !sums || bad_scratch(n, b, scratch, bytes)) return KBC_EINVAL;
  const Args a{n, b, u, nullptr, sums, x, nullptr, 0, 0};
  return launch<kL1>(a, static_cast<double *>(scratch), static_cast<hipStream_t>(stream));
}

kbc_status kbc_l1_normalize_backward_scratch(int64_t n, int32_t b, const float *x,
                                             const double *sums, const float *dx, float *du,
                                             void *scratch, size_t bytes, void *stream) {
  if (n < 1 || b < 1 || !x || !sums || !dx || !du || bad_scratch(n, b, scratch, bytes))
    return KBC_EINVAL;
  const Args a{n, b, x, dx, const_cast<double *>(sums), du, nullptr, 0, 0};
  return launch<kL1Backward>(a, static_cast<double *>(scratch), static_cast<hipStream_t>(stream));
}

kbc_status kbc_softmax_xent_scratch(int64_t n, int32_t b, const float *z, const float *t,
                                    double *col_loss, double *loss, float *dz, void *scratch,
                                    size_t bytes, void *stream) {
  if (n < 1 || b < 1 || !z || !t || !col_loss || !loss || !dz ||
      bad_scratch(n, b, scratch, bytes))
    return KBC_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const Args a{n, b, z, t, col_loss, dz, nullptr, 0, 0};
  const kbc_status st = launch<kXent>(a, static_cast<double *>(scratch), s);
  if (st != KBC_OK) return st;
  hipLaunchKernelGGL(mean_kernel, dim3(1), dim3(kMeanThreads), 0, s, b, col_loss, loss);
  return launched();
}

kbc_status kbc_softmax(int64_t n, int32_t b, const float *z, float *p, void *stream) {
  return kbc_softmax_scratch(n, b, z, p, nullptr, 0, stream);
}

kbc_status kbc_softmax_backward(int64_t n, int32_t b, const float *p, const float *dp, float *dz,
                                void *stream) {
  return kbc_softmax_backward_scratch(n, b, p, dp, dz, nullptr, 0, stream);
}

kbc_status kbc_l1_normalize(int64_t n, int32_t b, const float *u, float *x, double *sums,
                            void *stream) {
  return kbc_l1_normalize_scratch(n, b, u, x, sums, nullptr, 0, stream);
}

kbc_status kbc_l1_normalize_backward(int64_t n, int32_t b, const float *x, const double *sums,
                                     const float *dx, float *du, void *stream) {
  return kbc_l1_normalize_backward_scratch(n, b, x, sums, dx, du, nullptr, 0, stream);
}

kbc_status kbc_softmax_xent(int64_t n, int32_t b, const float *z, const float *t,
                            double *col_loss, double *loss, float *dz, void *stream) {
  return kbc_softmax_xent_scratch(n, b, z, t, col_loss, loss, dz, nullptr, 0, stream);
}

}  // extern "C"

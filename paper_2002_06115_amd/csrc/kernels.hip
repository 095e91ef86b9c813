// kernels.hip -- gfx950 kernels for relation-set following on a reified KB.
//
// All three passes (forward Y, backward dX, backward dR; Eq. 4 and its
// gradients) are the same operation on a differently sorted triple list: a
// segmented sum, over the triples of a row, of the elementwise product of two
// gathered b-wide rows,
//
//     out[row] = sum over triples p of the row of  w[p] * A[a[p]] (.) B[b_id[p]]
//
//     forward : rows = objects,   A = X  (a = subject),  B = R  (b_id = relation)
//     dX      : rows = subjects,  A = dY (a = object),   B = R  (b_id = relation)
//     dR      : rows = relations, A = dY (a = object),   B = X  (b_id = subject)
//
// Activations are entity-major and batch-contiguous ([N][b] float32), so each
// gather is one contiguous b-wide row: a lane group of LPT lanes reads it with
// VEC-float (16-byte when VEC = 4) loads, lane l owning columns
// [col0 + l*VEC, col0 + l*VEC + VEC).  The sorted triple list is cut into
// equal chunks and a lane group walks one chunk sequentially, so a row sum
// needs no cross-lane reduction at all: every lane accumulates its own
// columns and writes them when the row ends.  A row that crosses a chunk
// boundary writes one double partial per chunk to a workspace slot and the
// combine kernel adds them up in a fixed order.  No atomics anywhere: every
// output element is written by one lane (by two, with the same bits, in the
// last lanes of rows that are not a multiple of 4 floats), with a fixed
// summation order, so results are bitwise reproducible.  Rows of at most 4
// floats have a kernel of their own (narrow_kernel).
//
// Arithmetic: each product w * a * b is formed in double (the product of two
// floats is exact in double) and accumulated in double; the float output is
// one rounding of that sum.  The work is bound by memory traffic (two gathered
// rows per triple against two flops per element), so the double arithmetic
// costs no time while it keeps long Zipf-hub rows accurate.
#include "kernels.h"
#include "plan.h"

#include <hip/hip_ext.h>

#include <algorithm>
#include <climits>
#include <cstdio>
#include <map>
#include <string>
#include <tuple>
#include <mutex>
#include <utility>

// Structured-buffer loads (LLVM's amdgcn struct buffer load intrinsics): the
// bytes at `off` of record `idx` of a descriptor whose records are `stride`
// bytes apart.  A record index at or past the descriptor's record count
// returns zeros without a memory access, so a gathered row needs no multiply
// for its address and a marker's index (bit 31 set) needs no select.  (At
// file scope: an intrinsic declared by its assembler name needs external
// linkage.)
typedef float kbf_float4 __attribute__((ext_vector_type(4)));
__device__ kbf_float4 struct_buffer_load_f32x4(__amdgpu_buffer_rsrc_t rsrc, int idx, int off,
                                               int soff, int aux)
    __asm("llvm.amdgcn.struct.ptr.buffer.load.v4f32");

namespace kbf {

namespace {

constexpr int kBlock = 256;   // threads per workgroup (4 wavefronts of 64)
constexpr int kMaxLpt = 32;   // widest lane group (column_tiling)
// Workgroups of the stream kernel when the B table sits in LDS: 12 waves,
// so that two workgroups (two copies of a table of up to kMaxLdsB bytes) fill
// a CU at the six waves per SIMD that the kernel's registers allow; 16 waves,
// one workgroup per CU, for a table of up to kMaxLdsBig bytes.  The LDS
// variants are compiled for the larger block and read blockDim at run time.
constexpr int kBlockLds = 768;
constexpr int kBlockLdsBig = 1024;
constexpr int kUnroll = 8;    // entries per step; a lane group keeps their loads in flight
// The residual hop's empty-row fill: pieces per lane group, rows per batch.
constexpr int kFillPieces = 4;
constexpr int kFillBatch = 4;
static_assert(kChunkQuantum % kUnroll == 0, "a chunk is a whole number of steps");
static_assert(kUnroll == kStepEntries, "the planner's kSameA flags assume this step length");

// Buffer-resource word 3 for gfx9-family buffers, and an offset past any raw
// buffer this library makes (such a load returns zeros without touching
// memory; tables are at most this many bytes).
constexpr int kRawBufferWord3 = 0x00020000;
constexpr uint32_t kOutOfRange = 0xFFFFFFF0u;
// Largest record stride of a buffer descriptor (a 14-bit field), in bytes.
constexpr uint64_t kMaxStride = 16383;

// Checked builds (KBFOLLOW_CHECKED) validate every row, slot and combine
// index before it is used: KBF_CHECKED(i, n) is i when 0 <= i < n, else 0 (a
// valid index) with one more count in a device-wide counter, so a planning
// bug shows up as a count instead of an out-of-bounds access.  In normal
// builds KBF_CHECKED(i, n) is just (i): the same code as without checks.
#ifdef KBFOLLOW_CHECKED
__device__ unsigned long long g_violations;
__device__ __forceinline__ int64_t checked(int64_t i, int64_t n) {
  if (i >= 0 && i < n) return i;
  atomicAdd(&g_violations, 1ull);
  return 0;
}
#define KBF_CHECKED(i, n) checked((i), (n))
#else
#define KBF_CHECKED(i, n) (i)
#endif

template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F &f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
// f(std::integral_constant<int, i>) for i = 0 .. N-1, unrolled at compile time.
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// Value of lane SRC of this lane's group of LPT lanes (LPT a power of two,
// at most 32): ds_swizzle's bitmask mode (no LDS memory is touched), source
// lane = (lane & and_mask) | SRC within each 32-lane half.
template <int LPT, int SRC>
__device__ __forceinline__ int group_bcast(int v) {
  static_assert(LPT >= 1 && LPT <= 32 && (LPT & (LPT - 1)) == 0, "lane groups of 1..32");
  if constexpr (LPT == 1) {
    return v;
  } else {
    constexpr int and_mask = 0x1f & ~(LPT - 1);
    return __builtin_amdgcn_ds_swizzle(v, and_mask | (SRC << 5));
  }
}

typedef float native_float4 __attribute__((ext_vector_type(4)));
// The same at any float's / double's address: rows whose width is not a
// multiple of 4 floats start anywhere, and gfx950's 16-byte loads and stores
// take any 4-byte boundary.
typedef float float4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef double double2_any __attribute__((ext_vector_type(2), aligned(8)));

template <int VEC>
__device__ __forceinline__ void load_row(const float *__restrict__ p, float (&v)[VEC]) {
  if constexpr (VEC == 4) {
    const float4_any t = *reinterpret_cast<const float4_any *>(p);
    v[0] = t[0];
    v[1] = t[1];
    v[2] = t[2];
    v[3] = t[3];
  } else {
    v[0] = *p;
  }
}

// Record index that no table of this library reaches.
constexpr uint32_t kNoRecord = 0xFFFFFFFFu;

// 4 floats at byte `off` of record `idx` of a structured buffer (zeros when
// idx is past its last record).
__device__ __forceinline__ void gather_row(__amdgpu_buffer_rsrc_t rsrc, uint32_t idx,
                                           uint32_t off, float (&v)[4]) {
  const native_float4 t = struct_buffer_load_f32x4(rsrc, (int)idx, (int)off, 0, 0);
  v[0] = t[0];
  v[1] = t[1];
  v[2] = t[2];
  v[3] = t[3];
}

// 4 floats at byte offset `off` of a raw buffer (zeros when off is past its end).
__device__ __forceinline__ void load_row_buffer(__amdgpu_buffer_rsrc_t rsrc, uint32_t off,
                                                float (&v)[4]) {
  const auto t = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 0, 0);
  v[0] = __int_as_float(t[0]);
  v[1] = __int_as_float(t[1]);
  v[2] = __int_as_float(t[2]);
  v[3] = __int_as_float(t[3]);
}

// 4 floats of LDS at p (16-byte aligned).
__device__ __forceinline__ void lds_row(const float *p, float (&v)[4]) {
  const native_float4 t = *reinterpret_cast<const native_float4 *>(p);
  v[0] = t[0];
  v[1] = t[1];
  v[2] = t[2];
  v[3] = t[3];
}
// The columns a lane of 4 floats works on, c0 being where its place in the
// row begins (c0 < b).  Rows of b floats, b not a multiple of 4, end in a lane
// whose 4 columns would pass the row's end: it takes the last 4 of the row
// instead (so that every 16-byte load stays inside its row; b >= 5 there).
// The first `skip` of them belong to the lane before it: both compute them,
// the same sums in the same order, bit for bit.  In the stream kernel both
// store them too (one 16-byte store per lane; the same bits from both), unless
// the pass adds rows of Z, which may be the output: there a column is only
// stored by the lane it belongs to, so that no Z is read after its own row was
// written.
struct LaneCols {
  int c;     // first column read
  int skip;  // columns of these that belong to the lane before
};
template <bool RAGGED>
__device__ __forceinline__ LaneCols lane_cols(int c0, int b) {
  if constexpr (RAGGED) {
    const int c = min(c0, b - 4);
    return {c, c0 - c};
  } else {
    return {c0, 0};
  }
}

__device__ __forceinline__ void lds_store(float *p, const float (&v)[4]) {
  *reinterpret_cast<native_float4 *>(p) = native_float4{v[0], v[1], v[2], v[3]};
}

// Output rows are written once and not read again by the pass: non-temporal
// stores keep them from displacing gathered rows in the caches.
template <int VEC>
__device__ __forceinline__ void store_row(float *__restrict__ p, const double (&acc)[VEC]) {
  if constexpr (VEC == 4) {
    const native_float4 v = {(float)acc[0], (float)acc[1], (float)acc[2], (float)acc[3]};
    __builtin_nontemporal_store(v, reinterpret_cast<float4_any *>(p));
  } else {
    __builtin_nontemporal_store((float)acc[0], p);
  }
}

// store_row / store_slot without the first `skip` columns (LaneCols).
template <int VEC>
__device__ __forceinline__ void store_row_from(float *__restrict__ p, const double (&acc)[VEC],
                                               int skip) {
  if (VEC == 1 || skip == 0) {
    store_row<VEC>(p, acc);
  } else {
#pragma unroll
    for (int v = 1; v < VEC; ++v)
      if (v >= skip) __builtin_nontemporal_store((float)acc[v], p + v);
  }
}

template <int VEC>
__device__ __forceinline__ void load_slot(const double *__restrict__ p, double (&v)[VEC]) {
  if constexpr (VEC == 4) {
    const double2_any t0 = reinterpret_cast<const double2_any *>(p)[0];
    const double2_any t1 = reinterpret_cast<const double2_any *>(p)[1];
    v[0] = t0[0];
    v[1] = t0[1];
    v[2] = t1[0];
    v[3] = t1[1];
  } else {
    v[0] = *p;
  }
}

template <int VEC>
__device__ __forceinline__ void store_slot(double *__restrict__ p, const double (&acc)[VEC]) {
  if constexpr (VEC == 4) {
    reinterpret_cast<double2_any *>(p)[0] = double2_any{acc[0], acc[1]};
    reinterpret_cast<double2_any *>(p)[1] = double2_any{acc[2], acc[3]};
  } else {
    *p = acc[0];
  }
}

template <int VEC>
__device__ __forceinline__ void store_slot_from(double *__restrict__ p, const double (&acc)[VEC],
                                                int skip) {
  if (VEC == 1 || skip == 0) {
    store_slot<VEC>(p, acc);
  } else {
#pragma unroll
    for (int v = 1; v < VEC; ++v)
      if (v >= skip) p[v] = acc[v];
  }
}

__device__ __forceinline__ void store_slot_buffer(__amdgpu_buffer_rsrc_t rsrc, uint32_t off,
                                                  const double (&acc)[4]) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  const double2 lo = make_double2(acc[0], acc[1]), hi = make_double2(acc[2], acc[3]);
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, lo), rsrc, (int)off, 0, 0);
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, hi), rsrc, (int)(off + 16), 0,
                                         0);
}

// Stores of 4 floats / doubles at byte offset `off` of a raw buffer; rows
// written once per pass use the non-temporal policy.
constexpr int kNonTemporal = 2;
__device__ __forceinline__ void store_row_buffer(__amdgpu_buffer_rsrc_t rsrc, uint32_t off,
                                                 const double (&y)[4]) {
  const native_float4 v = {(float)y[0], (float)y[1], (float)y[2], (float)y[3]};
  __builtin_amdgcn_raw_buffer_store_b128(
      __builtin_bit_cast(__attribute__((ext_vector_type(4))) unsigned int, v), rsrc, (int)off, 0,
      kNonTemporal);
}

// One lane group (LPT lanes) per chunk of the entry stream; chunks are
// visited grid-stride so a capped (persistent) grid works too.  Every chunk
// holds the same number of entries, so the work is balanced whatever the row
// lengths.
//
// Inside a row the triples come in runs of equal B id.  The group reads the
// B row once, at the run's first triple, keeps it in registers for the run,
// and adds w * A[a] * B[b_id] for every triple with one double FMA per
// column (the product of two floats is exact in double).
//
// With BUF (A, B, the output and the workspace each under 4 GB, rows of at
// most kMaxStride bytes) all reads are buffer loads: A and B rows through
// structured buffers (record = row id), the residual variants' rows and the
// stores through raw 32-bit byte offsets.  Where no row is needed (A at
// markers and where the step's previous entry gathered the same row, B
// except at run starts) the record or offset is out of range, so the lane
// gets zeros and generates no memory traffic, and no load sits behind a
// branch.  A marker therefore finds A = 0 and a held B row of 0, so its FMA
// adds an exact zero; a repeated row takes the previous entry's values.
// Without BUF, plain loads read row 0 at markers and the values are masked
// instead.
//
// With LDSB (buffer loads only) the workgroup first copies its column
// slice of the whole B table into LDS, and a run start reads its B row from
// there when the FMAs need it.  No B row is then held in registers while a
// step's gathers are in flight, which leaves room for more waves per SIMD,
// and the B reads leave the L2 alone.  Used when the table fits (R for the
// forward and dX passes: at most kMaxLdsB bytes per slice with 768-thread
// workgroups, kMaxLdsBig with 1024; see launch_stream).
//
// The hard-KB variants with B in LDS (4 floats per lane; 8 lanes per group
// with the paired entry fetch, 8 or more for the residual hop) need 83 or 84
// VGPRs, more than six waves per SIMD allow; they are compiled for six waves
// (80 VGPRs, a few registers spilled around the chunk loop, outside the
// steps), which measured faster than losing the second workgroup per CU or
// keeping B in registers (residual forward on the large KB 0.89 -> 0.84 ms).
// The same cap on the soft-KB variants or on narrower lane groups spilled
// inside the loop and ran slower, so they keep the compiler's own
// allocation.
constexpr int kRaggedLane = -4;
template <int LPT, bool WEIGHTED, bool RES, bool LDSB>
constexpr int stream_min_waves() {
  return (LDSB && !WEIGHTED && (RES ? LPT >= 8 : LPT == 8)) ? 6 : 1;
}

//
// LANE: 4 floats per lane, or kRaggedLane: 4 where b >= 5 is not a multiple of 4
// (see LaneCols).
template <int LANE, int LPT, bool BUF, bool WEIGHTED, bool RES, bool LDSB>
__global__ __launch_bounds__((LDSB ? kBlockLdsBig : kBlock),
                             (stream_min_waves<LPT, WEIGHTED, RES, LDSB>())) void
stream_kernel(StreamArgs a) {
  constexpr bool RAGGED = LANE == kRaggedLane;
  static_assert(LANE == 4 || RAGGED, "narrower rows have a kernel of their own");
  constexpr int VEC = 4;
  static_assert(BUF || !LDSB, "the LDS copy of B goes with raw buffer loads");
  const int BLK = LDSB ? (int)blockDim.x : kBlock;  // kBlockLds or kBlockLdsBig
  const int GPB = BLK / LPT;
  constexpr int W = LPT * VEC;  // columns of one slice
  extern __shared__ float b_lds[];  // [B_rows][W] with LDSB
  const int lane = threadIdx.x % LPT;
  const int grp = threadIdx.x / LPT;
  const int c0 = blockIdx.y * (LPT * VEC) + lane * VEC;
  const bool active = c0 < a.b;
  const int c = lane_cols<RAGGED>(c0, a.b).c, skip = lane_cols<RAGGED>(c0, a.b).skip;
  const size_t bb = (size_t)a.b;
  // Lanes past b read column 0 and store nothing.
  const int cl = active ? c : 0;
  const uint32_t row_bytes = (uint32_t)a.b * (uint32_t)sizeof(float);

  // (Only used with BUF, where every table is known to be under 4 GB.)
  auto rsrc = [](const void *p, uint64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)(uint32_t)bytes,
                                             kRawBufferWord3);
  };
  // A and B are gathered by row: structured buffers of row_bytes records
  // (row_bytes is at most kMaxStride with BUF).  The residual variants keep
  // raw byte offsets, which measured faster there (their marker rows read
  // A too, so the record index needs a select either way, and the struct
  // addresses cost them registers).
  auto rows_rsrc = [&](const void *p, int64_t rows) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)row_bytes, (int)rows,
                                             kRawBufferWord3);
  };
  // A residual pass reads A at triples and Z at markers with one load per
  // entry: one raw buffer spans both arrays (under 4 GB, choose_stream).  The
  // offsets of A's rows in it start at a_off, which col_bytes already holds --
  // one register for every use, so the other raw buffers start as far ahead of
  // their arrays -- and those of Z's at a_off + z_delta (modulo 2^32).
  uint32_t a_off = 0, z_delta = 0;
  uint64_t span_bytes = (uint64_t)a.A_rows * row_bytes;
  if constexpr (RES && BUF) {
    const uint64_t ap = reinterpret_cast<uintptr_t>(a.A), zp = reinterpret_cast<uintptr_t>(a.Z);
    const uint64_t a_end = ap + (uint64_t)a.A_rows * row_bytes;
    const uint64_t z_end = zp + (uint64_t)a.out_rows * row_bytes;
    a_off = ap > zp ? (uint32_t)(ap - zp) : 0;
    z_delta = (uint32_t)(zp - ap);
    span_bytes = (a_end > z_end ? a_end : z_end) - (ap < zp ? ap : zp);
  }
  const uint32_t col_bytes = (uint32_t)cl * (uint32_t)sizeof(float) + a_off;
  auto ahead = [&](const void *p, uint64_t bytes) {
    return rsrc(static_cast<const char *>(p) - a_off, bytes + a_off);
  };
  const __amdgpu_buffer_rsrc_t arsrc =
      RES ? rsrc(reinterpret_cast<const char *>(a.A) - a_off, span_bytes)
          : rows_rsrc(a.A, a.A_rows);
  const __amdgpu_buffer_rsrc_t brsrc =
      RES ? ahead(a.B, (uint64_t)a.B_rows * row_bytes) : rows_rsrc(a.B, a.B_rows);
  const __amdgpu_buffer_rsrc_t orsrc = ahead(a.out, (uint64_t)a.out_rows * row_bytes);
  const __amdgpu_buffer_rsrc_t srsrc =
      rsrc(a.slots, (uint64_t)a.n_slots * a.b * sizeof(double));

  // This workgroup's chunk list: the blocks with blockIdx.x % n_lists == x
  // (all on XCD x) share list x, grid-stride.
  const int nl = a.n_lists;
  const int xl = (int)(blockIdx.x % (unsigned)nl);
  int64_t c_begin = 0, c_end = 0;
#pragma unroll
  for (int i = 0; i < kMaxChunkLists; ++i)
    if (i == xl) {
      c_begin = a.list_chunk[i];
      c_end = a.list_chunk[i + 1];
    }
  const int64_t wg_in_list = blockIdx.x / nl;
  const int64_t wgs_in_list = ((int64_t)gridDim.x - xl + nl - 1) / nl;
  const int64_t stride = wgs_in_list * GPB;

  if constexpr (LDSB) {
    // Columns [col0, col0 + W) of every B row; columns past b read as zeros.
    const int col0 = blockIdx.y * W;
    const int64_t n_lds = a.B_rows * W;
    for (int64_t i = (int64_t)threadIdx.x * VEC; i < n_lds; i += (int64_t)BLK * VEC) {
      const int64_t r = i / W;
      const int j = (int)(i % W);
      float v[VEC];
      if (col0 + j < a.b) {
        const int cj = lane_cols<RAGGED>(col0 + j, a.b).c;
        load_row<VEC>(a.B + (size_t)KBF_CHECKED(r, a.B_rows) * bb + cj, v);
      } else {
#pragma unroll
        for (int q = 0; q < VEC; ++q) v[q] = 0.0f;
      }
      lds_store(b_lds + i, v);
    }
    __syncthreads();
  }

  // Each lane loads K of a step's kUnroll entries (lane + k * LPT) and the
  // group shares them by broadcast, so one load instruction fetches the
  // entries of every lane group in the wavefront.  (The prefetch after a
  // chunk's last step reads the next chunk's first entries, or the stream's
  // last entry at its end, and is not used.)
  constexpr int K = (kUnroll + LPT - 1) / LPT;
  auto fetch = [&](int64_t p, int2 (&mine)[K], float (&wmine)[K]) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int64_t q = min(p + min(lane + k * LPT, kUnroll - 1), a.n - 1);
      mine[k] = a.entries[q];
      if constexpr (WEIGHTED) wmine[k] = a.weights[q];
    }
  };
  // Two steps' entries, 2 per lane (entries p + 2l and p + 2l + 1 of lane
  // l < kUnroll; lanes past it repeat the last pair).  p and the stream
  // length are multiples of kUnroll, so every pair is 16-byte aligned and
  // the clamp keeps it inside the stream.
  // Only for groups of exactly eight lanes: not in the residual variants,
  // whose register-capped LDS form spilled more with it and ran 0.7 % slower,
  // nor with wider groups, whose LDS form would need the same cap and whose
  // short chunks (small KBs) would then spill every other step.
  constexpr bool kPairFetch = !WEIGHTED && !RES && K == 1 && LPT == kUnroll;
  auto fetch2 = [&](int64_t p, int4 &mine) {
    const int64_t q = min(p + 2 * min(lane, kUnroll - 1), a.n - 2);
    mine = reinterpret_cast<const int4 *>(a.entries)[q / 2];
  };

  for (int64_t g = c_begin + wg_in_list * GPB + grp; g < c_end; g += stride) {
    const int64_t p0 = KBF_CHECKED(g, a.n / a.chunk) * a.chunk;
    const int64_t p1 = p0 + a.chunk;
    double acc[VEC];
    float held_b[VEC];  // the current run's B row
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      acc[v] = 0.0;
      held_b[v] = 0.0f;
    }

    // Software pipeline: the entries of the next step are loaded while this
    // step's gathers are in flight.  With lane groups of eight lanes or more
    // (and no weights) one 16-byte load per lane fetches two steps' entries
    // (lane l entries 2l and 2l + 1 of the pair), so the steps run in pairs
    // and only the second of a pair issues a fetch: one entry load per two
    // steps in front of their sixteen row gathers.
    int2 mine_next[K];
    float wmine_next[K];
    int4 mine2 = make_int4(0, 0, 0, 0);
    if constexpr (kPairFetch)
      fetch2(p0, mine2);
    else
      fetch(p0, mine_next, wmine_next);
    // One step of kUnroll entries from p; H is its half of a pair (0 or 1)
    // or -1 for the one-step fetch.
    auto step = [&](const int64_t p, auto hc) {
      constexpr int H = decltype(hc)::value;
      int2 e[kUnroll];
      float w[kUnroll];
      float xa[kUnroll][VEC], xb[kUnroll][VEC];
      static_for<kUnroll>([&](auto uc) {
        constexpr int u = decltype(uc)::value;
        if constexpr (H >= 0) {
          constexpr int src = (kUnroll / 2) * H + u / 2;
          const int ex = (u % 2) ? mine2.z : mine2.x;
          const int ey = (u % 2) ? mine2.w : mine2.y;
          e[u] = make_int2(group_bcast<LPT, src>(ex), group_bcast<LPT, src>(ey));
        } else {
          const int2 m = mine_next[u / LPT];
          e[u] = make_int2(group_bcast<LPT, u % LPT>(m.x), group_bcast<LPT, u % LPT>(m.y));
          if constexpr (WEIGHTED)
            w[u] = __int_as_float(group_bcast<LPT, u % LPT>(__float_as_int(wmine_next[u / LPT])));
        }
      });
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const bool triple = e[u].x >= 0;
        const bool run_start = triple && (e[u].x & kRunStart);
        // The entry before it in this step gathered the same A row: no read
        // (the FMAs below take that row again).  Never at a step's first
        // entry; the residual variants read the row again (the reuse cost
        // their register-capped LDS form more spills than it saved).
        const bool same_a = !RES && u > 0 && triple && (e[u].y & kSameA);
        const int32_t bid = e[u].y & kIdMask;  // a triple's B row
        // A marker that writes row j of a residual pass reads A[j] for gamma * A[j].
        const bool res_row = RES && !triple && e[u].y >= 0;
        const uint32_t ia = triple ? (uint32_t)(e[u].x & kIdMask) : (uint32_t)e[u].y;
        if constexpr (BUF && !RES) {
          // A triple's record is its id; a marker's x (-1) with the run-start
          // bit cleared is past every table, so it reads zeros.
#if defined(KBFOLLOW_CHECKED)
          const uint32_t ra =
              (triple && !same_a) ? (uint32_t)KBF_CHECKED(ia, a.A_rows) : kNoRecord;
#else
          const uint32_t ra = same_a ? kNoRecord : ((uint32_t)e[u].x & ~(uint32_t)kRunStart);
#endif
          gather_row(arsrc, ra, col_bytes, xa[u]);
          if constexpr (!LDSB)
            gather_row(brsrc, run_start ? (uint32_t)KBF_CHECKED(bid, a.B_rows) : kNoRecord,
                            col_bytes, xb[u]);
        } else if constexpr (BUF) {
          load_row_buffer(
              arsrc,
              (triple || res_row)
                  ? (uint32_t)KBF_CHECKED(ia, triple ? a.A_rows : a.out_rows) * row_bytes +
                        col_bytes + (triple ? 0u : z_delta)
                  : kOutOfRange,
              xa[u]);
          if constexpr (!LDSB)
            load_row_buffer(brsrc,
                                 run_start ? (uint32_t)KBF_CHECKED(bid, a.B_rows) * row_bytes +
                                                 col_bytes
                                           : kOutOfRange,
                                 xb[u]);
        } else {
          // A residual row comes from Z (A itself for the residual hop).
          const float *src = res_row ? a.Z : a.A;
          load_row<VEC>(src + (size_t)(triple ? KBF_CHECKED(ia, a.A_rows)
                                              : res_row ? KBF_CHECKED(ia, a.out_rows) : 0) *
                                  bb +
                              cl,
                        xa[u]);
          load_row<VEC>(a.B + (size_t)(run_start ? KBF_CHECKED(bid, a.B_rows) : 0) * bb + cl,
                        xb[u]);
        }
      }
      if constexpr (H < 0)
        fetch(p + kUnroll, mine_next, wmine_next);
      else if constexpr (H == 1)
        fetch2(p + kUnroll, mine2);
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const bool triple = e[u].x >= 0;
        const bool run_start = triple && (e[u].x & kRunStart);
        // A repeated A row was not read again: take the previous entry's
        // (plain loads read it again, the same values).
        if constexpr (BUF && !RES) {
          if (u > 0) {
            const bool same_a = triple && (e[u].y & kSameA);
#pragma unroll
            for (int v = 0; v < VEC; ++v) xa[u][v] = same_a ? xa[u - 1][v] : xa[u][v];
          }
        }
        // Run starts take the new B row; markers take the zeros their
        // out-of-range B load returned (masked explicitly without BUF).
        if constexpr (LDSB) {
          if (run_start) {
            lds_row(b_lds + (size_t)KBF_CHECKED(e[u].y & kIdMask, a.B_rows) * W + lane * VEC,
                         held_b);
          } else if (!triple) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) held_b[v] = 0.0f;
          }
        }
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
          if constexpr (!LDSB) {
            const float nb = (BUF || triple) ? xb[u][v] : 0.0f;
            held_b[v] = (run_start || !triple) ? nb : held_b[v];
          }
          double t = (double)xa[u][v];
          if constexpr (WEIGHTED) t *= (double)w[u];
          // Zero at markers (also the residual row's A and plain loads' row 0).
          if constexpr (RES || !BUF) t = triple ? t : 0.0;
          acc[v] = __builtin_fma(t, (double)held_b[v], acc[v]);
        }
        const int f = e[u].y;
        if (!triple) {
        if (active && f != INT_MIN) {
          double y[VEC];
#pragma unroll
          for (int v = 0; v < VEC; ++v)
            y[v] = (RES && f >= 0) ? acc[v] + (double)a.gamma * (double)xa[u][v] : acc[v];
          if constexpr (RAGGED && RES) {
            if (f >= 0)
              store_row_from<VEC>(a.out + (size_t)KBF_CHECKED(f, a.out_rows) * bb + c, y, skip);
            else
              store_slot_from<VEC>(a.slots + (size_t)KBF_CHECKED(-(f + 1), a.n_slots) * bb + c, y,
                                   skip);
          } else if (f >= 0) {
            if constexpr (BUF)
              store_row_buffer(
                  orsrc, (uint32_t)KBF_CHECKED(f, a.out_rows) * row_bytes + col_bytes, y);
            else
              store_row<VEC>(a.out + (size_t)KBF_CHECKED(f, a.out_rows) * bb + c, y);
          } else {
            if constexpr (BUF)
              store_slot_buffer(
                  srsrc,
                  ((uint32_t)KBF_CHECKED(-(f + 1), a.n_slots) * (uint32_t)a.b + (uint32_t)c) *
                      (uint32_t)sizeof(double),
                  y);
            else
              store_slot<VEC>(a.slots + (size_t)KBF_CHECKED(-(f + 1), a.n_slots) * bb + c, y);
          }
        }
        // The marker ends the row: restart the sum (only the lanes of
        // groups at a marker execute this).
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] = 0.0;
        }
      }
    };
    if constexpr (kPairFetch) {
      // Chunks are whole steps; an odd last step runs alone.
      for (int64_t p = p0; p < p1; p += 2 * kUnroll) {
        step(p, std::integral_constant<int, 0>{});
        if (p + kUnroll >= p1) break;
        step(p + kUnroll, std::integral_constant<int, 1>{});
      }
    } else {
      for (int64_t p = p0; p < p1; p += kUnroll) step(p, std::integral_constant<int, -1>{});
    }
  }
}

// -- narrow rows -------------------------------------------------------------
//
// Rows of at most kMaxNarrow floats: a lane holds a whole row, so a lane per
// chunk (the stream kernel's layout at these widths) leaves few waves to hide
// the gathers' latency, and its entry loads, 8 bytes from 64 chunks at once,
// touch 64 lines each.  Here 8 lanes share a chunk and every lane takes one of
// a step's 8 entries: one coalesced entry load, one A gather and one B read per
// 64 entries of a wave (B from LDS where its table fits), kNarrowSteps steps in
// flight.  The step's products are summed by a segmented scan over the 8 lanes,
// cut at its markers; a marker's lane then holds the sum of the entries before
// it back to the previous marker and writes it, and what follows the last
// marker goes on into the next step through lane 0.  The order of the
// additions is fixed, so results are bitwise reproducible.
//
// Forward stream kernel, before (a lane per chunk) and after: 20 M triples, b =
// 1: 260 -> 107 us; 43.7 M triples over 12.9 M entities, b = 1 / 2 / 3 / 4: 557 /
// 490 / 604 / 603 -> 357 / 406 / 458 / 440 us.  Bound by the gathers: a line per
// entry, about 1.2e11 a second.
constexpr int kNarrowSteps = 4;      // in flight; twice as many for one or two floats
constexpr int kNarrowWgs = 64;       // workgroups per CU at most, where each copies B
constexpr size_t kNarrowLds = 20 * 1024;  // eight workgroups' B tables fit a CU

template <int N>
__device__ __forceinline__ void load_floats(const float *p, float (&v)[N]) {
  __builtin_memcpy(v, p, N * sizeof(float));
}

// The double of the lane D below (in its row of 16), or of the mirrored lane of
// its group of 8.
template <int CTRL>
__device__ __forceinline__ double dpp_double(double v) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xf, 0xf, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
constexpr int kDppRowShr = 0x110, kDppHalfMirror = 0x141;

template <int N, bool WEIGHTED, bool RES, bool LDSB>
__global__ __launch_bounds__(kBlock) void narrow_kernel(StreamArgs a) {
  constexpr int U = N <= 2 ? 2 * kNarrowSteps : kNarrowSteps;
  extern __shared__ float narrow_b[];  // [B_rows][N] with LDSB
  const int l = threadIdx.x % kNarrowLanes;
  constexpr int GPB = kBlock / kNarrowLanes;

  const int nl = a.n_lists;
  const int xl = (int)(blockIdx.x % (unsigned)nl);
  int64_t c_begin = 0, c_end = 0;
#pragma unroll
  for (int i = 0; i < kMaxChunkLists; ++i)
    if (i == xl) {
      c_begin = a.list_chunk[i];
      c_end = a.list_chunk[i + 1];
    }
  const int64_t wgs_in_list = ((int64_t)gridDim.x - xl + nl - 1) / nl;
  const int64_t stride = wgs_in_list * GPB;

  if constexpr (LDSB) {
    for (int i = threadIdx.x; i < (int)a.B_rows * N; i += kBlock) narrow_b[i] = a.B[i];
    __syncthreads();
  }

  const int steps = a.chunk / kNarrowLanes;
  for (int64_t g = c_begin + (blockIdx.x / nl) * GPB + threadIdx.x / kNarrowLanes; g < c_end;
       g += stride) {
    const int64_t p0 = KBF_CHECKED(g, a.n / a.chunk) * a.chunk + l;
    auto entry = [&](int s, int2 &e, float &w) {
      if (s < steps) {
        e = a.entries[p0 + s * kNarrowLanes];
        if constexpr (WEIGHTED) w = a.weights[p0 + s * kNarrowLanes];
      } else {  // past the chunk: markers of no target
        e = make_int2(-1, INT_MIN);
        w = 0.0f;
      }
    };
    int2 next[U];
    float wnext[U];
#pragma unroll
    for (int u = 0; u < U; ++u) entry(u, next[u], wnext[u]);
    double prev[N];       // the previous step's scan
    bool carry = false;   // its last lane's row goes on
#pragma unroll
    for (int v = 0; v < N; ++v) prev[v] = 0.0;

    for (int s0 = 0; s0 < steps; s0 += U) {
      int2 e[U];
      float w[U];
      float xa[U][N], xb[U][N];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        e[u] = next[u];
        w[u] = wnext[u];
        const bool triple = e[u].x >= 0;
        const int32_t ia = triple ? (e[u].x & kIdMask) : 0;
        const float *row = a.A + (size_t)KBF_CHECKED(ia, a.A_rows) * N;
        if constexpr (RES)
          if (!triple && e[u].y >= 0) row = a.Z + (size_t)KBF_CHECKED(e[u].y, a.out_rows) * N;
        load_floats<N>(row, xa[u]);
        const int32_t ib = triple ? (e[u].y & kIdMask) : 0;
        if constexpr (!LDSB)
          load_floats<N>(a.B + (size_t)KBF_CHECKED(ib, a.B_rows) * N, xb[u]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) entry(s0 + U + u, next[u], wnext[u]);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool triple = e[u].x >= 0;
        if constexpr (LDSB) {
          const int32_t ib = triple ? (e[u].y & kIdMask) : 0;
          load_floats<N>(narrow_b + (size_t)KBF_CHECKED(ib, a.B_rows) * N, xb[u]);
        }
        // Where the lane's segment begins: after the last marker before it.
        const unsigned marks =
            (unsigned)(__ballot(!triple) >> (threadIdx.x % 64 / kNarrowLanes * kNarrowLanes)) &
            ((1u << kNarrowLanes) - 1);
        const unsigned below = marks & ((1u << l) - 1);
        const int start = below ? 32 - __builtin_clz(below) : 0;
        double sum[N];
#pragma unroll
        for (int v = 0; v < N; ++v) {
          double t = (double)xa[u][v];
          if constexpr (WEIGHTED) t *= (double)w[u];
          sum[v] = triple ? t * (double)xb[u][v] : 0.0;
          const double c = dpp_double<kDppHalfMirror>(prev[v]);
          sum[v] += (l == 0 && carry) ? c : 0.0;
        }
        const bool in1 = l - 1 >= start, in2 = l - 2 >= start, in4 = l - 4 >= start;
#pragma unroll
        for (int v = 0; v < N; ++v) {
          const double t1 = dpp_double<kDppRowShr + 1>(sum[v]);
          sum[v] += in1 ? t1 : 0.0;
          const double t2 = dpp_double<kDppRowShr + 2>(sum[v]);
          sum[v] += in2 ? t2 : 0.0;
          const double t4 = dpp_double<kDppRowShr + 4>(sum[v]);
          sum[v] += in4 ? t4 : 0.0;
          prev[v] = sum[v];
        }
        carry = !(marks >> (kNarrowLanes - 1) & 1);
        const int f = e[u].y;
        if (!triple && f != INT_MIN) {
          if (f >= 0) {
            float y[N];
#pragma unroll
            for (int v = 0; v < N; ++v)
              y[v] = (float)(RES ? sum[v] + (double)a.gamma * (double)xa[u][v] : sum[v]);
            float *out = a.out + (size_t)KBF_CHECKED(f, a.out_rows) * N;
            __builtin_memcpy(out, y, N * sizeof(float));
          } else {
            double *slot = a.slots + (size_t)KBF_CHECKED(-(f + 1), a.n_slots) * N;
#pragma unroll
            for (int v = 0; v < N; ++v) slot[v] = sum[v];
          }
        }
      }
    }
  }
}

// Adds slots [first, first + n) in increasing order; writes the float row or
// a next-level slot.  `block` of `n_blocks` blocks share the tasks.
template <int VEC, int LPT, bool RAGGED>
__device__ __forceinline__ void combine_tasks(const int4 *__restrict__ tasks, int64_t n_tasks,
                                              double *__restrict__ slots, int64_t n_slots,
                                              int32_t b, float *out, int64_t out_rows,
                                              const float *res, float gamma, int64_t block,
                                              int64_t n_blocks) {
  constexpr int W = LPT * VEC;
  constexpr int GPB = kBlock / LPT;
  const int lane = threadIdx.x % LPT;
  const int grp = threadIdx.x / LPT;
  const int c0 = blockIdx.y * W + lane * VEC;
  if (c0 >= b) return;  // no barrier below
  const int c = lane_cols<RAGGED>(c0, b).c, skip = lane_cols<RAGGED>(c0, b).skip;
  const size_t bb = (size_t)b;
  const int64_t stride = n_blocks * GPB;
  for (int64_t t = block * GPB + grp; t < n_tasks; t += stride) {
    const int4 tk = tasks[t];  // first, n, dst
    double acc[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = 0.0;
    for (int i = 0; i < tk.y; i += kUnroll) {
      const int n = min(kUnroll, tk.y - i);
      double part[kUnroll][VEC];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u)
        load_slot<VEC>(slots + (size_t)KBF_CHECKED(tk.x + i + min(u, n - 1), n_slots) * bb + c,
                       part[u]);
#pragma unroll
      for (int u = 0; u < kUnroll; ++u)
        if (u < n) {
#pragma unroll
          for (int v = 0; v < VEC; ++v) acc[v] += part[u][v];
        }
    }
    if (tk.z >= 0) {
      const size_t row = (size_t)KBF_CHECKED(tk.z, out_rows);
      if (res) {
        float r[VEC];
        load_row<VEC>(res + row * bb + c, r);
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] += (double)gamma * (double)r[v];
      }
      store_row_from<VEC>(out + row * bb + c, acc, skip);
    } else {
      store_slot_from<VEC>(slots + (size_t)KBF_CHECKED(-(int64_t)tk.z - 1, n_slots) * bb + c, acc,
                           skip);
    }
  }
}

// A wide combine task: one workgroup adds slots [first, first + n) of up to 32
// columns of the launch's slice blockIdx.y (so at most four workgroups per task
// and slice: the grid's width is a matter of the tasks alone; all tasks' first
// parts come first, so that each part is spread over the XCDs).  Its lane groups (of at most 8 lanes, so 32 of them or more) take
// every GPB-th slot each, eight loads in flight, and the first one adds the
// groups' sums in order: a thousand slots in about four rounds of loads, where
// tasks of 32 slots took two launches more for a hub row.
constexpr int kWideLpt = 8;
template <int VEC, int LPT, bool RAGGED>
__device__ __forceinline__ void combine_wide(const TailArgs &a, int64_t block) {
  constexpr int WL = LPT < kWideLpt ? LPT : kWideLpt;
  constexpr int W = WL * VEC;
  constexpr int GPB = kBlock / WL;
  __shared__ double part[GPB][W];
  const int lane = threadIdx.x % WL, grp = threadIdx.x / WL;
  const uint32_t blk = (uint32_t)block, n_wide = (uint32_t)a.n_wide;
  const int part0 = blockIdx.y * (LPT * VEC) + (int)(blk / n_wide) * W;
  if (part0 >= a.b) return;  // the whole workgroup: the last slice's columns end before
  const int c0 = part0 + lane * VEC;
  const bool active = c0 < a.b;
  const int c = active ? lane_cols<RAGGED>(c0, a.b).c : 0;
  const int skip = active ? lane_cols<RAGGED>(c0, a.b).skip : 0;
  const size_t bb = (size_t)a.b;
  const int4 tk = a.tasks[blk % n_wide];  // first, n, dst
  double acc[VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) acc[v] = 0.0;
  for (int i = grp; i < tk.y; i += GPB * kUnroll) {
    double p[kUnroll][VEC];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
      load_slot<VEC>(a.slots + (size_t)KBF_CHECKED(tk.x + min(i + u * GPB, tk.y - 1), a.n_slots) * bb + c,
                     p[u]);
#pragma unroll
    for (int u = 0; u < kUnroll; ++u)
      if (i + u * GPB < tk.y) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] += p[u][v];
      }
  }
#pragma unroll
  for (int v = 0; v < VEC; ++v) part[grp][lane * VEC + v] = acc[v];
  __syncthreads();
  if (grp != 0 || !active) return;
#pragma unroll
  for (int v = 0; v < VEC; ++v) acc[v] = 0.0;
  for (int k = 0; k < GPB; ++k)
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] += part[k][lane * VEC + v];
  if (tk.z >= 0) {
    const size_t row = (size_t)KBF_CHECKED(tk.z, a.out_rows);
    if (a.res) {
      float r[VEC];
      load_row<VEC>(a.res + row * bb + c, r);
#pragma unroll
      for (int v = 0; v < VEC; ++v) acc[v] += (double)a.gamma * (double)r[v];
    }
    store_row_from<VEC>(a.out + row * bb + c, acc, skip);
  } else {
    store_slot_from<VEC>(a.slots + (size_t)KBF_CHECKED(-(int64_t)tk.z - 1, a.n_slots) * bb + c, acc,
                         skip);
  }
}

// Writes the rows no triple reaches, given as pieces of consecutive rows
// (first, count); lanes over the columns as in the stream kernel.  PACKED: a
// lane group writes LPT consecutive pieces, whose descriptors its lanes fetch
// with one load (lane j the j-th) and share by shuffles, so that one load
// stands in front of the stores of 64 pieces per wave.  Otherwise one piece
// per group: the residual hop's rows each need a load of X of their own.
// `block` of `n_blocks` blocks share the pieces.
template <int VEC, int LPT, bool PACKED, bool RAGGED>
__device__ __forceinline__ void zero_pieces(const int2 *__restrict__ pieces, int64_t n_pieces,
                                            int32_t b, float *out, int64_t out_rows,
                                            const float *res, float gamma, int64_t block,
                                            int64_t n_blocks) {
  constexpr int W = LPT * VEC;
  constexpr int GPB = kBlock / LPT;
  const int lane = threadIdx.x % LPT;
  const int grp = threadIdx.x / LPT;
  const int c0 = blockIdx.y * W + lane * VEC;
  const bool active = c0 < b;
  const int c = lane_cols<RAGGED>(c0, b).c, skip = lane_cols<RAGGED>(c0, b).skip;
  const size_t bb = (size_t)b;
  if constexpr (PACKED) {
    const int64_t stride = n_blocks * kBlock;
    for (int64_t t0 = (block * GPB + grp) * LPT; t0 < n_pieces; t0 += stride) {
      const int64_t t = t0 + lane;
      int2 mine = make_int2(0, 0);  // past the end: a piece of no rows
      if (t < n_pieces) mine = pieces[t];
      const int base = (int)(threadIdx.x % 64) - lane;  // lane 0 of this group in the wave
      for (int j = 0; j < LPT; ++j) {
        const int first = __shfl(mine.x, base + j);
        const int count = __shfl(mine.y, base + j);
        if (!active) continue;  // after the shuffles, which every lane joins
        for (int i = 0; i < count; ++i) {
          const double z[VEC] = {};
          // Non-temporal, like every output row: plain stores would leave
          // the rows dirty in the caches, to be written back during the next
          // pass.
          store_row_from<VEC>(out + (size_t)KBF_CHECKED((int64_t)first + i, out_rows) * bb + c, z,
                              skip);
        }
      }
    }
  } else {
    // gamma * res[row] into out[row].  A lane group takes kFillPieces
    // consecutive pieces (every lane loads the same descriptors) and walks
    // their rows as one flat sequence, kFillBatch rows at a time: all of a
    // batch's row loads are issued before its stores, so the mostly one- or
    // two-row pieces of a Zipf KB still keep many loads in flight.  (res may
    // be out itself: each row is read and then written by the same lane.)
    if (!active) return;  // no barrier or shuffle below
    const int64_t stride = n_blocks * GPB * kFillPieces;
    for (int64_t t0 = (block * GPB + grp) * kFillPieces; t0 < n_pieces; t0 += stride) {
      int first[kFillPieces], start[kFillPieces], end[kFillPieces];
      int total = 0;
#pragma unroll
      for (int j = 0; j < kFillPieces; ++j) {
        const int2 pc = (t0 + j < n_pieces) ? pieces[t0 + j] : make_int2(0, 0);
        first[j] = pc.x;
        start[j] = total;
        total += pc.y;
        end[j] = total;
      }
      for (int k0 = 0; k0 < total; k0 += kFillBatch) {
        int row[kFillBatch];
        float r[kFillBatch][VEC];
#pragma unroll
        for (int u = 0; u < kFillBatch; ++u) {
          const int k = k0 + u;
          row[u] = -1;
#pragma unroll
          for (int j = 0; j < kFillPieces; ++j)
            row[u] = (k >= start[j] && k < end[j]) ? first[j] + (k - start[j]) : row[u];
#pragma unroll
          for (int v = 0; v < VEC; ++v) r[u][v] = 0.0f;
          if (row[u] >= 0)
            load_row<VEC>(res + (size_t)KBF_CHECKED((int64_t)row[u], out_rows) * bb + c, r[u]);
        }
#pragma unroll
        for (int u = 0; u < kFillBatch; ++u) {
          if (row[u] < 0) continue;
          double y[VEC];
#pragma unroll
          for (int v = 0; v < VEC; ++v) y[v] = 0.0 + (double)gamma * (double)r[u][v];
          store_row_from<VEC>(out + (size_t)KBF_CHECKED((int64_t)row[u], out_rows) * bb + c, y,
                              skip);
        }
      }
    }
  }
}

// +0.0, or gamma * res[i], to n floats from p on: 16 bytes per thread.  (A
// grid of as many workgroups as the chip holds, walking the range, wrote
// 1.66 GB of zeros at 4.6 TB/s; one store per thread writes them at 6.6.
// Plain stores reach 6.9, but the lines they leave in the caches made the
// stream kernel behind them 6 % slower.)
template <bool RES>
__global__ __launch_bounds__(kBlock) void fill_kernel(float *__restrict__ p, int64_t n,
                                                      const float *__restrict__ res, float gamma) {
  const int64_t i = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * 4;
  auto value = [&](float r) { return RES ? 0.0 + (double)gamma * (double)r : 0.0; };
  if (i + 4 <= n) {
    float r[4] = {};
    if constexpr (RES) load_row<4>(res + i, r);
    const double y[4] = {value(r[0]), value(r[1]), value(r[2]), value(r[3])};
    store_row<4>(p + i, y);
  } else {
    for (int64_t k = i; k < n; ++k) p[k] = (float)value(RES ? res[k] : 0.0f);
  }
}

// The blocks of a combine launch: blocks [0, wide_blocks) take the wide tasks, the
// next combine_blocks the others; true for the blocks after them.
template <int VEC, int LPT, bool RAGGED>
__device__ __forceinline__ bool combine_launch(const TailArgs &a) {
  if ((int64_t)blockIdx.x < a.wide_blocks) {
    combine_wide<VEC, LPT, RAGGED>(a, blockIdx.x);
    return false;
  }
  const int64_t block = (int64_t)blockIdx.x - a.wide_blocks;
  if (block >= a.combine_blocks) return true;
  combine_tasks<VEC, LPT, RAGGED>(a.tasks + a.n_wide, a.n_tasks - a.n_wide, a.slots, a.n_slots, a.b,
                                  a.out, a.out_rows, a.res, a.gamma, block, a.combine_blocks);
  return false;
}

// A later combine level.
template <int VEC, int LPT>
__global__ __launch_bounds__(kBlock) void combine_kernel(TailArgs a) {
  if (VEC == 4 && a.b % 4 != 0)
    combine_launch<VEC, LPT, VEC == 4>(a);
  else
    combine_launch<VEC, LPT, false>(a);
}

template <int VEC, int LPT, bool PACKED, bool RAGGED>
__device__ __forceinline__ void tail_blocks(const TailArgs &a) {
  if (combine_launch<VEC, LPT, RAGGED>(a)) {
    const int64_t before = a.wide_blocks + a.combine_blocks;
    zero_pieces<VEC, LPT, PACKED, RAGGED>(a.pieces, a.n_pieces, a.b, a.out, a.out_rows, a.res,
                                          a.gamma, (int64_t)blockIdx.x - before,
                                          (int64_t)gridDim.x - before);
  }
}

// The first combine level and the empty rows in one launch: the first blocks
// take the combine tasks, the others the empty-row pieces.  The two write disjoint rows; the combine's dependent slot reads
// overlap with the fill's stores instead of forming a launch of their own.
template <int VEC, int LPT, bool PACKED>
__global__ __launch_bounds__(kBlock) void tail_kernel(TailArgs a) {
  if (VEC == 4 && a.b % 4 != 0)
    tail_blocks<VEC, LPT, PACKED, VEC == 4>(a);
  else
    tail_blocks<VEC, LPT, PACKED, false>(a);
}

template <int LANE, bool BUF, bool WT, bool RES, bool LDSB>
const void *stream_fn(int lpt) {
  switch (lpt) {
    case 1:
      // (KBFOLLOW_MAX_LPT=1, which does not narrow the LDS variant's groups.)
      if constexpr (LDSB)
        return nullptr;
      else
        return reinterpret_cast<const void *>(&stream_kernel<LANE, 1, BUF, WT, RES, LDSB>);
    case 2: return reinterpret_cast<const void *>(&stream_kernel<LANE, 2, BUF, WT, RES, LDSB>);
    case 4: return reinterpret_cast<const void *>(&stream_kernel<LANE, 4, BUF, WT, RES, LDSB>);
    case 8: return reinterpret_cast<const void *>(&stream_kernel<LANE, 8, BUF, WT, RES, LDSB>);
    case 16: return reinterpret_cast<const void *>(&stream_kernel<LANE, 16, BUF, WT, RES, LDSB>);
    case 32: return reinterpret_cast<const void *>(&stream_kernel<LANE, 32, BUF, WT, RES, LDSB>);
  }
  return nullptr;
}

template <int LANE, bool BUF, bool LDSB>
const void *stream_fn_sel(int lpt, bool wt, bool res) {
  if (wt)
    return res ? stream_fn<LANE, BUF, true, true, LDSB>(lpt)
               : stream_fn<LANE, BUF, true, false, LDSB>(lpt);
  return res ? stream_fn<LANE, BUF, false, true, LDSB>(lpt)
             : stream_fn<LANE, BUF, false, false, LDSB>(lpt);
}

// Plain loads never take the LDS copy of B.
const void *stream_fn_for(const ColumnTiling &t, bool buf, bool lds, bool wt, bool res) {
  if (t.ragged) {
    if (!buf) return stream_fn_sel<kRaggedLane, false, false>(t.lpt, wt, res);
    return lds ? stream_fn_sel<kRaggedLane, true, true>(t.lpt, wt, res)
               : stream_fn_sel<kRaggedLane, true, false>(t.lpt, wt, res);
  }
  if (!buf) return stream_fn_sel<4, false, false>(t.lpt, wt, res);
  return lds ? stream_fn_sel<4, true, true>(t.lpt, wt, res)
             : stream_fn_sel<4, true, false>(t.lpt, wt, res);
}

template <int N, bool LDSB>
const void *narrow_fn(bool wt, bool res) {
  if (wt)
    return res ? reinterpret_cast<const void *>(&narrow_kernel<N, true, true, LDSB>)
               : reinterpret_cast<const void *>(&narrow_kernel<N, true, false, LDSB>);
  return res ? reinterpret_cast<const void *>(&narrow_kernel<N, false, true, LDSB>)
             : reinterpret_cast<const void *>(&narrow_kernel<N, false, false, LDSB>);
}

const void *narrow_fn_for(int32_t b, bool lds, bool wt, bool res) {
  switch (b) {
    case 1: return lds ? narrow_fn<1, true>(wt, res) : narrow_fn<1, false>(wt, res);
    case 2: return lds ? narrow_fn<2, true>(wt, res) : narrow_fn<2, false>(wt, res);
    case 3: return lds ? narrow_fn<3, true>(wt, res) : narrow_fn<3, false>(wt, res);
    case 4: return lds ? narrow_fn<4, true>(wt, res) : narrow_fn<4, false>(wt, res);
  }
  return nullptr;
}

// Workgroups of `fn` (`block` threads, lds_bytes of dynamic LDS) that fit
// one CU at once, from the runtime's occupancy calculator; cached per kernel,
// block and LDS size.  0 when the query fails.
int blocks_per_cu(const void *fn, int block, size_t lds_bytes) {
  static std::mutex mu;
  static std::map<std::tuple<const void *, int, size_t>, int> cache;
  std::lock_guard<std::mutex> lock(mu);
  const auto key = std::make_tuple(fn, block, lds_bytes);
  auto it = cache.find(key);
  if (it != cache.end()) return it->second;
  int n = 0;
  if ((lds_bytes > 0 && hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                            (int)kMaxLdsBig) != hipSuccess) ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, block, lds_bytes) != hipSuccess) {
    (void)hipGetLastError();
    n = 0;
  }
  cache[key] = n;
  return n;
}

template <int VEC>
const void *combine_fn(int lpt) {
  switch (lpt) {
    case 1: return reinterpret_cast<const void *>(&combine_kernel<VEC, 1>);
    case 2: return reinterpret_cast<const void *>(&combine_kernel<VEC, 2>);
    case 4: return reinterpret_cast<const void *>(&combine_kernel<VEC, 4>);
    case 8: return reinterpret_cast<const void *>(&combine_kernel<VEC, 8>);
    case 16: return reinterpret_cast<const void *>(&combine_kernel<VEC, 16>);
    case 32: return reinterpret_cast<const void *>(&combine_kernel<VEC, 32>);
  }
  return nullptr;
}

template <int VEC, bool PACKED>
const void *tail_fn(int lpt) {
  switch (lpt) {
    case 1: return reinterpret_cast<const void *>(&tail_kernel<VEC, 1, PACKED>);
    case 2: return reinterpret_cast<const void *>(&tail_kernel<VEC, 2, PACKED>);
    case 4: return reinterpret_cast<const void *>(&tail_kernel<VEC, 4, PACKED>);
    case 8: return reinterpret_cast<const void *>(&tail_kernel<VEC, 8, PACKED>);
    case 16: return reinterpret_cast<const void *>(&tail_kernel<VEC, 16, PACKED>);
    case 32: return reinterpret_cast<const void *>(&tail_kernel<VEC, 32, PACKED>);
  }
  return nullptr;
}

int64_t blocks_for(int64_t items, int per_block, int max_blocks) {
  int64_t g = (items + per_block - 1) / per_block;
  if (max_blocks > 0 && g > max_blocks) g = max_blocks;
  if (g > (int64_t)INT32_MAX) g = INT32_MAX;
  return g < 1 ? 1 : g;
}

}  // namespace

ColumnTiling column_tiling(int32_t b) { return column_tiling_max(b, kMaxLpt); }

ColumnTiling column_tiling_max(int32_t b, int max_lpt) {
  ColumnTiling t;
  // Rows whose width is not a multiple of 4 are read 4 floats per lane too,
  // from 5 floats on (see LaneCols): one float per lane needs up to four
  // times the gather instructions, which are what the stream kernels' time
  // follows (forward stream kernel at b = 10 on a KB of 12.9 M entities and
  // 43.7 M triples 2680 -> 780 us, at b = 93 on one of 43 k entities and 190 k
  // triples 47 -> 19 us).
  t.ragged = b % 4 != 0 && b >= kMinRagged;
  t.vec = (b % 4 == 0 || t.ragged) ? 4 : 1;
  const int lanes = (b + t.vec - 1) / t.vec;
  // Lane groups of at most kMaxLpt lanes: wider rows are cut into column
  // slices of 128 columns (4 floats per lane), each a pass of its own over the
  // entries.  A slice's rows are still whole cache lines, and the table a
  // slice gathers from is half the size, so more of it stays in the
  // Infinity Cache: at b = 256 on a 2 M-entity KB, 64-lane groups took
  // 4.02 / 4.03 ms for the dX / dR passes, two 32-lane slices 3.71 / 3.82.
  int lpt = 1;
  while (lpt < lanes && lpt < max_lpt) lpt <<= 1;
  t.lpt = lpt;
  t.width = lpt * t.vec;
  t.n_slices = (b + t.width - 1) / t.width;
  return t;
}

namespace {

// The stream-kernel instance, grid and LDS size launch_stream uses for `a`.
struct StreamChoice {
  const void *fn = nullptr;
  dim3 grid;
  int block = 0;
  size_t lds_bytes = 0;
  int vec = 0, lpt = 0;
  bool narrow = false, ragged = false, buf = false, wt = false, res = false, ldsb = false;
};

hipError_t choose_stream(const StreamArgs &a, const StreamOptions &o, StreamChoice *c) {
  const ColumnTiling t = column_tiling_max(a.b, kMaxLpt);
  if (a.chunk % kChunkQuantum != 0 || a.n % a.chunk != 0) return hipErrorInvalidValue;
  // Raw-buffer offsets are 32-bit and a structured buffer's record stride is
  // at most kMaxStride bytes: tables of 4 GB or more, or rows of more than
  // 4095 floats, take plain loads.
  const uint64_t row_bytes = (uint64_t)a.b * sizeof(float);
  const uint64_t lim = kOutOfRange;
  // The residual passes read A and Z through one raw buffer over both.
  const uint64_t a0 = reinterpret_cast<uintptr_t>(a.A), z0 = reinterpret_cast<uintptr_t>(a.Z);
  const uint64_t span = !a.residual ? 0
                                    : std::max(a0 + (uint64_t)a.A_rows * row_bytes,
                                               z0 + (uint64_t)a.out_rows * row_bytes) -
                                          std::min(a0, z0);
  const uint64_t a_off = a.residual && a0 > z0 ? a0 - z0 : 0;
  const bool buf = !o.plain_loads && span <= lim && row_bytes <= kMaxStride &&
                   (uint64_t)a.A_rows * row_bytes <= lim &&
                   a_off + (uint64_t)a.B_rows * row_bytes <= lim &&
                   a_off + (uint64_t)a.out_rows * row_bytes <= lim &&
                   (uint64_t)a.n_slots * (uint64_t)a.b * sizeof(double) <= lim;
  const bool wt = a.weights != nullptr, res = a.residual != 0;
  if (a.n_lists < 1 || a.n_lists > kMaxChunkLists || a.list_chunk[0] != 0 ||
      a.list_chunk[a.n_lists] != a.n / a.chunk)
    return hipErrorInvalidValue;
  // Every list gets the same number of workgroups (blockIdx.x % n_lists
  // picks the list), enough for its longest list.
  int64_t longest = 0;
  for (int x = 0; x < a.n_lists; ++x) {
    if (a.list_chunk[x + 1] < a.list_chunk[x]) return hipErrorInvalidValue;
    longest = std::max<int64_t>(longest, a.list_chunk[x + 1] - a.list_chunk[x]);
  }
  const int nl = a.n_lists;
  if (a.b <= kMaxNarrow) {
    const size_t table = (size_t)a.B_rows * (size_t)a.b * sizeof(float);
    const bool lds = o.b_in_lds != 0 && table <= kNarrowLds;
    constexpr int64_t groups = kBlock / kNarrowLanes;
    int64_t per_list = std::max<int64_t>(1, (longest + groups - 1) / groups);
    // With B in LDS each workgroup copies it, so there are only so many (eight
    // rounds of those the CUs hold at once; one round was 4 % slower).
    if (lds) per_list = std::min(per_list, std::max<int64_t>(1, (int64_t)kNarrowWgs * std::max(1, o.n_cu) / nl));
    if (per_list * nl > (int64_t)INT32_MAX) return hipErrorInvalidValue;
    c->fn = narrow_fn_for(a.b, lds, wt, res);
    if (!c->fn) return hipErrorInvalidValue;
    c->grid = dim3((unsigned)(per_list * nl));
    c->block = kBlock;
    c->lds_bytes = lds ? table : 0;
    c->vec = a.b;
    c->wt = wt;
    c->res = res;
    c->ldsb = lds;
    c->narrow = true;
    return hipSuccess;
  }
  // The register variant's lane groups: at most o.max_lpt lanes wide.
  const ColumnTiling tr =
      column_tiling_max(a.b, std::max(1, std::min(o.max_lpt, kMaxLpt)));
  const void *reg_fn = stream_fn_for(tr, buf, false, wt, res);
  if (!reg_fn) return hipErrorInvalidValue;
  c->buf = buf;
  c->wt = wt;
  c->res = res;
  c->vec = t.vec;
  c->ragged = t.ragged;
  // B's column slice in LDS when it fits and the LDS variant keeps at least
  // as many waves on a CU as the register variant: where it needs more
  // registers per lane than its workgroup can be given (b = 5 .. 16, the
  // soft KB), B stays in registers.  A slice of at most kMaxLdsB bytes
  // goes with two 768-thread workgroups per CU; for the hard KB a slice of up
  // to kMaxLdsBig bytes goes with one 1024-thread workgroup, and rows wider
  // than 32 columns whose slice is too large are cut into 32-column slices
  // (one 128-byte line of every row each) when that makes B fit.  The grid
  // is as many workgroups as the CUs hold at once, each copying its slice of
  // the table once and walking its chunks grid-stride.
  if (buf && o.b_in_lds != 0) {
    const bool hard = !wt && !res;
    ColumnTiling tl = t;
    size_t lds_bytes = (size_t)a.B_rows * (size_t)tl.width * sizeof(float);
    if (hard && lds_bytes > kMaxLdsB && t.width > 32) {
      tl = column_tiling_max(a.b, 8);
      lds_bytes = (size_t)a.B_rows * (size_t)tl.width * sizeof(float);
    }
    const int blk = lds_bytes <= kMaxLdsB ? kBlockLds : kBlockLdsBig;
    if (lds_bytes <= (hard ? kMaxLdsBig : kMaxLdsB)) {
      const void *fn = stream_fn_for(tl, true, true, wt, res);
      if (!fn) return hipErrorInvalidValue;
      const int per_cu = blocks_per_cu(fn, blk, lds_bytes);
      const int reg_per_cu = blocks_per_cu(reg_fn, kBlock, 0);
      // The LDS variant's large workgroups must still reach every CU: with
      // fewer the small ones of the register variant spread a small KB better
      // (43 k entities, b = 32: 155 workgroups of 768 threads, 8.8 us, against 466
      // of 256, 8.2; 1000 entities, b = 256: forward / dR 7.4 / 9.8 us
      // against 5.6 / 5.6).
      const bool spreads =
          longest * nl * tl.n_slices >= (int64_t)(o.n_cu > 0 ? o.n_cu : 1) * (blk / tl.lpt);
      if (per_cu > 0 &&
          (o.b_in_lds > 1 || (spreads && per_cu * blk >= reg_per_cu * kBlock))) {
        const int64_t cap = (int64_t)per_cu * (o.n_cu > 0 ? o.n_cu : 1);
        const int64_t per_list = std::max<int64_t>(1, std::min<int64_t>(
            (longest + blk / tl.lpt - 1) / (blk / tl.lpt), cap / nl));
        if (per_list * nl > (int64_t)INT32_MAX) return hipErrorInvalidValue;
        c->fn = fn;
        c->grid = dim3((unsigned)(per_list * nl), (unsigned)tl.n_slices);
        c->block = blk;
        c->lds_bytes = lds_bytes;
        c->lpt = tl.lpt;
        c->ldsb = true;
        return hipSuccess;
      }
    }
  }
  const int64_t per_list = std::max<int64_t>(1, (longest + kBlock / tr.lpt - 1) / (kBlock / tr.lpt));
  if (per_list * nl > (int64_t)INT32_MAX) return hipErrorInvalidValue;
  c->fn = reg_fn;
  c->grid = dim3((unsigned)(per_list * nl), (unsigned)tr.n_slices);
  c->block = kBlock;
  c->lds_bytes = 0;
  c->lpt = tr.lpt;
  c->ldsb = false;
  return hipSuccess;
}

const char *tf(bool v) { return v ? "true" : "false"; }

}  // namespace

hipError_t launch_stream(const StreamArgs &a, const StreamOptions &o, hipStream_t s,
                         hipEvent_t start, hipEvent_t stop) {
  if (a.n == 0) return hipSuccess;
  StreamChoice c;
  hipError_t e = choose_stream(a, o, &c);
  if (e != hipSuccess) return e;
  StreamArgs arg = a;
  void *params[] = {&arg};
  if (start || stop)
    return hipExtLaunchKernel(c.fn, c.grid, dim3(c.block), params, c.lds_bytes, s, start, stop, 0);
  return hipLaunchKernel(c.fn, c.grid, dim3(c.block), params, c.lds_bytes, s);
}

std::string describe_stream(const StreamArgs &a, const StreamOptions &o) {
  if (a.n == 0) return "";
  StreamChoice c;
  if (choose_stream(a, o, &c) != hipSuccess) return "";
  char buf[160];
  if (c.narrow) {
    std::snprintf(buf, sizeof buf, "narrow_kernel<%d, %s, %s, %s>", c.vec, tf(c.wt), tf(c.res),
                  tf(c.ldsb));
    return buf;
  }
  std::snprintf(buf, sizeof buf, "stream_kernel<%d, %d, %s, %s, %s, %s>",
                c.ragged ? kRaggedLane : c.vec, c.lpt, tf(c.buf), tf(c.wt), tf(c.res), tf(c.ldsb));
  return buf;
}

std::string describe_fill(bool res) { return std::string("fill_kernel<") + tf(res) + ">"; }

std::string describe_tail(const TailArgs &a) {
  if (a.n_tasks == 0 && a.n_pieces == 0) return "";
  const ColumnTiling t = column_tiling(a.b);
  char buf[96];
  std::snprintf(buf, sizeof buf, "tail_kernel<%d, %d, %s>", t.vec, t.lpt, tf(a.res == nullptr));
  return buf;
}

std::string describe_combine(int32_t b) {
  const ColumnTiling t = column_tiling(b);
  char buf[96];
  std::snprintf(buf, sizeof buf, "combine_kernel<%d, %d>", t.vec, t.lpt);
  return buf;
}

// Blocks of the wide and the other combine tasks of a launch.
static void combine_grid(TailArgs *a, const ColumnTiling &t) {
  a->wide_blocks = a->n_wide * (t.lpt / std::min(t.lpt, kWideLpt));
  a->combine_blocks =
      a->n_tasks > a->n_wide ? blocks_for(a->n_tasks - a->n_wide, kBlock / t.lpt, 0) : 0;
}

hipError_t launch_combine(const int4 *tasks, int64_t n_tasks, int64_t n_wide, double *slots,
                          int64_t n_slots, int32_t b, float *out, int64_t out_rows,
                          const float *res, float gamma, hipStream_t s) {
  if (n_tasks == 0) return hipSuccess;
  const ColumnTiling t = column_tiling(b);
  const void *fn = t.vec == 4 ? combine_fn<4>(t.lpt) : combine_fn<1>(t.lpt);
  if (!fn) return hipErrorInvalidValue;
  TailArgs a{tasks, n_tasks, n_wide, slots, n_slots, nullptr, 0, b, out, out_rows, res, gamma, 0, 0};
  combine_grid(&a, t);
  const dim3 grid((unsigned)(a.wide_blocks + a.combine_blocks), (unsigned)t.n_slices);
  void *params[] = {&a};
  return hipLaunchKernel(fn, grid, dim3(kBlock), params, 0, s);
}

hipError_t launch_fill(float *p, int64_t n, const float *res, float gamma, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = blocks_for(n, kBlock * 4, 0);
  if (blocks * kBlock > (int64_t)UINT32_MAX) return hipErrorInvalidValue;  // see prefill_rows
  void *params[] = {&p, &n, &res, &gamma};
  const void *fn = res ? reinterpret_cast<const void *>(&fill_kernel<true>)
                       : reinterpret_cast<const void *>(&fill_kernel<false>);
  return hipLaunchKernel(fn, dim3((unsigned)blocks), dim3(kBlock), params, 0, s);
}

hipError_t launch_tail(const TailArgs &args, hipStream_t s) {
  if (args.n_tasks == 0 && args.n_pieces == 0) return hipSuccess;
  const ColumnTiling t = column_tiling(args.b);
  const bool packed = args.res == nullptr;
  const void *fn = t.vec == 4 ? (packed ? tail_fn<4, true>(t.lpt) : tail_fn<4, false>(t.lpt))
                              : (packed ? tail_fn<1, true>(t.lpt) : tail_fn<1, false>(t.lpt));
  if (!fn) return hipErrorInvalidValue;
  TailArgs a = args;
  // One combine task per lane group.  Empty rows, packed: LPT pieces per
  // lane group, 256 per block; residual: kFillPieces pieces per lane group.
  combine_grid(&a, t);
  const int64_t zero_blocks =
      a.n_pieces > 0
          ? blocks_for(a.n_pieces, packed ? kBlock : (kBlock / t.lpt) * kFillPieces, 0)
          : 0;
  const int64_t blocks = a.wide_blocks + a.combine_blocks + zero_blocks;
  if (blocks > (int64_t)INT32_MAX) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks, (unsigned)t.n_slices);
  void *params[] = {&a};
  return hipLaunchKernel(fn, grid, dim3(kBlock), params, 0, s);
}

hipError_t checked_violations(unsigned long long *count, bool reset) {
#ifdef KBFOLLOW_CHECKED
  hipError_t e = hipMemcpyFromSymbol(count, HIP_SYMBOL(g_violations), sizeof *count);
  if (e != hipSuccess || !reset) return e;
  const unsigned long long zero = 0;
  return hipMemcpyToSymbol(HIP_SYMBOL(g_violations), &zero, sizeof zero);
#else
  (void)count;
  (void)reset;
  return hipErrorNotSupported;
#endif
}

}  // namespace kbf

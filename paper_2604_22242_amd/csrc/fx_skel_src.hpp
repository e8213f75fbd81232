// The fixed parts of generated kernel source: skeleton kernels written as
// text, shared by both source modes (the run-time one, from a tape's node
// list, and the compile-time one, from an expression's type).  Each piece
// relies on the generated part to define:
//   st_t, ct_t, acc_out_t   storage, compute and dimension-sum output types
//   FX_N, FX_BLOCK, FX_EPT  vector width (elements), block size, EPT
//   FX_NIN                  number of loaded input streams
//   FX_PARAMS / FX_ARGS     the kernel's expression parameters and their names
//   FX_MAP, FX_FINISH       the map before summation and the finish after it
//   fx_load<N>(FX_ARGS, i, raw)   the inputs' N elements at i into raw
//   fx_eval<N>(FX_ARGS, raw, r)   the expression on those N elements
//   fx_at(FX_ARGS, i)             the expression at element i
// The skeletons are those of the compile-time kernels: EPT vectors per input
// loaded before any arithmetic, per-thread sums in FP64 or compensated,
// FP64 wave64 + LDS block sums and the single-pass agent-scope ticket finish.
#pragma once

#include "fx.h"

namespace fx {

// Kernel names of a result kind: [vector variant, one-element variant].
inline int skeleton_kernels(int kind, const char** names) {
  switch (kind) {
    case 0: names[0] = "fx_rtc_ew"; return 1;
    case FX_R_ACCU: case FX_R_NORM: names[0] = "fx_rtc_full"; return 1;
    case FX_R_COLSUM: names[0] = "fx_rtc_colsum_v"; names[1] = "fx_rtc_colsum_s"; return 2;
    default: names[0] = "fx_rtc_rowsum_v"; names[1] = "fx_rtc_rowsum_s"; return 2;
  }
}


// Loads: N consecutive elements at p, one 16-byte streaming load (N = FX_N;
// any element may start it: columns need not be whole vectors) or one element
// (N = 1).
inline constexpr char kLoads[] = R"(typedef unsigned int fx_u32x4 __attribute__((ext_vector_type(4)));
typedef fx_u32x4 fx_u32x4_at __attribute__((aligned(alignof(st_t))));
template <int N> struct fx_ld {
  __device__ static __forceinline__ void run(const st_t* p, st_t* o) {
    const fx_u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const fx_u32x4_at*>(p));
    __builtin_memcpy(o, &v, 16);
  }
};
template <> struct fx_ld<1> {
  __device__ static __forceinline__ void run(const st_t* p, st_t* o) { o[0] = *p; }
};
template <int N> struct fx_raw { st_t v[FX_NIN][N]; };
)";

// Element-wise: tiles of FX_BLOCK * FX_EPT vectors, the EPT loads of every
// input issued before any arithmetic; the last block also does the
// n % FX_N scalar tail.
inline constexpr char kElementwise[] = R"(
__device__ __forceinline__ void fx_store(st_t* z, const ct_t* r) {
  st_t s[FX_N];
#pragma unroll
  for (int j = 0; j < FX_N; ++j) s[j] = (st_t)r[j];
  fx_u32x4 v;
  __builtin_memcpy(&v, s, 16);
  *reinterpret_cast<fx_u32x4*>(z) = v;
}

extern "C" __global__ __launch_bounds__(FX_BLOCK) void fx_rtc_ew(FX_PARAMS, st_t* __restrict__ z,
                                                                 long n) {
  const long nv = n / FX_N;
  const long tile = (long)FX_BLOCK * FX_EPT;
  for (long t = blockIdx.x; t * tile < nv; t += gridDim.x) {
    const long v0 = t * tile + threadIdx.x;
    if ((t + 1) * tile <= nv) {
      fx_raw<FX_N> raw[FX_EPT];
      ct_t r[FX_EPT][FX_N];
#pragma unroll
      for (int k = 0; k < FX_EPT; ++k) fx_load<FX_N>(FX_ARGS, (v0 + (long)k * FX_BLOCK) * FX_N, raw[k]);
      __builtin_amdgcn_sched_barrier(0);  // every load ahead of the arithmetic
#pragma unroll
      for (int k = 0; k < FX_EPT; ++k) fx_eval<FX_N>(FX_ARGS, raw[k], r[k]);
#pragma unroll
      for (int k = 0; k < FX_EPT; ++k) fx_store(z + (v0 + (long)k * FX_BLOCK) * FX_N, r[k]);
    } else {
#pragma unroll
      for (int k = 0; k < FX_EPT; ++k) {
        const long v = v0 + (long)k * FX_BLOCK;
        if (v < nv) {
          fx_raw<FX_N> raw;
          ct_t r[FX_N];
          fx_load<FX_N>(FX_ARGS, v * FX_N, raw);
          fx_eval<FX_N>(FX_ARGS, raw, r);
          fx_store(z + v * FX_N, r);
        }
      }
    }
  }
  if (blockIdx.x == gridDim.x - 1)
    for (long i = nv * FX_N + threadIdx.x; i < n; i += FX_BLOCK) z[i] = (st_t)fx_at(FX_ARGS, i);
}
)";

// Sums, as in the compile-time skeletons: per-thread sums in FP64 where the
// compute type is FP32, compensated ones (Neumaier's refinement of Kahan's
// method: c collects the exact rounding error of every addition into s, taken
// with Knuth's TwoSum) where it is FP64, one add per element, handed upward in
// FP64; the block sum is a
// wave64 butterfly and then the waves' results in order; partials are
// published with agent-scope stores and the block that draws the last ticket
// of an agent-scope counter adds them in index order after one acquire, then
// clears the counter and them.
inline constexpr char kSums[] = R"(
template <class C> struct fx_acc_of {
  C s = 0, c = 0;
  __device__ __forceinline__ void add(C t) {
#pragma clang fp contract(off)
    const C u = s + t;
    const C tv = u - s, sv = u - tv;  // TwoSum: the exact error of s + t
    c += (s - sv) + (t - tv);
    s = u;
  }
  __device__ __forceinline__ double value() const {
    return __builtin_isfinite(s) ? (double)s + (double)c : (double)s;
  }
};
template <> struct fx_acc_of<float> {
  double s = 0;
  __device__ __forceinline__ void add(float t) { s += (double)t; }
  __device__ __forceinline__ double value() const { return s; }
};
typedef fx_acc_of<ct_t> fx_acc;
__device__ __forceinline__ void fx_add(fx_acc& a, ct_t t) { a.add(t); }
__device__ __forceinline__ double fx_value(const fx_acc& a) { return a.value(); }
// one chain per vector lane, added in FP64 in lane order
template <int N> __device__ __forceinline__ double fx_lanes_value(const fx_acc (&a)[N]) {
  double t = fx_value(a[0]);
#pragma unroll
  for (int j = 1; j < N; ++j) t += fx_value(a[j]);
  return t;
}

__device__ __forceinline__ double fx_block_sum(double v, double* lds) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  __syncthreads();
  if (lane == 0) lds[wave] = v;
  __syncthreads();
  double t = 0;
  for (unsigned w = 0; w < blockDim.x / 64; ++w) t += lds[w];
  return t;
}

__device__ __forceinline__ void fx_publish(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool fx_last_ticket(unsigned* counter, unsigned expected) {
  __shared__ bool last;
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0)
    last = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
           expected - 1;
  __syncthreads();
  if (last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  return last;
}
__device__ __forceinline__ void fx_reset(unsigned* counter) {
  __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
)";

// Full reduction: out = FX_FINISH(sum FX_MAP(E_i)), one FP64 value; blocks
// walk tiles of FX_BLOCK * FX_EPT vectors grid-stride.
inline constexpr char kFull[] = R"(
extern "C" __global__ __launch_bounds__(FX_BLOCK) void fx_rtc_full(FX_PARAMS, long n, double* partials,
                                                                   unsigned* counter, double* out) {
  __shared__ double lds[FX_BLOCK / 64];
  fx_acc acc[FX_N];
  const long nv = n / FX_N;
  const long tile = (long)FX_BLOCK * FX_EPT;
  for (long t = blockIdx.x; t * tile < nv; t += gridDim.x) {
    const long v0 = t * tile + threadIdx.x;
    if ((t + 1) * tile <= nv) {
      fx_raw<FX_N> raw[FX_EPT];
      ct_t r[FX_EPT][FX_N];
#pragma unroll
      for (int k = 0; k < FX_EPT; ++k) fx_load<FX_N>(FX_ARGS, (v0 + (long)k * FX_BLOCK) * FX_N, raw[k]);
      __builtin_amdgcn_sched_barrier(0);  // every load ahead of the arithmetic
#pragma unroll
      for (int k = 0; k < FX_EPT; ++k) fx_eval<FX_N>(FX_ARGS, raw[k], r[k]);
#pragma unroll
      for (int k = 0; k < FX_EPT; ++k)
#pragma unroll
        for (int j = 0; j < FX_N; ++j) fx_add(acc[j], FX_MAP(r[k][j]));
    } else {
#pragma unroll
      for (int k = 0; k < FX_EPT; ++k) {
        const long v = v0 + (long)k * FX_BLOCK;
        if (v < nv) {
          fx_raw<FX_N> raw;
          ct_t r[FX_N];
          fx_load<FX_N>(FX_ARGS, v * FX_N, raw);
          fx_eval<FX_N>(FX_ARGS, raw, r);
#pragma unroll
          for (int j = 0; j < FX_N; ++j) fx_add(acc[j], FX_MAP(r[j]));
        }
      }
    }
  }
  if (blockIdx.x == gridDim.x - 1)
    for (long i = nv * FX_N + threadIdx.x; i < n; i += FX_BLOCK) fx_add(acc[0], FX_MAP(fx_at(FX_ARGS, i)));
  const double s = fx_block_sum(fx_lanes_value(acc), lds);
  if (gridDim.x == 1) {
    if (threadIdx.x == 0) *out = FX_FINISH(s);
    return;
  }
  if (threadIdx.x == 0) fx_publish(partials + blockIdx.x, s);
  if (fx_last_ticket(counter, gridDim.x)) {
    double t = 0;
    for (unsigned b = threadIdx.x; b < gridDim.x; b += FX_BLOCK) {
      t += partials[b];
      partials[b] = 0.0;
    }
    t = fx_block_sum(t, lds);
    if (threadIdx.x == 0) {
      *out = FX_FINISH(t);
      fx_reset(counter);
    }
  }
}
)";

// Column sums: block (column c, chunk s) sums rows [s*rpc, (s+1)*rpc) of
// column c, a contiguous run; with split > 1 the chunk partials go to
// partials[c*split + s] and the last block of column c adds them in chunk
// order.  rpc is a multiple of N; the last rows that are no whole vector are
// taken as one that overlaps the one before (n_rows >= N).  FX_BLOCK bounds the
// threads; a launch has as many as the column has work for, by the same rule as
// the compile-time skeleton (128 x 32768 FP32, matrix workload: 64 threads 13 us,
// 512 92).
inline constexpr char kColsum[] = R"(
template <int N>
__device__ __forceinline__ void fx_colsum(FX_PARAMS, long n_rows, int split, long rpc, double* partials,
                                          unsigned* counters, acc_out_t* out) {
  __shared__ double lds[FX_BLOCK / 64];
  const long col = blockIdx.x;
  const int s = blockIdx.y;
  const long r0 = (long)s * rpc;
  const long r1 = n_rows < r0 + rpc ? n_rows : r0 + rpc;
  const long base = col * n_rows + r0;
  const long nv = r1 > r0 ? (r1 - r0) / N : 0;
  const long nvt = r1 > r0 + nv * N ? nv + 1 : nv;  // with the overlapping vector
  fx_acc acc[N];
  const long tile = (long)blockDim.x * FX_EPT;
  for (long t0 = 0; t0 < nvt; t0 += tile) {
    const long v0 = t0 + threadIdx.x;
    if (t0 + tile <= nv) {
      fx_raw<N> raw[FX_EPT];
      ct_t r[FX_EPT][N];
#pragma unroll
      for (int k = 0; k < FX_EPT; ++k) fx_load<N>(FX_ARGS, base + (v0 + (long)k * blockDim.x) * N, raw[k]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < FX_EPT; ++k) fx_eval<N>(FX_ARGS, raw[k], r[k]);
#pragma unroll
      for (int k = 0; k < FX_EPT; ++k)
#pragma unroll
        for (int j = 0; j < N; ++j) fx_add(acc[j], r[k][j]);
    } else {
#pragma unroll
      for (int k = 0; k < FX_EPT; ++k) {
        const long v = v0 + (long)k * blockDim.x;
        if (v < nvt) {
          const int lo = v < nv ? 0 : (int)((nv + 1) * N - (r1 - r0));
          fx_raw<N> raw;
          ct_t r[N];
          fx_load<N>(FX_ARGS, base + v * N - lo, raw);
          fx_eval<N>(FX_ARGS, raw, r);
#pragma unroll
          for (int j = 0; j < N; ++j) fx_add(acc[j], j >= lo ? r[j] : (ct_t)0);
        }
      }
    }
  }
  const double sum = fx_block_sum(fx_lanes_value(acc), lds);
  if (split == 1) {
    if (threadIdx.x == 0) out[col] = (acc_out_t)sum;
    return;
  }
  if (threadIdx.x == 0) fx_publish(partials + col * split + s, sum);
  if (fx_last_ticket(counters + col, split)) {
    if (threadIdx.x == 0) {
      double t = 0;
      for (int q = 0; q < split; ++q) t += partials[col * split + q];
      out[col] = (acc_out_t)t;
      fx_reset(counters + col);
    }
    __syncthreads();
    for (int q = threadIdx.x; q < split; q += blockDim.x) partials[col * split + q] = 0.0;
  }
}
extern "C" __global__ __launch_bounds__(FX_BLOCK) void fx_rtc_colsum_v(FX_PARAMS, long n_rows, int split,
    long rpc, double* partials, unsigned* counters, acc_out_t* out) {
  fx_colsum<FX_N>(FX_ARGS, n_rows, split, rpc, partials, counters, out);
}
extern "C" __global__ __launch_bounds__(FX_BLOCK) void fx_rtc_colsum_s(FX_PARAMS, long n_rows, int split,
    long rpc, double* partials, unsigned* counters, acc_out_t* out) {
  fx_colsum<1>(FX_ARGS, n_rows, split, rpc, partials, counters, out);
}
)";

// Row sums, as the compile-time skeleton: a block owns rl * N rows and every
// split-th step of S * FX_EPT columns, thread group g (rl threads: one column's
// rows as vectors) every S-th column of a step; the groups' sums are added
// through LDS and with split > 1 the last block of a row tile adds the chunk
// partials.  The matrix's last rows that are no whole vector are taken as one
// that overlaps the one before (n_rows >= N).
inline constexpr char kRowsum[] = R"(
__device__ __forceinline__ double fx_groups(const double* lds, int rows, int i, int groups) {
  double t = lds[i];
  for (int g = 1; g < groups; ++g) t += lds[g * rows + i];
  return t;
}
template <int N>
__device__ __forceinline__ void fx_rowsum(FX_PARAMS, long n_rows, long n_cols, int split, int rl,
                                          double* partials, unsigned* counters,
                                          acc_out_t* out) {
  __shared__ double lds[FX_BLOCK * N];
  // where columns are no whole number of cache lines, the row tiles of one
  // chunk (which share lines) run on one of the eight XCDs
  unsigned b = blockIdx.y * gridDim.x + blockIdx.x;
  if (n_rows * (long)sizeof(st_t) % 128) {
    const unsigned G = gridDim.x * gridDim.y, xcd = b % 8;
    b = xcd * (G / 8) + (xcd < G % 8 ? xcd : G % 8) + b / 8;
  }
  const int s = b / gridDim.x, tile = b % gridDim.x, t = threadIdx.x;
  const int rows = rl * N, S = FX_BLOCK / rl;
  const int lr = t % rl, g = t / rl;
  const long row0 = (long)tile * rows;
  const long first = row0 + lr * N;
  const int sh = first + N > n_rows && first < n_rows ? (int)(first + N - n_rows) : 0;
  const long r0 = first - sh;  // lanes below sh repeat rows of the vector before
  fx_acc acc[N];
  if (first < n_rows) {
    long c = (long)s * (FX_EPT * S) + g;
    for (; c + (FX_EPT - 1) * S < n_cols; c += (long)split * (FX_EPT * S)) {
      fx_raw<N> raw[FX_EPT];
      ct_t r[FX_EPT][N];
#pragma unroll
      for (int k = 0; k < FX_EPT; ++k) fx_load<N>(FX_ARGS, r0 + (c + k * S) * n_rows, raw[k]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k < FX_EPT; ++k) fx_eval<N>(FX_ARGS, raw[k], r[k]);
#pragma unroll
      for (int j = 0; j < N; ++j)  // row j's FX_EPT columns, in column order
#pragma unroll
        for (int k = 0; k < FX_EPT; ++k) fx_add(acc[j], r[k][j]);
    }
    for (; c < n_cols; c += S) {  // (fewer than FX_EPT of them)
      fx_raw<N> raw;
      ct_t r[N];
      fx_load<N>(FX_ARGS, r0 + c * n_rows, raw);
      fx_eval<N>(FX_ARGS, raw, r);
#pragma unroll
      for (int j = 0; j < N; ++j) fx_add(acc[j], r[j]);
    }
  }
  if (S == 1 && split == 1) {  // a row is one thread's
    if (first < n_rows)
#pragma unroll
      for (int j = 0; j < N; ++j)
        if (j >= sh) out[r0 + j] = (acc_out_t)fx_value(acc[j]);
    return;
  }
#pragma unroll
  for (int j = 0; j < N; ++j)
    if (j >= sh) lds[t * N + j - sh] = fx_value(acc[j]);
  __syncthreads();
  for (int i = t; i < rows; i += FX_BLOCK) {
    if (row0 + i >= n_rows) break;
    const double v = fx_groups(lds, rows, i, S);
    if (split == 1) out[row0 + i] = (acc_out_t)v;
    else fx_publish(partials + (long)s * n_rows + row0 + i, v);
  }
  if (split == 1) return;
  if (fx_last_ticket(counters + tile, split)) {
    const int fl = rl > 64 ? rl : rows < 64 ? rows : 64, F = FX_BLOCK / fl, f = t / fl;
    double sum[N];
#pragma unroll
    for (int j = 0; j < N; ++j) sum[j] = 0;
    constexpr int U = N >= 8 ? 4 : 8;
    for (int q = f; q < split; q += U * F) {
      double v[U][N];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < N; ++j) {
          const int i = t % fl + fl * j;
          const bool in = i < rows && row0 + i < n_rows && q + u * F < split;
          v[u][j] = in ? partials[(long)(q + u * F) * n_rows + row0 + i] : 0.0;
        }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < N; ++j) sum[j] += v[u][j];
    }
#pragma unroll
    for (int j = 0; j < N; ++j)
      if (t % fl + fl * j < rows) lds[f * rows + t % fl + fl * j] = sum[j];
    __syncthreads();
    for (int i = t; i < rows; i += FX_BLOCK)
      if (row0 + i < n_rows) out[row0 + i] = (acc_out_t)fx_groups(lds, rows, i, F);
    for (int i = t % fl; i < rows && row0 + i < n_rows; i += fl)
      for (int q = f; q < split; q += F) partials[(long)q * n_rows + row0 + i] = 0.0;
    if (t == 0) fx_reset(counters + tile);
  }
}
extern "C" __global__ __launch_bounds__(FX_BLOCK) void fx_rtc_rowsum_v(FX_PARAMS, long n_rows, long n_cols,
    int split, int rl, double* partials, unsigned* counters, acc_out_t* out) {
  fx_rowsum<FX_N>(FX_ARGS, n_rows, n_cols, split, rl, partials, counters, out);
}
extern "C" __global__ __launch_bounds__(FX_BLOCK) void fx_rtc_rowsum_s(FX_PARAMS, long n_rows, long n_cols,
    int split, int rl, double* partials, unsigned* counters, acc_out_t* out) {
  fx_rowsum<1>(FX_ARGS, n_rows, n_cols, split, rl, partials, counters, out);
}
)";

}  // namespace fx

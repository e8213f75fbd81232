// Skeleton kernels for gfx950 and their host launchers.
//
// Each skeleton is a fixed recipe with the expression as a template
// parameter (Sec. 3: one skeleton kernel serves virtually every expression of
// the form Y = <rhs>).  The skeletons here:
//   k_ew        Z[i] = E(i)                      ("copy" skeleton)
//   k_full      sum_i map(E(i)) -> one value     (accu, dot, norm_fro)
//   k_colsum    sum over rows, per column        (sum(E, 0))
//   k_colsum_thin  same for very short columns (one thread per column)
//   k_rowsum    sum over columns, per row        (sum(E, 1))
//
// Memory access: wave64, each lane moves one vector of N elements (16 bytes
// by default) per load; a block covers a contiguous tile of
// blockDim * EPT vectors, the EPT loads of every leaf are independent and
// issued before any result is stored.  Full reductions combine the block
// partials in FP64 in one pass: the last block to finish (agent-scope
// ticket) adds them in index order, so a fixed launch configuration gives
// bitwise-reproducible results.
#pragma once

#include <algorithm>
#include <type_traits>
#include <utility>

#include "fx_expr.hpp"

// Cache policy of streamed loads and stores (measured on MI355X: streaming
// loads raise the read ceiling from 6.4 to 7.1 TB/s).  FX_NT_STORES forces
// streaming stores everywhere; by default the element-wise kernel chooses
// per launch: stores from the size of its output (kStreamStoresAbove), loads
// from all it touches (kCachedLoadsUpTo).
#ifndef FX_NT_LOADS
#define FX_NT_LOADS 1
#endif
#ifndef FX_NT_STORES
#define FX_NT_STORES 0
#endif


namespace fx {

constexpr int kMaxBlock = 512;
constexpr bool kNT = FX_NT_LOADS != 0;    // streaming policy for loads
constexpr bool kNTS = FX_NT_STORES != 0;  // streaming policy for stores

// Outputs larger than MI355X's 256 MiB last-level cache (the Infinity Cache)
// are written with streaming stores.  Measured for X%Y + 2W in FP32: up to a
// 256 MiB output, ordinary stores run at 6.6-6.7 TB/s (the output stays in
// that cache) against 6.1-6.2 streaming; from 320 MiB on, ordinary stores
// fall to 6.0-6.1 TB/s and streaming stores keep 6.2-6.3.
constexpr uint64_t kStreamStoresAbove = uint64_t(256) << 20;
// Inputs and output that fit that cache together are read with ordinary loads,
// which leave the inputs there for the next call on them.  The matrix workload's
// Z, three inputs and an output, streaming against ordinary loads, us repeated
// (after the caches were flushed):
//   of 8 MiB each    FP32  5.2 (10.0)    4.5 (10.6)    BF16  8.1 (10.6)   6.0 (11.4)
//   of 32 MiB        FP32 23.7 (26.3)   20.0 (25.6)    BF16 25.3 (27.5)  21.3 (26.7)
//   of 64 MiB        FP32 42.8 (45.5)   37.3 (45.7)    BF16 44.9 (47.0)  38.8 (46.7)
//   of 96 MiB        FP32 62.1 (64.2)   71.2 (68.0)    BF16 65.1 (67.2)  68.8 (67.3)
// Reductions keep streaming loads at every size: FP32 column sums of 32 MiB
// inputs 17.5 (20.4) against 17.9 (21.9), of 64 MiB 31.0 (33.6), 30.2 (36.9).
// Tapes keep them too: they are bound by their interpreter.
constexpr uint64_t kCachedLoadsUpTo = uint64_t(256) << 20;

// Maps applied to each element before summation.
struct map_id {
  template <class C> __device__ static C f(C x) { return x; }
  __host__ __device__ static double finish(double s) { return s; }
  __host__ __device__ static uint64_t finish(uint64_t s) { return s; }
};
struct map_sq {
  template <class C> __device__ static C f(C x) { return x * x; }
  __device__ static double finish(double s) { return ::sqrt(s); }
};

// Add the map M of a thread's EPT x N values of one tile to its
// lane sums, one element at a time (lane j's chain takes vector 0's, then
// vector 1's ... element j).
template <class M, int N, int EPT, class C>
__device__ __forceinline__ void add_tile(lane_accum<C, N>& acc, const lanes<C, N> (&r)[EPT]) {
#pragma unroll
  for (int k = 0; k < EPT; ++k)
#pragma unroll
    for (int j = 0; j < N; ++j) acc.a[j].add(M::f(r[k].v[j]));
}
template <class M, int N, class C>
__device__ __forceinline__ void add_lanes(lane_accum<C, N>& acc, const lanes<C, N>& r) {
#pragma unroll
  for (int j = 0; j < N; ++j) acc.a[j].add(M::f(r.v[j]));
}

// EPT vectors of N elements at base, base + stride, ...: every leaf's loads
// are issued before any arithmetic (two phases: the register leaves of all
// EPT vectors, then the tree from registers, with a scheduling barrier
// between them; left to itself the scheduler may hold a vector's loads back
// until the previous one has arrived when little arithmetic follows).
// Expression types with their own evaluation strategy (the run-time tape)
// overload this.
template <int N, int EPT, bool NTL = kNT, class E>
__device__ __forceinline__ void eval_tile(const E& e, int64_t base, int64_t stride,
                                          lanes<typename E::ct, N> (&r)[EPT]) {
  constexpr int L = leaves_of<E>::value;
  if constexpr (L >= 1 && L <= kMaxFusedLeaves) {
    lanes<typename E::ct, N> regs[EPT][L];
    const uint8_t* no_alias = nullptr;
#pragma unroll
    for (int k = 0; k < EPT; ++k) e.template gather<0, N, NTL>(regs[k], no_alias, base + k * stride);
    __builtin_amdgcn_sched_barrier(0);  // keep every load ahead of the arithmetic
#pragma unroll
    for (int k = 0; k < EPT; ++k) r[k] = e.template at_regs<0, N, NTL>(regs[k], base + k * stride);
  } else {
#pragma unroll
    for (int k = 0; k < EPT; ++k) r[k] = e.template at_vec<N, NTL>(base + k * stride);
  }
}

// Fused<E>: the loads of all EPT vectors first, then the arithmetic.
template <int N, int EPT, bool NTL = kNT, class E>
__device__ __forceinline__ void eval_tile(const Fused<E>& f, int64_t base, int64_t stride,
                                          lanes<typename E::ct, N> (&r)[EPT]) {
  lanes<typename E::ct, N> regs[EPT][Fused<E>::L];
#pragma unroll
  for (int k = 0; k < EPT; ++k) f.e.template gather<0, N, NTL>(regs[k], f.alias, base + k * stride);
#pragma unroll
  for (int k = 0; k < EPT; ++k) {
    f.template resolve<N>(regs[k]);
    r[k] = f.e.template at_regs<0, N, NTL>(regs[k], base + k * stride);
  }
}

// Workgroups are dispatched to the eight XCDs round-robin by block id, and
// each XCD has its own L2.  Where a leading dimension is not a multiple of
// the 128-byte line (10000 floats = 40000 B), vertically adjacent tiles
// share the line their column runs straddle; under the plain order those two
// tiles run on different XCDs and both fetch it from HBM (12% more reads for
// submatrices, 25% with transposes).  xcd_order() gives each XCD a
// contiguous run of tiles instead (a bijection on [0, G)), so the second
// fetch of a shared line is an L2 hit.
constexpr uint32_t kXcds = 8;
__device__ __forceinline__ uint32_t xcd_order(uint32_t b, uint32_t G) {
  const uint32_t per = G / kXcds, extra = G % kXcds;
  const uint32_t xcd = b % kXcds, k = b / kXcds;
  return xcd * per + (xcd < extra ? xcd : extra) + k;
}

// ============================================================================
// Element-wise: Z[i] = E(i), i < n.

// NTS: streaming stores, NTL: streaming loads.  The policies are template
// parameters: a run-time choice between two otherwise identical stores is merged
// by the compiler into one store, which drops the streaming hint.
template <class E, class T, int N, int EPT, bool NTS, bool NTL = kNT>
__global__ __launch_bounds__(kMaxBlock) void k_ew(E e, T* __restrict__ z, int64_t n) {
  using C = typename E::ct;
  const int64_t nv = n / N;  // whole vectors
  const int64_t tile = (int64_t)blockDim.x * EPT;
  // tile t exists while t * tile < nv (no 64-bit division: gfx950 has no
  // scalar divide, and its emulation would delay every wave's first load)
  for (int64_t t = blockIdx.x; t * tile < nv; t += gridDim.x) {
    const int64_t v0 = t * tile + threadIdx.x;
    if ((t + 1) * tile <= nv) {
      lanes<C, N> r[EPT];
      eval_tile<N, EPT, NTL>(e, v0 * N, (int64_t)blockDim.x * N, r);
#pragma unroll
      for (int k = 0; k < EPT; ++k) store_lanes<N, NTS>(z, (v0 + k * blockDim.x) * N, r[k]);
    } else {
#pragma unroll
      for (int k = 0; k < EPT; ++k) {
        const int64_t v = v0 + k * blockDim.x;
        if (v < nv) store_lanes<N, NTS>(z, v * N, e.template at_vec<N, NTL>(v * N));
      }
    }
  }
  if (N > 1 && blockIdx.x == gridDim.x - 1) {
    for (int64_t i = nv * N + threadIdx.x; i < n; i += blockDim.x) z[i] = static_cast<T>(e.at(i));
  }
}

// ============================================================================
// Full reduction: out = finish(sum_i map(E(i))).  partials: gridDim.x wide
// values; counter: one unsigned, zero on entry, zero again on exit.

template <class E, class M, class O, int N, int EPT>
__global__ __launch_bounds__(kMaxBlock) void k_full(E e, int64_t n, typename wide<typename E::ct>::type* partials,
                                                  unsigned* counter, O* out) {
  using C = typename E::ct;
  using D = typename wide<C>::type;
  __shared__ D lds[kMaxBlock / 64];
  lane_accum<C, N> acc;
  const int64_t nv = n / N;
  const int64_t tile = (int64_t)blockDim.x * EPT;
  // tile t exists while t * tile < nv (no 64-bit division: gfx950 has no
  // scalar divide, and its emulation would delay every wave's first load)
  for (int64_t t = blockIdx.x; t * tile < nv; t += gridDim.x) {
    const int64_t v0 = t * tile + threadIdx.x;
    if ((t + 1) * tile <= nv) {
      lanes<C, N> r[EPT];
      eval_tile<N, EPT>(e, v0 * N, (int64_t)blockDim.x * N, r);
      add_tile<M>(acc, r);
    } else {
#pragma unroll
      for (int k = 0; k < EPT; ++k) {
        const int64_t v = v0 + k * blockDim.x;
        if (v < nv) add_lanes<M>(acc, e.template at_vec<N, kNT>(v * N));
      }
    }
  }
  if (N > 1 && blockIdx.x == gridDim.x - 1) {
    for (int64_t i = nv * N + threadIdx.x; i < n; i += blockDim.x) acc.a[0].add(M::f(e.at(i)));
  }
  D s = block_sum<D>(acc.value(), lds);
  if (gridDim.x == 1) {
    if (threadIdx.x == 0) *out = static_cast<O>(M::finish(s));
    return;
  }
  if (threadIdx.x == 0) publish(partials + blockIdx.x, s);
  if (take_last_ticket(counter, gridDim.x)) {
    D t = 0;
    for (unsigned b = threadIdx.x; b < gridDim.x; b += blockDim.x) {
      t += partials[b];
      partials[b] = D(0);
    }
    t = block_sum<D>(t, lds);
    if (threadIdx.x == 0) {
      *out = static_cast<O>(M::finish(t));
      reset_counter(counter);
    }
  }
}

// ============================================================================
// Column sums.  Block (column c, chunk s) sums rows [s*rpc, (s+1)*rpc) of
// column c: a contiguous run read blockDim * N elements at a time, EPT loads
// per input in flight.  With split > 1 the chunk partials go to
// partials[c*split + s] and the block that draws the last ticket on
// counters[c] adds them in chunk order.  rpc is a multiple of N; the rows of the
// last chunk that are no whole vector are taken as one that ends with the
// column and overlaps the one before (n_rows >= N), its first lanes left out.
//
// Columns that are no multiple of N rows long start at any element, where
// loads of single elements, the alternative, are bound by their issue: 6001 x
// 2999 FP16 80 us, with vectors at any element 28.

template <class E, class O, int N, int EPT>
__global__ __launch_bounds__(kMaxBlock) void k_colsum(E e, int64_t n_rows, int split, int64_t rpc,
                                                    typename wide<typename E::ct>::type* partials,
                                                    unsigned* counters, O* out) {
  using C = typename E::ct;
  using D = typename wide<C>::type;
  __shared__ D lds[kMaxBlock / 64];
  const int64_t col = blockIdx.x;
  const int s = blockIdx.y;
  const int64_t r0 = (int64_t)s * rpc;
  const int64_t r1 = min(n_rows, r0 + rpc);
  const int64_t base = col * n_rows + r0;
  const int64_t nv = r1 > r0 ? (r1 - r0) / N : 0;
  // vectors with the overlapping one
  const int64_t nvt = r1 > r0 + nv * N ? nv + 1 : nv;
  lane_accum<C, N> acc;
  const int64_t tile = (int64_t)blockDim.x * EPT;
  for (int64_t t0 = 0; t0 < nvt; t0 += tile) {
    const int64_t v0 = t0 + threadIdx.x;
    if (t0 + tile <= nv) {
      lanes<C, N> r[EPT];
      eval_tile<N, EPT>(e, base + v0 * N, (int64_t)blockDim.x * N, r);
      add_tile<map_id>(acc, r);
    } else {
#pragma unroll
      for (int k = 0; k < EPT; ++k) {
        const int64_t v = v0 + k * blockDim.x;
        if (v < nvt) {
          // lanes from `lo` on are new (0 but for the overlapping vector)
          const int lo = v < nv ? 0 : (int)((nv + 1) * N - (r1 - r0));
          const lanes<C, N> r = e.template at_vec<N, kNT>(base + v * N - lo);
#pragma unroll
          for (int j = 0; j < N; ++j) acc.a[j].add(j >= lo ? r.v[j] : C(0));
        }
      }
    }
  }
  const D sum = block_sum<D>(acc.value(), lds);
  if (split == 1) {
    if (threadIdx.x == 0) out[col] = static_cast<O>(sum);
    return;
  }
  if (threadIdx.x == 0) publish(partials + col * split + s, sum);
  if (take_last_ticket(counters + col, split)) {
    if (threadIdx.x == 0) {
      out[col] = static_cast<O>(sum_strided<D>(partials + col * split, 1, split));
      reset_counter(counters + col);
    }
    __syncthreads();
    for (int q = threadIdx.x; q < split; q += blockDim.x) partials[col * split + q] = D(0);
  }
}

// Short columns: thread c sums column c, rows in order, no cross-thread combine.
// What bounds it is the loads: lanes lie a column apart, so that each one touches
// a cache line of its own, and a wave has as many in flight as the loop lets it.
// Two vectors per input at a time, the rows at the end as one vector that ends
// with the column (n_rows >= N, its first lanes left out), ordinary loads (the
// next vector is often in the same line).  Matrix workload, 32 x 2^21 BF16: 193
// us; a row at a time 592 with the library's exp, 1400 with the check that
// exp_lanes makes between two rows.  16 x 2^22 FP32 likewise 205, 656, 1350; 9 x
// 7456540 FP64 489, 754 (its exp has no such check).
template <class E, class O, int N>
__global__ __launch_bounds__(kMaxBlock) void k_colsum_thin(E e, int64_t n_rows, int64_t n_cols, O* out) {
  using C = typename E::ct;
  constexpr int U = 2;
  for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < n_cols;
       c += (int64_t)gridDim.x * blockDim.x) {
    const int64_t base = c * n_rows;
    accum<C> acc;
    int64_t r = 0;
    for (; r + U * N <= n_rows; r += U * N) {
      lanes<C, N> v[U];
      eval_tile<N, U, false>(e, base + r, N, v);
#pragma unroll
      for (int k = 0; k < U; ++k)
#pragma unroll
        for (int j = 0; j < N; ++j) acc.add(v[k].v[j]);
    }
    for (; r < n_rows; r += N) {
      const int lo = r + N > n_rows ? (int)(r + N - n_rows) : 0;
      const lanes<C, N> v = e.template at_vec<N, false>(base + r - lo);
#pragma unroll
      for (int j = 0; j < N; ++j) acc.add(j >= lo ? v.v[j] : C(0));
    }
    out[c] = static_cast<O>(acc.value());
  }
}

// ============================================================================
// Row sums.  A block owns a tile of rl * N rows (rl lanes hold one column's
// rows as vectors, so the block reads S = blockDim / rl columns at a time) and chunk s of the columns: steps s, s + split, ... of
// S * EPT columns each.  Thread group g takes every S-th column of a step, EPT
// loads per input in flight.  The S partial sums of a row are added through
// LDS in group order; with split > 1 the chunk partials go to
// partials[s*n_rows + r], and the block that draws the last ticket of its row
// tile (counters[blockIdx.x]) adds them, all its waves reading, in a fixed
// order.  The last rows of a tile that are no whole vector are taken as one that
// ends with the matrix's rows and overlaps the one before (n_rows >= N); single
// elements, the alternative for n_rows no multiple of N, made 133 us of 6001 x
// 2999 FP16 where this takes 35.
//
// What bounds it is HBM (BF16: the expression's arithmetic), provided that
// * the partials are few and the finish short.  With a chunk per wave and no
//   combine in the block the BF16 matrix workload published 128 partials per
//   row, which its last blocks added one wave per 512 rows: 210 us;
// * the blocks sweep memory together.  With a contiguous run of columns per
//   chunk the chunks' streams lie megabytes apart: FP32 matrix workload 149 us,
//   with interleaved steps and otherwise alike 126, with two blocks per CU 118
//   (its column sums, contiguous by nature: 118-120).
// Now BF16 97, FP32 118, FP64 234 us; with the former kernel 210, 151, 270.
// Dynamic LDS: blockDim * N values.

// Lanes that share a column: a wave's 64, n_rows in vectors of `vec` elements where
// that is less, and fewer (down to 128-byte runs) where that gives the finish at
// least 16 row tiles to work on; 4 from 2^24 elements on, where longer runs matter
// more (500 x 134217 FP64 315 us with 8 lanes, 257 with 32; 512 x 8192 21 and 23),
// but for half storage, whose tiles have the most rows (6001 x 2999 FP16 35 us with
// 32 lanes, 40 with 64; 1000 x 16777 BF16 32 with 16, 49 with 64).
// 32 where 64 make
//  * between half a row tile and one per CU: then every tile is whole, in one
//    block, and needs no finish (50000 x 20 FP32 5 us against 17, 100000 x 64 BF16 13
//    and 33, 65536 x 256 FP32 32 and 34);
//  * between 2 and 3 1/4 per CU, of which two run at a time and the rest fill half
//    a round (200000 x 256 FP32 102 and 110, 100000 x 100 FP64 40 and 48).
// Tall matrices take several waves down a column, up to the whole block,
//  * where the block has more thread groups than the matrix keeps in columns, and
//    the tiles still cover the chip.  Half storage: while a group has at most four
//    columns (2^20 x 1 13.4 us with 64 lanes, 5.6 with 256; 10^6 x 10 26 and 17).
//    Others the whole block up to 10 columns (3 * 10^6 x 2 FP32 27 and 16, 10^6 x 6
//    15 and 13, x 10 22 and 21; x 20 39 and 40);
//  * where columns start at multiples of 16 KB, which share few cache sets: longer
//    runs, while two to eight tiles per CU are left (262144 x 64 FP64 72 us with 64
//    lanes, 59 with 256, 262144 x 256 289 and 239; 2^20 x 64 268 and 318).
// And a grid holds less than 2^32 threads: beyond, every thread has rows of its own.
constexpr int kRowsumMinLanes = 8, kRowsumMinTiles = 16, kRowsumLargeTiles = 4;
constexpr int64_t kRowsumLarge = int64_t(1) << 24;
inline int rowsum_lanes(int64_t n_rows, int64_t n_cols, int vec, int elem, int block) {
  int rl = 1;
  while (rl < 64 && (int64_t)rl * vec < n_rows) rl *= 2;
  const int64_t least = elem == 2 || n_rows * n_cols < kRowsumLarge ? kRowsumMinTiles : kRowsumLargeTiles;
  while (rl > kRowsumMinLanes && n_rows < least * rl * vec) rl /= 2;
  if (rl < 64) return rl;
  const int64_t cus = device_cus();
  auto tiles = [&](int lanes) { return (n_rows - 1) / ((int64_t)lanes * vec) + 1; };
  const bool same_sets = n_rows * elem % 16384 == 0;
  const int64_t t64 = tiles(rl);
  if (t64 > cus / 2 && t64 <= cus) return rl / 2;
  if (t64 > 2 * cus && 4 * t64 <= 13 * cus && n_cols >= 16 && !same_sets) return rl / 2;
  if (elem != 2 && n_cols <= 10 && 2 * tiles(block) > 3 * cus) return block;
  while (block % (2 * rl) == 0) {
    const int64_t t = tiles(2 * rl);
    const bool few = elem == 2 && n_cols <= 4 * (block / rl) && t > cus;
    if (!few && !(same_sets && t >= 2 * cus && t <= 8 * cus)) break;
    rl *= 2;
  }
  return tiles(rl) * block > 0xffffffffll ? block : rl;
}

// Row idx of the tile: the sum over groups of lds[g * rows + idx], in order.
template <class D>
__device__ __forceinline__ D sum_groups(const D* lds, int rows, int idx, int groups) {
  D t = lds[idx];
  for (int g = 1; g < groups; ++g) t += lds[g * rows + idx];
  return t;
}

template <class E, class O, int N, int EPT>
__global__ __launch_bounds__(kMaxBlock) void k_rowsum(E e, int64_t n_rows, int64_t n_cols, int split,
                                                    int rl,
                                                    typename wide<typename E::ct>::type* partials,
                                                    unsigned* counters, O* out) {
  using C = typename E::ct;
  using D = typename wide<C>::type;
  extern __shared__ __align__(16) unsigned char fx_dyn_lds[];
  D* lds = reinterpret_cast<D*>(fx_dyn_lds);
  // Where columns are no whole number of cache lines, vertically adjacent row
  // tiles share lines: the tiles of one chunk then run on one XCD (6001 x 2999
  // FP32 47 -> 43 us, FP64 88 -> 81; with aligned columns the plain order is
  // the faster, 8192 x 8192 FP64 234 against 251)
  uint32_t b = blockIdx.y * gridDim.x + blockIdx.x;
  if (n_rows * (int64_t)sizeof(typename E::storage) % 128) b = xcd_order(b, gridDim.x * gridDim.y);
  const int s = b / gridDim.x, tile = b % gridDim.x, t = threadIdx.x;
  const int rows = rl * N, S = blockDim.x / rl;  // rows per tile, columns per step
  const int lr = t % rl, g = t / rl;
  const int64_t row0 = (int64_t)tile * rows;
  const int64_t first = row0 + lr * N;
  const int sh = first + N > n_rows && first < n_rows ? (int)(first + N - n_rows) : 0;
  const int64_t r0 = first - sh;  // lanes below sh repeat rows of the vector before
  accum<C> acc[N];
  if (first < n_rows) {
    int64_t c = (int64_t)s * (EPT * S) + g;
    for (; c + (EPT - 1) * S < n_cols; c += (int64_t)split * (EPT * S)) {
      lanes<C, N> r[EPT];
      eval_tile<N, EPT>(e, r0 + c * n_rows, S * n_rows, r);
#pragma unroll
      for (int j = 0; j < N; ++j)  // row j's EPT columns, in column order
#pragma unroll
        for (int k = 0; k < EPT; ++k) acc[j].add(r[k].v[j]);
    }
    for (; c < n_cols; c += S) {  // (fewer than EPT of them)
      lanes<C, N> r = e.template at_vec<N, kNT>(r0 + c * n_rows);
#pragma unroll
      for (int j = 0; j < N; ++j) acc[j].add(r.v[j]);
    }
  }
  if (S == 1 && split == 1) {  // a row is one thread's
    if (first < n_rows)
#pragma unroll
      for (int j = 0; j < N; ++j)
        if (j >= sh) out[r0 + j] = static_cast<O>(acc[j].value());
    return;
  }
#pragma unroll
  for (int j = 0; j < N; ++j)  // [group][row]
    if (j >= sh) lds[t * N + j - sh] = acc[j].value();
  __syncthreads();
  for (int i = t; i < rows; i += blockDim.x) {
    if (row0 + i >= n_rows) break;
    const D v = sum_groups(lds, rows, i, S);
    if (split == 1) out[row0 + i] = static_cast<O>(v);
    else publish(partials + (int64_t)s * n_rows + row0 + i, v);
  }
  if (split == 1) return;
  if (take_last_ticket(counters + tile, split)) {
    // fl lanes side by side over rows; each of the F thread groups adds every
    // F-th chunk of its rows, then the groups' sums are added in order
    const int fl = rl > 64 ? rl : rows < 64 ? rows : 64, F = blockDim.x / fl, f = t / fl;
    D sum[N];
#pragma unroll
    for (int j = 0; j < N; ++j) sum[j] = 0;
    constexpr int U = N >= 8 ? 4 : 8;  // chunks in flight per row
    for (int q = f; q < split; q += U * F) {
      D v[U][N];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < N; ++j) {
          const int i = t % fl + fl * j;
          const bool in = i < rows && row0 + i < n_rows && q + u * F < split;
          v[u][j] = in ? partials[(int64_t)(q + u * F) * n_rows + row0 + i] : D(0);
        }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < N; ++j) sum[j] += v[u][j];
    }
    // (rows / fl <= N: rl * N rows, 64 or rl of them per step unless the whole
    // tile is smaller)
#pragma unroll
    for (int j = 0; j < N; ++j)
      if (t % fl + fl * j < rows) lds[f * rows + t % fl + fl * j] = sum[j];
    __syncthreads();
    for (int i = t; i < rows; i += blockDim.x)
      if (row0 + i < n_rows) out[row0 + i] = static_cast<O>(sum_groups(lds, rows, i, F));
    // (a loop of its own: beside the loads above it costs the whole kernel
    // registers, 8192 x 8192 BF16 152 us against 93)
    for (int i = t % fl; i < rows && row0 + i < n_rows; i += fl)
      for (int q = f; q < split; q += F) partials[(int64_t)q * n_rows + row0 + i] = D(0);
    if (t == 0) reset_counter(counters + tile);
  }
}

// Zero-fill (used for sums over empty dimensions; a kernel rather than a
// memset node, so the call can sit inside a captured graph).
template <class O>
__global__ __launch_bounds__(256) void k_fill_zero(O* out, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    out[i] = O(0);
}

// ============================================================================
// Host side: configuration resolution and dispatch.

template <int V> using ic = std::integral_constant<int, V>;

// Largest EPT compiled for an expression type (the run-time tape keeps one
// slot file per lane in registers and caps it lower).
template <class E> struct max_ept { static constexpr int value = 8; };
template <class E> struct max_ept<Fused<E>> { static constexpr int value = max_ept<E>::value; };

template <int MAX = 8, class F> inline int with_ept(int ept, F&& f) {
  switch (ept) {
    case 1: return f(ic<1>{});
    case 2: if constexpr (MAX >= 2) return f(ic<2>{}); break;
    case 4: if constexpr (MAX >= 4) return f(ic<4>{}); break;
    case 8: if constexpr (MAX >= 8) return f(ic<8>{}); break;
  }
  return fail(FX_E_UNSUPPORTED, "ept %d not compiled for this expression (max %d)", ept, MAX);
}

// Expression types compiled for 8-byte vectors as well (the run-time tape,
// whose launch the autotuner searches); the others take one element (any
// alignment) or 16 bytes.
template <class E> struct vec8_compiled { static constexpr bool value = false; };
template <class E> struct vec8_compiled<Fused<E>> { static constexpr bool value = vec8_compiled<E>::value; };
template <class E> constexpr bool vec8_compiled_v = vec8_compiled<E>::value;

// Expression types whose element-wise kernel is compiled with ordinary loads as
// well (kCachedLoadsUpTo).
template <class E> struct cached_loads { static constexpr bool value = true; };
template <class E> constexpr bool cached_loads_v = cached_loads<E>::value;

// Vector width in elements: one element, 8 bytes (where compiled) or 16 bytes.
template <class T, class E = void, class F> inline int with_vec(int vec_elems, F&& f) {
  constexpr int W = 16 / (int)sizeof(T);
  constexpr bool V8 = W >= 4 && vec8_compiled_v<E>;
  if (vec_elems == 1) return f(ic<1>{});
  if (vec_elems == W) return f(ic<W>{});
  if constexpr (V8) {
    if (vec_elems == W / 2) return f(ic<W / 2>{});
  }
  return fail(FX_E_UNSUPPORTED, "vector of %d elements not compiled (1 or %d%s)", vec_elems, W,
              V8 ? " or half of it" : "");
}

// The widest vector, up to 16 bytes, that a column of `rows` elements holds (one
// element or 16 bytes for expression types with their own evaluation).
template <class T, class E, int N = 16 / (int)sizeof(T), class F> inline int with_rows(int64_t rows, F&& f) {
  if (rows >= N) return f(ic<N>{});
  if constexpr (N > 1) return with_rows<T, E, vec8_compiled_v<E> ? 1 : N / 2>(rows, f);
  return f(ic<1>{});
}

// Resolve a configuration for `n_elems` elements of storage size `elem` with
// `n_leaves` distinct inputs.  kind: 0 element-wise, FX_R_* reductions;
// vectors: false where a column is shorter than a vector (one element then);
// funcs: divisions and function calls in the expression.
launch resolve(int kind, int elem, int64_t n_rows, int64_t n_cols, const fx_launch* cfg,
               bool vectors, int funcs = 0);

// Workspace layout: [counters, 256-byte aligned][FP64/u64 partials].
struct ws_layout {
  size_t counter_bytes = 0, partial_bytes = 0;
  size_t total() const { return counter_bytes + partial_bytes; }
};
ws_layout workspace_for(int kind, int64_t n_rows, int64_t n_cols, const launch& L, int elem, int vec);

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

template <class E> int check_expr(const E& e, int64_t* n_rows, int64_t* n_cols) {
  leaf_info li = info_of(e);
  if (!li.shape_ok) return fail(FX_E_SHAPE, "operands of the expression differ in shape");
  if (li.any_null) return fail(FX_E_ARG, "NULL input pointer");
  if (li.n_rows < 0 || li.n_cols < 0) return fail(FX_E_ARG, "negative dimension");
  *n_rows = li.n_rows;
  *n_cols = li.n_cols;
  return FX_OK;
}

// Storage bytes per element of the distinct arrays that e reads (diagonals, one
// element per column, not counted).
template <class E> int bytes_of(const E& e) { return info_of(e).bytes; }
template <class E> int bytes_of(const Fused<E>& f) {
  leaf_id ids[Fused<E>::L];
  int n = 0, b = info_of(f).bytes;
  f.e.leaf_ids(ids, n);
  for (int k = 0; k < Fused<E>::L; ++k)
    if (f.alias[k] != k) b -= (int)ids[k].size;
  return b;
}

// A defaulted EPT never exceeds what is compiled for the expression type.
template <class E> inline void clamp_ept(launch& L, const fx_launch* cfg) {
  if (!(cfg && cfg->ept)) L.ept = std::min(L.ept, max_ept<E>::value);
}

// Z = E element-wise (Sec. 3: assignment through the copy skeleton).
template <class E, class T>
int eval_direct(T* z, const E& e, const fx_launch* cfg, hipStream_t st);
template <class E, class T>
int eval(T* z, const E& e, const fx_launch* cfg, hipStream_t st) {
  if constexpr (leaves_of<E>::value >= 2 && leaves_of<E>::value <= kMaxFusedLeaves) {
    const auto f = fuse_leaves(e);
    if (f.has_alias()) return eval_direct(z, f, cfg, st);
  }
  return eval_direct(z, e, cfg, st);
}
template <class E, class T>
int eval_direct(T* z, const E& e, const fx_launch* cfg, hipStream_t st) {
  int64_t rows, cols;
  if (int rc = check_expr(e, &rows, &cols)) return rc;
  const int64_t n = rows * cols;
  if (n == 0) return FX_OK;
  if (!z) return fail(FX_E_ARG, "NULL output pointer");
  if (int rc = check_launch(cfg)) return rc;
  launch L = resolve(0, sizeof(T), rows, cols, cfg, true);
  clamp_ept<E>(L, cfg);
  const int vec = L.vec_bytes / (int)sizeof(T);
  return with_vec<T, E>(vec, [&](auto Nc) {
    return with_ept<max_ept<E>::value>(L.ept, [&](auto Ec) {
      constexpr int N = decltype(Nc)::value, EPT = decltype(Ec)::value;
      // (the policies are compiled for 16-byte vectors, the default where
      // they matter)
      if constexpr (N * sizeof(T) == 16) {
        if constexpr (kNT && cached_loads_v<E>) {
          if ((uint64_t)n * (sizeof(T) + bytes_of(e)) <= kCachedLoadsUpTo) {
            hipLaunchKernelGGL((k_ew<E, T, N, EPT, kNTS, false>), dim3(L.split), dim3(L.block), 0, st, e, z, n);
            return hip_check(hipGetLastError(), "k_ew launch");
          }
        }
        if (kNTS || (uint64_t)n * sizeof(T) > kStreamStoresAbove) {
          hipLaunchKernelGGL((k_ew<E, T, N, EPT, true>), dim3(L.split), dim3(L.block), 0, st, e, z, n);
          return hip_check(hipGetLastError(), "k_ew launch");
        }
      }
      hipLaunchKernelGGL((k_ew<E, T, N, EPT, kNTS>), dim3(L.split), dim3(L.block), 0, st, e, z, n);
      return hip_check(hipGetLastError(), "k_ew launch");
    });
  });
}

inline unsigned* ws_counters(void* ws) { return static_cast<unsigned*>(ws); }
template <class D> inline D* ws_partials(void* ws, const ws_layout& W) {
  return reinterpret_cast<D*>(static_cast<char*>(ws) + W.counter_bytes);
}

// out = finish(sum map(E)) as FP64 (u64 for u32 expressions).
template <class M, class E>
int reduce_full_direct(const E& e, void* out, void* ws, size_t ws_bytes, const fx_launch* cfg,
                       hipStream_t st);
template <class M, class E>
int reduce_full(const E& e, void* out, void* ws, size_t ws_bytes, const fx_launch* cfg,
                hipStream_t st) {
  if constexpr (leaves_of<E>::value >= 2 && leaves_of<E>::value <= kMaxFusedLeaves) {
    const auto f = fuse_leaves(e);
    if (f.has_alias()) return reduce_full_direct<M>(f, out, ws, ws_bytes, cfg, st);
  }
  return reduce_full_direct<M>(e, out, ws, ws_bytes, cfg, st);
}
template <class M, class E>
int reduce_full_direct(const E& e, void* out, void* ws, size_t ws_bytes, const fx_launch* cfg,
                       hipStream_t st) {
  using T = typename E::storage;
  using D = typename wide<typename E::ct>::type;
  int64_t rows, cols;
  if (int rc = check_expr(e, &rows, &cols)) return rc;
  if (!out) return fail(FX_E_ARG, "NULL output pointer");
  if (int rc = check_launch(cfg)) return rc;
  const int64_t n = rows * cols;
  launch L = resolve(FX_R_ACCU, sizeof(T), rows, cols, cfg, true, functions<E>::value);
  clamp_ept<E>(L, cfg);
  const int vec = L.vec_bytes / (int)sizeof(T);
  ws_layout W = workspace_for(FX_R_ACCU, rows, cols, L, sizeof(T), vec);
  if (W.total() > 0 && (!ws || ws_bytes < W.total()))
    return fail(FX_E_WORKSPACE, "workspace of %zu bytes needed, %zu given", W.total(), ws_bytes);
  return with_vec<T, E>(vec, [&](auto Nc) {
    return with_ept<max_ept<E>::value>(L.ept, [&](auto Ec) {
      constexpr int N = decltype(Nc)::value, EPT = decltype(Ec)::value;
      hipLaunchKernelGGL((k_full<E, M, D, N, EPT>), dim3(L.split), dim3(L.block), 0, st, e, n,
                         ws ? ws_partials<D>(ws, W) : nullptr, ws ? ws_counters(ws) : nullptr,
                         static_cast<D*>(out));
      return hip_check(hipGetLastError(), "k_full launch");
    });
  });
}

// sum(E, 0) or sum(E, 1) into out (accumulator dtype O).
template <class O, class E>
int reduce_dim_direct(int kind, const E& e, O* out, void* ws, size_t ws_bytes,
                      const fx_launch* cfg, hipStream_t st);
template <class O, class E>
int reduce_dim(int kind, const E& e, O* out, void* ws, size_t ws_bytes, const fx_launch* cfg,
               hipStream_t st) {
  if constexpr (leaves_of<E>::value >= 2 && leaves_of<E>::value <= kMaxFusedLeaves) {
    const auto f = fuse_leaves(e);
    if (f.has_alias()) return reduce_dim_direct(kind, f, out, ws, ws_bytes, cfg, st);
  }
  return reduce_dim_direct(kind, e, out, ws, ws_bytes, cfg, st);
}
template <class O, class E>
int reduce_dim_direct(int kind, const E& e, O* out, void* ws, size_t ws_bytes,
                      const fx_launch* cfg, hipStream_t st) {
  using T = typename E::storage;
  using D = typename wide<typename E::ct>::type;
  int64_t rows, cols;
  if (int rc = check_expr(e, &rows, &cols)) return rc;
  if (int rc = check_launch(cfg)) return rc;
  const int64_t nout = kind == FX_R_COLSUM ? cols : rows;
  if (nout == 0) return FX_OK;
  if (!out) return fail(FX_E_ARG, "NULL output pointer");
  if (rows * cols == 0) {
    const int grid = (int)std::min<int64_t>(ceil_div(nout, 256), 1024);
    hipLaunchKernelGGL((k_fill_zero<O>), dim3(grid), dim3(256), 0, st, out, nout);
    return hip_check(hipGetLastError(), "k_fill_zero launch");
  }
  const int W16 = 16 / (int)sizeof(T);
  launch L = resolve(kind, sizeof(T), rows, cols, cfg, rows >= W16, functions<E>::value);
  clamp_ept<E>(L, cfg);
  const int vec = L.vec_bytes / (int)sizeof(T);
  ws_layout W = workspace_for(kind, rows, cols, L, sizeof(T), vec);
  if (W.total() > 0 && (!ws || ws_bytes < W.total()))
    return fail(FX_E_WORKSPACE, "workspace of %zu bytes needed, %zu given", W.total(), ws_bytes);
  D* parts = ws ? ws_partials<D>(ws, W) : nullptr;
  unsigned* ctr = ws ? ws_counters(ws) : nullptr;
  if (kind == FX_R_COLSUM) {
    if (L.split == 0) {  // thin columns: one thread per column
      const int grid = (int)std::min<int64_t>(ceil_div(cols, L.block), 1 << 20);
      return with_rows<T, E>(rows, [&](auto Nc) {
        hipLaunchKernelGGL((k_colsum_thin<E, O, decltype(Nc)::value>), dim3(grid), dim3(L.block), 0, st, e,
                           rows, cols, out);
        return hip_check(hipGetLastError(), "k_colsum_thin launch");
      });
    }
    const int64_t rpc = ceil_div(ceil_div(rows, L.split), vec) * vec;
    return with_vec<T, E>(vec, [&](auto Nc) {
      return with_ept<max_ept<E>::value>(L.ept, [&](auto Ec) {
        constexpr int N = decltype(Nc)::value, EPT = decltype(Ec)::value;
        hipLaunchKernelGGL((k_colsum<E, O, N, EPT>), dim3((unsigned)cols, L.split), dim3(L.block), 0,
                           st, e, rows, L.split, rpc, parts, ctr, out);
        return hip_check(hipGetLastError(), "k_colsum launch");
      });
    });
  }
  const int rl = rowsum_lanes(rows, cols, vec, sizeof(T), L.block);
  const int64_t rblocks = ceil_div(rows, (int64_t)rl * vec);
  return with_vec<T, E>(vec, [&](auto Nc) {
    return with_ept<max_ept<E>::value>(L.ept, [&](auto Ec) {
      constexpr int N = decltype(Nc)::value, EPT = decltype(Ec)::value;
      hipLaunchKernelGGL((k_rowsum<E, O, N, EPT>), dim3((unsigned)rblocks, L.split), dim3(L.block),
                         sizeof(D) * L.block * N, st, e, rows, cols, L.split, rl, parts, ctr, out);
      return hip_check(hipGetLastError(), "k_rowsum launch");
    });
  });
}

// ---- dtype dispatch shared by the C entry points -------------------------

template <class T> struct tag { using type = T; };

// Floating-point storage dtypes.
template <class F> int with_fp(fx_dtype dt, F&& f) {
  switch (dt) {
    case FX_F32: return f(tag<float>{});
    case FX_F64: return f(tag<double>{});
    case FX_BF16: return f(tag<bf16_t>{});
    case FX_F16: return f(tag<f16_t>{});
    default: break;
  }
  return fail(FX_E_DTYPE, "dtype %d not supported here (floating point only)", (int)dt);
}

template <class T> using acc_out_t = std::conditional_t<std::is_same_v<T, double>, double, float>;

inline hipStream_t S(void* s) { return static_cast<hipStream_t>(s); }

inline int check_n(int64_t n) { return n < 0 ? fail(FX_E_ARG, "negative size %lld", (long long)n) : FX_OK; }
inline int check_shape(fx_shape s) {
  return (s.n_rows < 0 || s.n_cols < 0) ? fail(FX_E_ARG, "negative dimension") : FX_OK;
}

}  // namespace fx

// Strided views: submatrix, transpose and diagonal leaves (Sec. 3 builds
// the element access of a transposed matrix by swapping row and column in
// the index; Sec. 4 uses the centre submatrix with half the rows and
// columns, and diagonals).
//
//   Sub<T>    element (r, c) = p[off + r + c * ld]      (submatrix)
//   Trans<T>  element (r, c) = p[off + c + r * ld]      (transposed matrix)
//   Diag<T>   element (r, 0) = p[off + r * stride]      (diagonal, a vector)
//
// t(E) moves a transpose down to the leaves at compile time:
// (B + C).t() is B.t() + C.t(), and a double transpose cancels.
//
// Evaluation.  A diagonal is a vector, so expressions over diagonals run
// through the linear skeletons.  Expressions with Sub or Trans leaves run
// through k_ew2d: one block per output tile, each thread a vector of N
// consecutive rows in several columns.  Dense and submatrix leaves are
// read straight from HBM, 16-byte vectors at any element; a part of the
// expression all of whose leaves are transposed, such as t(B + C), is first
// evaluated over its source tile and staged in LDS by the whole block, read
// along the source's columns and written at an odd column pitch (so the
// strided LDS writes do not conflict); the threads then read their transposed
// vectors from LDS.
#pragma once

#include "fx_kernels.hpp"

namespace fx {

// ---- view leaves -------------------------------------------------------------

template <class T> struct Sub : expr_tag {
  using storage = T;
  using ct = ct_t<T>;
  const T* p;
  int64_t off, ld, n_rows, n_cols;
  __device__ __forceinline__ ct at(int64_t i) const {  // linear access (not on the fast path)
    const int64_t r = i % n_rows, c = i / n_rows;
    return static_cast<ct>(p[off + r + c * ld]);
  }
  template <int N, bool NT>
  __device__ __forceinline__ lanes<ct, N> at_vec(int64_t i) const {
    lanes<ct, N> x;
#pragma unroll
    for (int j = 0; j < N; ++j) x.v[j] = at(i + j);
    return x;
  }
  void collect(leaf_info& li) const {
    if (!p && n_rows * n_cols > 0) li.any_null = true;
    li.add_shape(n_rows, n_cols);
  }
  static constexpr int kLeaves = 0;  // not de-duplicated
  template <int OFF, int N, bool NT, class R>
  __device__ __forceinline__ void gather(R*, const uint8_t*, int64_t) const {}
  template <int OFF, int N, bool NT, class R>
  __device__ __forceinline__ lanes<ct, N> at_regs(const R*, int64_t i) const {
    return at_vec<N, NT>(i);
  }
  void leaf_ids(leaf_id*, int&) const {}
};

template <class T> struct Trans : expr_tag {
  using storage = T;
  using ct = ct_t<T>;
  const T* p;
  int64_t off, ld, n_rows, n_cols;
  __device__ __forceinline__ ct at(int64_t i) const {  // linear access (not on the fast path)
    const int64_t r = i % n_rows, c = i / n_rows;
    return static_cast<ct>(p[off + c + r * ld]);
  }
  template <int N, bool NT>
  __device__ __forceinline__ lanes<ct, N> at_vec(int64_t i) const {
    lanes<ct, N> x;
#pragma unroll
    for (int j = 0; j < N; ++j) x.v[j] = at(i + j);
    return x;
  }
  void collect(leaf_info& li) const {
    if (!p && n_rows * n_cols > 0) li.any_null = true;
    li.add_shape(n_rows, n_cols);
  }
  static constexpr int kLeaves = 0;
  template <int OFF, int N, bool NT, class R>
  __device__ __forceinline__ void gather(R*, const uint8_t*, int64_t) const {}
  template <int OFF, int N, bool NT, class R>
  __device__ __forceinline__ lanes<ct, N> at_regs(const R*, int64_t i) const {
    return at_vec<N, NT>(i);
  }
  void leaf_ids(leaf_id*, int&) const {}
};

template <class T> struct Diag : expr_tag {
  using storage = T;
  using ct = ct_t<T>;
  const T* p;
  int64_t off, stride, n_rows;
  static constexpr int64_t n_cols = 1;
  __device__ __forceinline__ ct at(int64_t i) const {
    return static_cast<ct>(p[off + i * stride]);
  }
  template <int N, bool NT>
  __device__ __forceinline__ lanes<ct, N> at_vec(int64_t i) const {
    lanes<ct, N> x;
#pragma unroll
    for (int j = 0; j < N; ++j) x.v[j] = at(i + j);
    return x;
  }
  void collect(leaf_info& li) const {
    if (!p && n_rows > 0) li.any_null = true;
    li.add_shape(n_rows, 1);
  }
  static constexpr int kLeaves = 0;
  template <int OFF, int N, bool NT, class R>
  __device__ __forceinline__ void gather(R*, const uint8_t*, int64_t) const {}
  template <int OFF, int N, bool NT, class R>
  __device__ __forceinline__ lanes<ct, N> at_regs(const R*, int64_t i) const {
    return at_vec<N, NT>(i);
  }
  void leaf_ids(leaf_id*, int&) const {}
};

// ---- front end ----------------------------------------------------------------

// submat(X, r0, c0, rows, cols): rows x cols block of X from (r0, c0).
template <class T> inline Sub<T> submat(const Leaf<T>& x, int64_t r0, int64_t c0, int64_t rows,
                                        int64_t cols) {
  Sub<T> s;
  s.p = x.p;
  s.off = r0 + c0 * x.n_rows;
  s.ld = x.n_rows;
  s.n_rows = rows;
  s.n_cols = cols;
  return s;
}
// diag(X, k): diagonal k of X (k > 0 above the main diagonal) as a column.
template <class T> inline Diag<T> diag(const Leaf<T>& x, int64_t k) {
  Diag<T> d;
  d.p = x.p;
  d.off = (k < 0 ? -k : 0) + (k > 0 ? k : 0) * x.n_rows;
  d.stride = x.n_rows + 1;
  d.n_rows = std::max<int64_t>(0, k >= 0 ? std::min(x.n_rows, x.n_cols - k)
                                         : std::min(x.n_rows + k, x.n_cols));
  return d;
}

// Is a leaf range inside its matrix?  (Host check for submat / diag.)
template <class T> inline bool view_inside(const Leaf<T>& x, int64_t r0, int64_t c0,
                                           int64_t rows, int64_t cols) {
  return r0 >= 0 && c0 >= 0 && rows >= 0 && cols >= 0 && r0 + rows <= x.n_rows &&
         c0 + cols <= x.n_cols;
}

template <class T> inline Trans<T> t(const Leaf<T>& x) {
  Trans<T> r;
  r.p = x.p;
  r.off = 0;
  r.ld = x.n_rows;
  r.n_rows = x.n_cols;
  r.n_cols = x.n_rows;
  return r;
}
template <class T> inline Trans<T> t(const Sub<T>& x) {
  Trans<T> r;
  r.p = x.p;
  r.off = x.off;
  r.ld = x.ld;
  r.n_rows = x.n_cols;
  r.n_cols = x.n_rows;
  return r;
}
template <class T> inline Sub<T> t(const Trans<T>& x) {
  Sub<T> r;
  r.p = x.p;
  r.off = x.off;
  r.ld = x.ld;
  r.n_rows = x.n_cols;
  r.n_cols = x.n_rows;
  return r;
}
template <class Op, class A> inline auto t(const Unary<Op, A>& u) {
  auto a = t(u.a);
  return Unary<Op, decltype(a)>{{}, a};
}
template <class Op, class A, class B> inline auto t(const Binary<Op, A, B>& b) {
  auto x = t(b.a);
  auto y = t(b.b);
  return Binary<Op, decltype(x), decltype(y)>{{}, x, y};
}
template <class Op, class A, bool LEFT> inline auto t(const Scalar<Op, A, LEFT>& s) {
  auto a = t(s.a);
  Scalar<Op, decltype(a), LEFT> r{{}, a, s.k};
  r.aux = s.aux;
  r.mode = s.mode;
  return r;
}
template <class To, class A> inline auto t(const Convert<To, A>& cv) {
  auto a = t(cv.a);
  return Convert<To, decltype(a)>{{}, a};
}
template <class T> inline auto t(const dmat<T>& m) { return t(m.expr()); }

// ---- traits -------------------------------------------------------------------

// Is every leaf transposed (and there is one)?  Such a part of the expression
// is staged as one LDS tile.
template <class E> struct all_trans { static constexpr bool value = false; };
template <class T> struct all_trans<Trans<T>> { static constexpr bool value = true; };
template <class Op, class A> struct all_trans<Unary<Op, A>> : all_trans<A> {};
template <class Op, class A, bool L> struct all_trans<Scalar<Op, A, L>> : all_trans<A> {};
template <class Op, class A, class B> struct all_trans<Binary<Op, A, B>> {
  static constexpr bool value = all_trans<A>::value && all_trans<B>::value;
};

// Number of LDS tiles (the largest all-transposed parts), and whether the
// expression needs the 2-D skeleton.
template <class E, bool WHOLE = all_trans<E>::value> struct trans_count { static constexpr int value = 0; };
template <class E> struct trans_count<E, true> { static constexpr int value = 1; };
template <class Op, class A> struct trans_count<Unary<Op, A>, false> : trans_count<A> {};
template <class Op, class A, bool L> struct trans_count<Scalar<Op, A, L>, false> : trans_count<A> {};
template <class To, class A> struct trans_count<Convert<To, A>, false> : trans_count<A> {};
template <class Op, class A, class B> struct trans_count<Binary<Op, A, B>, false> {
  static constexpr int value = trans_count<A>::value + trans_count<B>::value;
};

template <class E> struct needs_2d { static constexpr bool value = false; };
template <class T> struct needs_2d<Sub<T>> { static constexpr bool value = true; };
template <class T> struct needs_2d<Trans<T>> { static constexpr bool value = true; };
template <class Op, class A> struct needs_2d<Unary<Op, A>> : needs_2d<A> {};
template <class Op, class A, bool L> struct needs_2d<Scalar<Op, A, L>> : needs_2d<A> {};
template <class To, class A> struct needs_2d<Convert<To, A>> : needs_2d<A> {};
template <class Op, class A, class B> struct needs_2d<Binary<Op, A, B>> {
  static constexpr bool value = needs_2d<A>::value || needs_2d<B>::value;
};

// ---- 2-D evaluation -------------------------------------------------------------

constexpr int kTileThreads = 256;

// Tile geometry.  With transposed parts (KT > 0) the tile is 128 rows (64 of
// 8-byte types), so that a column of a direct leaf is read in 512-byte runs
// (256 of 2-byte types), by 32 columns (Q = 1; 17 KB of LDS per staged part) or
// 64 (Q = 4 and 2-byte types; 33 KB).  The wider tile is the faster one where
// columns start at multiples of 16 KB and its blocks are many (4096 x 4096
// FP64 a*A + t(B + C) + log(D^2): 126 us against 142; 8192 x 8192 FP32 245
// and 247), the narrow one elsewhere (5856 x 5856 FP64 248 against 254, 10000 x
// 10000 FP64 716 and 730; with few blocks the wide ones fill the chip unevenly,
// 3001 x 3001 FP32 30 and 44).  Without transposed parts the tile is (64 N) x
// (4 Q): 1 KB runs (square tiles, 256-byte runs: measured slower), Q columns per
// thread.
//
// One element per thread row (N = 1; tiles of 16 x 64, 64 x 16 without
// transposed parts) is for small results and for short columns.  Up to 4 MB of
// a result with transposed parts the tiles of vectors are too few to cover their
// own latency (FP32 512 x 512: 2*(t(X) + Y) + 2*(X + t(Y)) 3.1 us against 5.4 in
// paired tiles, 1024 x 1024 4.3 and 5.8, 1500 x 1500 9.4 and 7.6; BF16 expr2 1001
// x 1001 4.6 and 8.1, 2000 x 2000 11.4 and 10.7).  Without them, columns of up
// to 32 rows leave most of a 64 N row tile idle (sum of two submatrices of 4 x
// 131072 FP32: 7.9 us against 12.6, 16 x 32768: 3.7 and 4.8, 64 x 8192: 2.8 and
// 2.9).
constexpr uint64_t kElementBelow = uint64_t(4) << 20;
constexpr int kElementRows = 32;
template <int KT, int N, int Q, class T> struct tile_geo {
  static constexpr int TR = KT == 0 ? 64 * N : N == 1 ? 16 : sizeof(T) == 8 ? 64 : 128;
  static constexpr int TC = KT == 0 ? 4 * Q : N == 1 || Q == 4 || sizeof(T) == 2 ? 64 : 32;
  static constexpr int RV = TR / N;              // threads down a column
  static constexpr int CG = kTileThreads / RV;   // columns at a time
  static constexpr int P = TR + 1;               // LDS column pitch
};
// The wide tile (Q = 4) is compiled where two of its blocks, at least, share a
// CU's 160 KB of LDS: for at most two staged parts of 4- or 8-byte types.  More
// parts take the narrow one, whose LDS is half (five parts 83 KB, nine 149).
template <int KT, int N, class T> constexpr bool wide_tile() {
  using G = tile_geo<KT, N, 4, T>;
  return KT == 0 || 2 * (N + KT * G::TC * G::P) * sizeof(ct_t<T>) <= 160 * 1024;
}

// The tile being computed (G: its geometry; NTL: streaming loads of the direct
// leaves).
template <class C, class G, bool NTL> struct tile_ctx {
  static constexpr bool nt = NTL;
  C* lds;
  int64_t r0, c0;
};

// Cache policy of the direct leaves, by the bytes of the distinct arrays and the
// output, and by where the columns start.  Ordinary loads leave the data in the
// last-level cache for the next call on them, and serve the second read of a line
// that two runs straddle; streaming loads leave that cache to the output.  us
// with streaming against ordinary loads, on inputs that change from call to call
// (repeated):
//  * with transposed parts and columns of whole cache lines, streaming from 176
//    MiB on (FP32 3040 x 3040 expr2, 176 MiB: 40.3, 41.1 (31.5, 28.4); 4096 x 4096,
//    320 MiB: 52, 67 repeated), in paired tiles, which read an array once, from
//    104 MiB (3040 x 3040 expr1, 106 MiB: 23.4, 28.5 (22.9, 20.2); 4096 x 4096 40.2,
//    47.1 (39.2, 32.2));
//  * with columns that are no whole lines, ordinary ones at any size, for the lines
//    read by two tiles (FP32 7000 x 7000 expr1 171, 149; FP64 5000 x 5000 153, 134;
//    FP32 10000 x 10000 expr1 267, 250 repeated);
//  * submatrices, whose runs are long: streaming from 176 MiB with whole lines
//    (FP32 8192 x 8192 "2", a sum of two, 192 MiB: 33, 37 repeated), from twice
//    that without (10000 x 10000 "2", 286 MiB: 50.4, 46.7 repeated; "4", 477 MiB:
//    92, 100).  Up to there what ordinary loads win on repeated inputs they lose on
//    new ones (FP64 4096 x 4096 "2" 18.0, 21.6 (17.1, 15.6));
//  * submatrices whose columns start at multiples of 16 KB, which share a few sets
//    of the caches, stream as well between the 32 MB of the eight L2 caches and 64
//    MiB (FP32 4096 x 4096 "2": 12.7, 13.8 (9.4, 10.7); 16384 x 1000 8.0, 8.6
//    repeated).
constexpr uint64_t kMiB = uint64_t(1) << 20;
constexpr uint64_t kStreamFrom = 176 * kMiB, kStreamPairsFrom = 104 * kMiB, kSetsFrom = 32 * kMiB,
                   kSetsTo = 64 * kMiB;
constexpr int kSetsPitch = 16384;

// Is every column pitch of e a multiple of `bytes`?
template <class T> inline bool pitch_of(const Leaf<T>& e, int bytes) { return e.n_rows * sizeof(T) % bytes == 0; }
template <class T> inline bool pitch_of(const Sub<T>& e, int bytes) { return e.ld * sizeof(T) % bytes == 0; }
template <class T> inline bool pitch_of(const Trans<T>& e, int bytes) { return e.ld * sizeof(T) % bytes == 0; }
template <class T> inline bool pitch_of(const Diag<T>&, int) { return true; }
template <class Op, class A> inline bool pitch_of(const Unary<Op, A>& e, int bytes) { return pitch_of(e.a, bytes); }
template <class Op, class A, bool L> inline bool pitch_of(const Scalar<Op, A, L>& e, int bytes) {
  return pitch_of(e.a, bytes);
}
template <class To, class A> inline bool pitch_of(const Convert<To, A>& e, int bytes) {
  return pitch_of(e.a, bytes);
}
template <class Op, class A, class B> inline bool pitch_of(const Binary<Op, A, B>& e, int bytes) {
  return pitch_of(e.a, bytes) && pitch_of(e.b, bytes);
}

// Storage bytes per element of the result that e reads, each array once.
struct view_arrays {
  const void* p[16];
  int n = 0, bytes = 0;
  void add(const void* q, int elem) {
    for (int i = 0; i < n; ++i)
      if (p[i] == q) return;
    if (n < 16) p[n++] = q;
    bytes += elem;
  }
};
template <class T> inline void arrays_in(const Leaf<T>& e, view_arrays& v) { v.add(e.p, sizeof(T)); }
template <class T> inline void arrays_in(const Sub<T>& e, view_arrays& v) { v.add(e.p, sizeof(T)); }
template <class T> inline void arrays_in(const Trans<T>& e, view_arrays& v) { v.add(e.p, sizeof(T)); }
template <class T> inline void arrays_in(const Diag<T>&, view_arrays&) {}
template <class Op, class A> inline void arrays_in(const Unary<Op, A>& e, view_arrays& v) { arrays_in(e.a, v); }
template <class Op, class A, bool L> inline void arrays_in(const Scalar<Op, A, L>& e, view_arrays& v) {
  arrays_in(e.a, v);
}
template <class To, class A> inline void arrays_in(const Convert<To, A>& e, view_arrays& v) { arrays_in(e.a, v); }
template <class Op, class A, class B> inline void arrays_in(const Binary<Op, A, B>& e, view_arrays& v) {
  arrays_in(e.a, v);
  arrays_in(e.b, v);
}

// src2<N>(e, r, c): an all-transposed expression at row r, columns c .. c+N-1
// of the view: N consecutive rows of every source.  Ordinary (not streaming)
// loads: where the leading dimension is no whole number of cache lines, the
// lines a run straddles are read again by the tile beside it, long after, and
// must stay in the last-level cache until then (10000 x 10000 FP32 a*A +
// t(B + C) + log(D^2): 419 us with streaming loads and 64 x 64 tiles staged
// leaf by leaf, 378 now).
template <int N, class T>
__device__ __forceinline__ lanes<ct_t<T>, N> src2(const Trans<T>& e, int64_t r, int64_t c) {
  return load_lanes<N, false>(e.p, e.off + c + r * e.ld);
}
template <int N, class Op, class A>
__device__ __forceinline__ lanes<typename A::ct, N> src2(const Unary<Op, A>& e, int64_t r, int64_t c) {
  lanes<typename A::ct, N> v = src2<N>(e.a, r, c);
  apply_lanes<Op, mod_none>(v.v);
  return v;
}
template <int N, class Op, class A, bool L>
__device__ __forceinline__ lanes<typename A::ct, N> src2(const Scalar<Op, A, L>& e, int64_t r, int64_t c) {
  lanes<typename A::ct, N> v = src2<N>(e.a, r, c);
#pragma unroll
  for (int j = 0; j < N; ++j) v.v[j] = e.apply1(v.v[j]);
  return v;
}
template <int N, class Op, class A, class B>
__device__ __forceinline__ lanes<typename A::ct, N> src2(const Binary<Op, A, B>& e, int64_t r, int64_t c) {
  lanes<typename A::ct, N> u = src2<N>(e.a, r, c);
  lanes<typename A::ct, N> w = src2<N>(e.b, r, c);
#pragma unroll
  for (int j = 0; j < N; ++j) u.v[j] = Op::apply(u.v[j], w.v[j]);
  return u;
}

// at2<TOFF, N>(e, r, c, x): rows r..r+N-1 of column c.  TOFF numbers the
// all-transposed parts depth-first (their LDS tiles).
template <int TOFF, int N, class T, class X>
__device__ __forceinline__ lanes<ct_t<T>, N> at2(const Leaf<T>& e, int64_t r, int64_t c, const X&) {
  return load_lanes<N, kNT && X::nt>(e.p, r + c * e.n_rows);
}
template <int TOFF, int N, class T, class X>
__device__ __forceinline__ lanes<ct_t<T>, N> at2(const Sub<T>& e, int64_t r, int64_t c, const X&) {
  return load_lanes<N, kNT && X::nt>(e.p, e.off + r + c * e.ld);
}
template <int TOFF, int N, class T, class X>
__device__ __forceinline__ lanes<ct_t<T>, N> at2(const Diag<T>& e, int64_t r, int64_t, const X&) {
  return e.template at_vec<N, kNT>(r);
}
template <int TOFF, int N, class C, class G, bool NTL>
__device__ __forceinline__ lanes<C, N> staged(int64_t r, int64_t c, const tile_ctx<C, G, NTL>& x) {
  const C* buf = x.lds + TOFF * (G::TC * G::P) + (int)(c - x.c0) * G::P + (int)(r - x.r0);
  lanes<C, N> v;
#pragma unroll
  for (int j = 0; j < N; ++j) v.v[j] = buf[j];
  return v;
}
template <int TOFF, int N, class T, class X>
__device__ __forceinline__ lanes<ct_t<T>, N> at2(const Trans<T>&, int64_t r, int64_t c, const X& x) {
  return staged<TOFF, N>(r, c, x);
}
template <int TOFF, int N, class Op, class A, class X>
__device__ __forceinline__ lanes<typename A::ct, N> at2(const Unary<Op, A>& e, int64_t r, int64_t c,
                                                        const X& x) {
  if constexpr (all_trans<A>::value) {
    return staged<TOFF, N>(r, c, x);
  } else {
    lanes<typename A::ct, N> v = at2<TOFF, N>(e.a, r, c, x);
    apply_lanes<Op, mod_none>(v.v);
    return v;
  }
}
template <int TOFF, int N, class Op, class A, bool L, class X>
__device__ __forceinline__ lanes<typename A::ct, N> at2(const Scalar<Op, A, L>& e, int64_t r,
                                                        int64_t c, const X& x) {
  if constexpr (all_trans<A>::value) {
    return staged<TOFF, N>(r, c, x);
  } else {
    lanes<typename A::ct, N> v = at2<TOFF, N>(e.a, r, c, x);
#pragma unroll
    for (int j = 0; j < N; ++j) v.v[j] = e.apply1(v.v[j]);
    return v;
  }
}
template <int TOFF, int N, class Op, class A, class B, class X>
__device__ __forceinline__ lanes<typename A::ct, N> at2(const Binary<Op, A, B>& e, int64_t r,
                                                        int64_t c, const X& x) {
  if constexpr (all_trans<Binary<Op, A, B>>::value) {
    return staged<TOFF, N>(r, c, x);
  } else {
    lanes<typename A::ct, N> u = at2<TOFF, N>(e.a, r, c, x);
    lanes<typename A::ct, N> w = at2<TOFF + trans_count<A>::value, N>(e.b, r, c, x);
#pragma unroll
    for (int j = 0; j < N; ++j) u.v[j] = Op::apply(u.v[j], w.v[j]);
    return u;
  }
}
template <int TOFF, int N, class To, class A, class X>
__device__ __forceinline__ lanes<To, N> at2(const Convert<To, A>& e, int64_t r, int64_t c, const X& x) {
  static_assert(trans_count<A>::value == 0, "a transposed leaf below conv_to is not staged");
  lanes<typename A::ct, N> v = at2<0, N>(e.a, r, c, x);
  lanes<To, N> o;
#pragma unroll
  for (int j = 0; j < N; ++j) o.v[j] = static_cast<To>(v.v[j]);
  return o;
}

// stage<TOFF, N>: every all-transposed part is evaluated over its source tile
// into LDS.  Consecutive threads take consecutive view columns, which are
// consecutive source rows; all of a thread's loads are issued before the first
// LDS write.  Vectors past the view's last column are moved back to end with
// it (the repeated columns are written twice, alike), rows past its last
// repeat that row into LDS rows nothing reads.
template <int TOFF, int N, class E, class C, class G, bool NTL>
__device__ __forceinline__ void stage(const E& e, const tile_ctx<C, G, NTL>& x, int64_t rows, int64_t cols) {
  if constexpr (all_trans<E>::value) {
    C* buf = x.lds + TOFF * (G::TC * G::P);
    constexpr int CV = G::TC / N, PER = G::TR * CV / kTileThreads;
    lanes<C, N> v[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int idx = threadIdx.x + k * kTileThreads;
      v[k] = src2<N>(e, min(x.r0 + idx / CV, rows - 1), min(x.c0 + (idx % CV) * N, cols - N));
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int idx = threadIdx.x + k * kTileThreads;
      const int cl = (int)(min(x.c0 + (idx % CV) * N, cols - N) - x.c0);
#pragma unroll
      for (int j = 0; j < N; ++j)
        if (cl + j >= 0) buf[(cl + j) * G::P + idx / CV] = v[k].v[j];
    }
  }
}
template <int TOFF, int N, class Op, class A, class X>
__device__ __forceinline__ void stage_parts(const Unary<Op, A>& e, const X& x, int64_t rows, int64_t cols);
template <int TOFF, int N, class Op, class A, bool L, class X>
__device__ __forceinline__ void stage_parts(const Scalar<Op, A, L>& e, const X& x, int64_t rows, int64_t cols);
template <int TOFF, int N, class Op, class A, class B, class X>
__device__ __forceinline__ void stage_parts(const Binary<Op, A, B>& e, const X& x, int64_t rows, int64_t cols);
template <int TOFF, int N, class E, class X>
__device__ __forceinline__ void stage_parts(const E& e, const X& x, int64_t rows, int64_t cols) {
  stage<TOFF, N>(e, x, rows, cols);  // a leaf
}
template <int TOFF, int N, class Op, class A, class X>
__device__ __forceinline__ void stage_parts(const Unary<Op, A>& e, const X& x, int64_t rows, int64_t cols) {
  if constexpr (all_trans<A>::value) stage<TOFF, N>(e, x, rows, cols);
  else stage_parts<TOFF, N>(e.a, x, rows, cols);
}
template <int TOFF, int N, class Op, class A, bool L, class X>
__device__ __forceinline__ void stage_parts(const Scalar<Op, A, L>& e, const X& x, int64_t rows,
                                            int64_t cols) {
  if constexpr (all_trans<A>::value) stage<TOFF, N>(e, x, rows, cols);
  else stage_parts<TOFF, N>(e.a, x, rows, cols);
}
template <int TOFF, int N, class Op, class A, class B, class X>
__device__ __forceinline__ void stage_parts(const Binary<Op, A, B>& e, const X& x, int64_t rows,
                                            int64_t cols) {
  if constexpr (all_trans<Binary<Op, A, B>>::value) {
    stage<TOFF, N>(e, x, rows, cols);
  } else {
    stage_parts<TOFF, N>(e.a, x, rows, cols);
    stage_parts<TOFF + trans_count<A>::value, N>(e.b, x, rows, cols);
  }
}

// Z (dense rows x cols) = E over a grid of tiles, numbered down the tile
// columns (tile t: tile row t % tile_rows, tile column t / tile_rows) and
// taken in xcd_order.  (Launching the partner tiles (I, J) and (J, I) side
// by side, to find a transposed operand's tile in the last-level cache,
// measured slower on the 10k x 10k expressions.)  N > 1 needs rows and cols of
// at least N.
template <class E, class T, int N, int Q, bool NTL, bool NTS>
__global__ __launch_bounds__(kTileThreads) void k_ew2d(E e, T* __restrict__ z, int64_t rows,
                                                      int64_t cols, uint32_t tile_rows) {
  using C = typename E::ct;
  constexpr int KT = trans_count<E>::value;
  using G = tile_geo<KT, N, Q, T>;
  // N values ahead: the last vector of a tile of fewer than N rows starts above it
  __shared__ C lds[KT > 0 ? N + KT * G::TC * G::P : 1];
  const uint32_t t = xcd_order(blockIdx.x, gridDim.x);
  const tile_ctx<C, G, NTL> x{lds + (KT > 0 ? N : 0), (int64_t)(t % tile_rows) * G::TR, (int64_t)(t / tile_rows) * G::TC};
  if constexpr (KT > 0) {
    stage_parts<0, N>(e, x, rows, cols);
    __syncthreads();
  }
  const int rv = threadIdx.x % G::RV, cg = threadIdx.x / G::RV;
  const int64_t first = x.r0 + rv * N;
  if (first >= rows) return;
  // the last rows, where they are no whole vector, are computed as one that
  // ends with the column; its first `sh` rows are another thread's, and are not
  // stored (the output may be an input read in place)
  const int sh = first + N > rows ? (int)(first + N - rows) : 0;
  const int64_t r = first - sh;
  // U columns at a time: all their loads, then their stores (columns past the
  // last repeat it and are not stored)
  constexpr int QT = G::TC / G::CG, U = QT < 4 ? QT : 4;
#pragma unroll
  for (int q = 0; q < QT; q += U) {
    lanes<C, N> v[U];
    const int64_t c = x.c0 + cg + G::CG * q;
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = at2<0, N>(e, r, min(c + G::CG * u, cols - 1), x);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (c + G::CG * u >= cols) break;
      T* col = z + (c + G::CG * u) * rows;
      if (sh == 0) {
        store_lanes<N, NTS>(col, r, v[u]);
      } else {
#pragma unroll
        for (int j = 0; j < N; ++j)
          if (j >= sh) col[r + j] = static_cast<T>(v[u].v[j]);
      }
    }
  }
}

// ---- paired tiles: a matrix read both directly and transposed ----------------
//
// When an expression over square matrices names a matrix both directly and
// transposed (expr1: X and X.t()), output tiles (I, J) and (J, I) need the same
// two tiles of it.  One block then computes both: every thread loads its
// vectors of tiles (I, J) and (J, I) of every distinct matrix once, all in
// flight together.  A direct leaf of an output tile is in the very registers
// of the thread that computes it; for the transposed leaves the partner tile
// goes through LDS, one output tile after the other in the same buffers (all
// four tiles in LDS at once, as before, left two blocks per CU).  Each matrix
// is read from HBM once.  Whole matrices of the output's type only, at most
// kPairMats distinct ones;
// tiles of 64 x 64, 32 x 32 for 8-byte types.  2*(t(X) + Y) + 2*(X + t(Y)):
// FP32 10000 x 10000 261 -> 247 us; FP64 3001 x 3001, until then on the general
// kernel, 53 -> 38; BF16 10000 x 10000 286 -> 172.
constexpr int kPairMats = 2;
template <class T> constexpr int kPairSide = sizeof(T) == 8 ? 32 : 64;

// Every leaf a whole matrix, direct or transposed, of the output's storage type T
// (the kernel reads its matrices as that).
template <class E, class T> struct pairable { static constexpr bool value = false; };
template <class T> struct pairable<Leaf<T>, T> { static constexpr bool value = true; };
template <class T> struct pairable<Trans<T>, T> { static constexpr bool value = true; };
template <class Op, class A, class T> struct pairable<Unary<Op, A>, T> : pairable<A, T> {};
template <class Op, class A, bool L, class T> struct pairable<Scalar<Op, A, L>, T> : pairable<A, T> {};
template <class Op, class A, class B, class T> struct pairable<Binary<Op, A, B>, T> {
  static constexpr bool value = pairable<A, T>::value && pairable<B, T>::value;
};
template <class E> struct pair_leaves { static constexpr int value = 0; };
template <class T> struct pair_leaves<Leaf<T>> { static constexpr int value = 1; };
template <class T> struct pair_leaves<Trans<T>> { static constexpr int value = 1; };
template <class Op, class A> struct pair_leaves<Unary<Op, A>> : pair_leaves<A> {};
template <class Op, class A, bool L> struct pair_leaves<Scalar<Op, A, L>> : pair_leaves<A> {};
template <class Op, class A, class B> struct pair_leaves<Binary<Op, A, B>> {
  static constexpr int value = pair_leaves<A>::value + pair_leaves<B>::value;
};
constexpr int kPairMaxLeaves = 16;

struct pair_tab {
  uint8_t mid[kPairMaxLeaves];  // leaf (depth-first) -> distinct matrix
  const void* mat[kPairMats];   // distinct matrices
  int32_t n_mats;
};

// One vector of an output tile: its rows rl.. and column cl in the tile, the
// direct values of the distinct matrices there, the partner tiles in LDS.
template <class C, int N, int S> struct pair_ctx {
  const C* lds;
  const uint8_t* mid;
  int rl, cl;
  lanes<C, N> d[kPairMats];
};

template <int LOFF, class T, class C, int N, int S>
__device__ __forceinline__ lanes<C, N> at2p(const Leaf<T>&, const pair_ctx<C, N, S>& x) {
  const bool second = x.mid[LOFF] != 0;
  lanes<C, N> v;
#pragma unroll
  for (int j = 0; j < N; ++j) v.v[j] = second ? x.d[1].v[j] : x.d[0].v[j];
  return v;
}
template <int LOFF, class T, class C, int N, int S>
__device__ __forceinline__ lanes<C, N> at2p(const Trans<T>&, const pair_ctx<C, N, S>& x) {
  const C* b = x.lds + x.mid[LOFF] * (S * (S + 1)) + x.rl * (S + 1) + x.cl;
  lanes<C, N> v;
#pragma unroll
  for (int j = 0; j < N; ++j) v.v[j] = b[j * (S + 1)];
  return v;
}
template <int LOFF, class Op, class A, class C, int N, int S>
__device__ __forceinline__ lanes<C, N> at2p(const Unary<Op, A>& e, const pair_ctx<C, N, S>& x) {
  lanes<C, N> v = at2p<LOFF>(e.a, x);
  apply_lanes<Op, mod_none>(v.v);
  return v;
}
template <int LOFF, class Op, class A, bool L, class C, int N, int S>
__device__ __forceinline__ lanes<C, N> at2p(const Scalar<Op, A, L>& e, const pair_ctx<C, N, S>& x) {
  lanes<C, N> v = at2p<LOFF>(e.a, x);
#pragma unroll
  for (int j = 0; j < N; ++j) v.v[j] = e.apply1(v.v[j]);
  return v;
}
template <int LOFF, class Op, class A, class B, class C, int N, int S>
__device__ __forceinline__ lanes<C, N> at2p(const Binary<Op, A, B>& e, const pair_ctx<C, N, S>& x) {
  lanes<C, N> u = at2p<LOFF>(e.a, x);
  lanes<C, N> w = at2p<LOFF + pair_leaves<A>::value>(e.b, x);
#pragma unroll
  for (int j = 0; j < N; ++j) u.v[j] = Op::apply(u.v[j], w.v[j]);
  return u;
}

// Rows r..r+N-1 of a column that starts at p, of which only those below `rows`
// exist (the others repeat the last): N independent loads of one element.
template <int N, class T>
__device__ __forceinline__ lanes<ct_t<T>, N> load_end(const T* p, int64_t r, int64_t rows) {
  lanes<ct_t<T>, N> v;
#pragma unroll
  for (int j = 0; j < N; ++j) v.v[j] = static_cast<ct_t<T>>(p[min(r + j, rows - 1)]);
  return v;
}

// One block per tile pair I <= J (p enumerates them column by column).
template <class E, class T, bool NTL, bool NTS>
__global__ __launch_bounds__(kTileThreads) void k_ew2d_pair(E e, pair_tab tab, T* __restrict__ z,
                                                           int64_t n) {
  using C = typename E::ct;
  constexpr int S = kPairSide<T>, N = 16 / (int)sizeof(T), P = S + 1;
  constexpr int PER = S * S / N / kTileThreads;  // vectors per thread and tile
  static_assert(PER * N * kTileThreads == S * S, "whole vectors per thread");
  __shared__ C lds[kPairMats * S * P];
  const int64_t p = xcd_order(blockIdx.x, gridDim.x);
  int64_t J = (int64_t)((::sqrt(8.0 * (double)p + 1.0) - 1.0) * 0.5);
  while (J * (J + 1) / 2 > p) --J;
  while ((J + 1) * (J + 2) / 2 <= p) ++J;
  const int64_t I = p - J * (J + 1) / 2;
  const bool diagonal = I == J;
  // v[m][w][k]: this thread's vectors of tile (I, J) (w = 0) and (J, I) (w = 1)
  lanes<C, N> v[kPairMats][2][PER];
#pragma unroll
  for (int m = 0; m < kPairMats; ++m)
#pragma unroll
    for (int w = 0; w < 2; ++w)
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int idx = threadIdx.x + k * kTileThreads;
        const int64_t r = (w ? J : I) * S + (idx % (S / N)) * N, c = (w ? I : J) * S + idx / (S / N);
        if (m >= tab.n_mats || (w && diagonal) || r >= n || c >= n) continue;
        const T* col = static_cast<const T*>(tab.mat[m]) + c * n;
        v[m][w][k] = r + N <= n ? load_lanes<N, kNT && NTL>(col, r) : load_end<N>(col, r, n);
      }
#pragma unroll
  for (int s = 0; s < 2; ++s) {  // output tile (I, J), then (J, I)
    if (s && diagonal) break;
    if (s) __syncthreads();  // the first tile's reads are done
#pragma unroll
    for (int m = 0; m < kPairMats; ++m)
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int idx = threadIdx.x + k * kTileThreads;
        C* buf = lds + m * (S * P) + idx / (S / N) * P + (idx % (S / N)) * N;
        if (m < tab.n_mats)
#pragma unroll
          for (int j = 0; j < N; ++j) buf[j] = diagonal ? v[m][0][k].v[j] : v[m][1 - s][k].v[j];
      }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int idx = threadIdx.x + k * kTileThreads;
      pair_ctx<C, N, S> x{lds, tab.mid, (idx % (S / N)) * N, idx / (S / N), {v[0][s][k], v[1][s][k]}};
      const int64_t r = (s ? J : I) * S + x.rl, c = (s ? I : J) * S + x.cl;
      if (r >= n || c >= n) continue;
      const lanes<C, N> o = at2p<0>(e, x);
      if (r + N <= n) {
        store_lanes<N, NTS>(z, r + c * n, o);
      } else {
#pragma unroll
        for (int j = 0; j < N; ++j)
          if (r + j < n) z[r + j + c * n] = static_cast<T>(o.v[j]);
      }
    }
  }
}

// Host: the leaves (depth-first) of a pairable expression.
template <class T> inline void pair_leaf_list(const Leaf<T>& e, const void** p, int64_t* off,
                                              int64_t* ld, bool* tr, int& k) {
  p[k] = e.p; off[k] = 0; ld[k] = e.n_rows; tr[k] = false; ++k;
}
template <class T> inline void pair_leaf_list(const Trans<T>& e, const void** p, int64_t* off,
                                              int64_t* ld, bool* tr, int& k) {
  p[k] = e.p; off[k] = e.off; ld[k] = e.ld; tr[k] = true; ++k;
}
template <class Op, class A> inline void pair_leaf_list(const Unary<Op, A>& e, const void** p,
                                                        int64_t* off, int64_t* ld, bool* tr, int& k) {
  pair_leaf_list(e.a, p, off, ld, tr, k);
}
template <class Op, class A, bool L> inline void pair_leaf_list(const Scalar<Op, A, L>& e,
                                                                const void** p, int64_t* off,
                                                                int64_t* ld, bool* tr, int& k) {
  pair_leaf_list(e.a, p, off, ld, tr, k);
}
template <class Op, class A, class B> inline void pair_leaf_list(const Binary<Op, A, B>& e,
                                                                 const void** p, int64_t* off,
                                                                 int64_t* ld, bool* tr, int& k) {
  pair_leaf_list(e.a, p, off, ld, tr, k);
  pair_leaf_list(e.b, p, off, ld, tr, k);
}

// Build the pair table if the paired kernel applies: n x n result, every leaf
// a whole n x n matrix, at most kPairMats distinct ones, one of them read both
// ways.
template <class E> inline bool pair_plan(const E& e, int64_t n, pair_tab* tab) {
  constexpr int L = pair_leaves<E>::value;
  if (L > kPairMaxLeaves) return false;
  const void* p[kPairMaxLeaves];
  int64_t off[kPairMaxLeaves], ld[kPairMaxLeaves];
  bool tr[kPairMaxLeaves];
  int k = 0;
  pair_leaf_list(e, p, off, ld, tr, k);
  bool dir[kPairMats] = {false, false}, trn[kPairMats] = {false, false};
  tab->n_mats = 0;
  for (int i = 0; i < L; ++i) {
    if (off[i] != 0 || ld[i] != n) return false;
    int m = 0;
    while (m < tab->n_mats && tab->mat[m] != p[i]) ++m;
    if (m == tab->n_mats) {
      if (m == kPairMats) return false;
      tab->mat[m] = p[i];
      ++tab->n_mats;
    }
    tab->mid[i] = (uint8_t)m;
    (tr[i] ? trn : dir)[m] = true;
  }
  for (int m = 0; m < tab->n_mats; ++m)
    if (dir[m] && trn[m]) return true;
  return false;
}

// Z = E for an expression with submatrix or transposed leaves.
template <class E, class T>
int eval_views(T* z, const E& e, hipStream_t st) {
  int64_t rows, cols;
  if (int rc = check_expr(e, &rows, &cols)) return rc;
  if (rows * cols == 0) return FX_OK;
  if (!z) return fail(FX_E_ARG, "NULL output pointer");
  constexpr int NV = 16 / (int)sizeof(T);
  constexpr int KT = trans_count<E>::value;
  const uint64_t bytes = (uint64_t)rows * (uint64_t)cols * sizeof(T);
  const bool vec = KT > 0 ? rows >= NV && cols >= NV && bytes > kElementBelow : rows > kElementRows;
  const bool nts = kNTS || bytes > kStreamStoresAbove;
  const bool lines = pitch_of(e, 128), sets = pitch_of(e, kSetsPitch);
  view_arrays in;
  arrays_in(e, in);
  const uint64_t total = bytes + (uint64_t)rows * (uint64_t)cols * in.bytes;
  const bool few_sets = KT == 0 && sets && total > kSetsFrom;
  const uint64_t from = KT == 0 ? (lines ? 1 : 2) * kStreamFrom : pairable<E, T>::value ? kStreamPairsFrom : kStreamFrom;
  const bool ntl = total > from ? KT == 0 || lines : few_sets && total <= kSetsTo;
  auto with_policy = [&](auto&& go) {
    if (ntl) return nts ? go(std::true_type{}, std::true_type{}) : go(std::true_type{}, std::false_type{});
    return nts ? go(std::false_type{}, std::true_type{}) : go(std::false_type{}, std::false_type{});
  };
  if constexpr (KT > 0 && pairable<E, T>::value) {
    pair_tab tab;
    if (vec && rows == cols && pair_plan(e, rows, &tab)) {
      const int64_t t = ceil_div(rows, (int64_t)kPairSide<T>);
      if (t * (t + 1) / 2 > 0x7fffffff)
        return fail(FX_E_UNSUPPORTED, "%lld x %lld exceeds the tile grid", (long long)rows, (long long)cols);
      return with_policy([&](auto l, auto st_) {
        hipLaunchKernelGGL((k_ew2d_pair<E, T, decltype(l)::value, decltype(st_)::value>),
                           dim3((unsigned)(t * (t + 1) / 2)), dim3(kTileThreads), 0, st, e, tab, z, rows);
        return hip_check(hipGetLastError(), "k_ew2d_pair launch");
      });
    }
  }
  // one column per thread where four would leave threads without a column or
  // the chip with few blocks (sums of two submatrices: BF16 4900 x 4900, 5
  // blocks per CU, 6.7 us against 7.3; FP32 3000 x 3000, 2 per CU, 4.3 and 4.6,
  // 4000 x 4000, 4 per CU, 8.6 and 8.0); the narrow tile of transposed parts as
  // above
  const int64_t wide = ceil_div(cols, tile_geo<KT, NV, 4, T>::TC) * ceil_div(rows, tile_geo<KT, NV, 4, T>::TR);
  const bool narrow = KT > 0 ? !(sets && wide >= (int64_t)16 * device_cus())
                             : cols < tile_geo<KT, NV, 4, T>::TC ||
                                   (wide < (int64_t)(sizeof(T) == 4 ? 3 : 8) * device_cus() && !few_sets);
  auto launch = [&](auto Nc, auto Qc, auto l, auto st_) {
    constexpr int N = decltype(Nc)::value, Q = decltype(Qc)::value;
    using G = tile_geo<KT, N, Q, T>;
    const int64_t tc = ceil_div(cols, G::TC), tr = ceil_div(rows, G::TR);
    if (tr * tc > 0x7fffffff)
      return fail(FX_E_UNSUPPORTED, "%lld x %lld exceeds the tile grid", (long long)rows, (long long)cols);
    hipLaunchKernelGGL((k_ew2d<E, T, N, Q, decltype(l)::value, decltype(st_)::value>),
                       dim3((unsigned)(tr * tc)), dim3(kTileThreads), 0, st, e, z, rows, cols, (uint32_t)tr);
    return hip_check(hipGetLastError(), "k_ew2d launch");
  };
  if (!vec) return launch(ic<1>{}, ic<4>{}, std::false_type{}, std::false_type{});
  return with_policy([&](auto l, auto st_) {
    if constexpr (wide_tile<KT, NV, T>()) {
      if (!narrow) return launch(ic<NV>{}, ic<4>{}, l, st_);
    }
    return launch(ic<NV>{}, ic<1>{}, l, st_);
  });
}

}  // namespace fx

// A user's program on top of the expression front end: expressions over strided
// views, and sums of expressions with functions, that no entry point of the
// library instantiates.
#include "fx_views.hpp"

using namespace fx;

// 2*(X^T + Y) + (X + Y^T) over n x n matrices of storage T, written as Z's storage
// TZ: every matrix is read both ways.
template <class TZ, class T>
static int pair(void* z, const void* x, const void* y, int64_t n, void* st) {
  const auto X = leaf<T>(x, n, n), Y = leaf<T>(y, n, n);
  return eval_views(static_cast<TZ*>(z), 2 * (t(X) + Y) + (X + t(Y)), S(st));
}

// 2*X + A^T%X + B^T%X + C^T%X + D^T%X + E^T%X (m: X, A, B, C, D, E): five transposed parts.
template <class T> static int five(void* z, const void* const* m, int64_t n, void* st) {
  auto M = [&](int q) { return leaf<T>(m[q], n, n); };
  const auto X = M(0);
  return eval_views(static_cast<T*>(z), 2 * X + t(M(1)) % X + t(M(2)) % X + t(M(3)) % X + t(M(4)) % X +
                                            t(M(5)) % X, S(st));
}

// The sum of X / (1 + Y%Y), or the column sums of exp(X)%sqrt(|Y|) / (1 + Y%Y).
template <class T>
static int sums(int kind, const void* x, const void* y, fx_shape s, void* out, void* ws, size_t bytes, void* st) {
  const auto X = leaf<T>(x, s.n_rows, s.n_cols), Y = leaf<T>(y, s.n_rows, s.n_cols);
  if (kind == FX_R_ACCU) return reduce_full<map_id>(X / (1 + Y % Y), out, ws, bytes, nullptr, S(st));
  return reduce_dim(FX_R_COLSUM, exp(X) % sqrt(abs(Y)) / (1 + Y % Y), static_cast<acc_out_t<T>*>(out), ws,
                    bytes, nullptr, S(st));
}

extern "C" {

int user_sums_f32(int kind, const void* x, const void* y, fx_shape s, void* out, void* ws, size_t bytes, void* st) {
  return sums<float>(kind, x, y, s, out, ws, bytes, st);
}
int user_sums_f64(int kind, const void* x, const void* y, fx_shape s, void* out, void* ws, size_t bytes, void* st) {
  return sums<double>(kind, x, y, s, out, ws, bytes, st);
}

int user_five_f32(void* z, const void* const* m, int64_t n, void* st) { return five<float>(z, m, n, st); }
int user_five_f64(void* z, const void* const* m, int64_t n, void* st) { return five<double>(z, m, n, st); }

int user_pair_bf16_of_f32(void* z, const void* x, const void* y, int64_t n, void* st) {
  return pair<bf16_t, float>(z, x, y, n, st);
}
int user_pair_f32_of_bf16(void* z, const void* x, const void* y, int64_t n, void* st) {
  return pair<float, bf16_t>(z, x, y, n, st);
}
int user_pair_f16_of_bf16(void* z, const void* x, const void* y, int64_t n, void* st) {
  return pair<f16_t, bf16_t>(z, x, y, n, st);
}

}  // extern "C"

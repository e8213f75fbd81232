// A user's program on top of the expression front end: expressions over strided
// views that no entry point of the library instantiates.
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

extern "C" {

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

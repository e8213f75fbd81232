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

extern "C" {

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

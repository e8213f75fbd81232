// Learned launch-configuration model: a two-layer perceptron
//   x -> standardise -> h = relu(W1 x + b1) -> logits = W2 h + b2
// whose logits are split into one softmax head per launch knob (block, EPT,
// vector width, split), trained with softmax cross-entropy against the
// exhaustive autotuner's best configuration and Adam.  FP32 throughout, plain
// FMA arithmetic (the layers are 25x64 and 64x12: far too small for matrix
// cores to matter).
//
// Kernels:
//   k_mlp_rows    one 64-thread (or wider) group per batch row, the weights
//                 staged in LDS: forward, loss, dlogits, dh (the batch's rows
//                 optionally gathered through an index list)
//   k_mlp_params  one thread per parameter: gradient summed over the batch
//                 in row order (deterministic), then the Adam update
//   k_mlp_forward forward and per-head argmax, one row per block or rows looped
//                 over per block
// Parameters are one flat array: W1 [H x F] row-major, b1 [H], W2 [C x H],
// b2 [C], C = sum of head sizes.
#include <math.h>
#include <string.h>

#include <atomic>
#include <mutex>
#include <new>
#include <vector>

#include "fx_kernels.hpp"

namespace fx {

constexpr int kMlpMaxF = 64, kMlpMaxH = 256, kMlpMaxC = 64, kMlpMaxHeads = 8;

struct mlp_dims {
  int F, H, C, n_heads;
  int head_off[kMlpMaxHeads + 1];
  __host__ __device__ int W1() const { return 0; }
  __host__ __device__ int b1() const { return H * F; }
  __host__ __device__ int W2() const { return H * F + H; }
  __host__ __device__ int b2() const { return H * F + H + C * H; }
  __host__ __device__ int n_params() const { return H * F + H + C * H + C; }
};

__device__ __forceinline__ int64_t imin(int64_t a, int64_t b) { return a < b ? a : b; }

// A block works on R groups of rows at once, `tpr` threads each (tpr: a
// multiple of 64 covering max(F, H, C); R = 256 / tpr, at least 1).  What
// bounds these kernels is latency, not arithmetic (a row is 2.5 K
// multiply-adds): every parameter a block needs is loaded once, all loads in
// flight together, and the per-row dot products then read LDS.  Weight rows
// are padded to odd pitches there, so that threads reading down a column hit
// different banks.
struct mlp_launch {
  int tpr, groups;      // threads per row, rows (or row groups) per block
  int p1, p2;           // pitches of the staged W1 and W2
  uint32_t f_inv, h_inv;  // i / F = umulhi(i, f_inv) for i < 2^16, likewise H
  int weights;          // floats of staged weights (0: left in global memory)
  int per_row;          // floats per row: xn, h, logits, class terms, head losses
};
// Models whose weights exceed this leave them in global memory (the L1 and L2
// then serve the repeated reads).
constexpr int kMlpStagedFloats = 12 * 1024;

// The weights as the row code reads them: staged in LDS or in place.
template <bool STAGED> struct mlp_weights {
  const float *w1, *w2;
  int p1, p2;
  // `ready()` runs while the loads are in flight
  template <class F>
  __device__ __forceinline__ mlp_weights(const mlp_dims& d, const mlp_launch& L,
                                         const float* __restrict__ P, float* lds, F&& ready) {
    if constexpr (STAGED) {
      constexpr int PER = 12;  // loads in flight per thread
      const int n1 = d.H * d.F, n2 = d.C * d.H, n = n1 + n2, step = blockDim.x;
      float* s1 = lds;
      float* s2 = lds + d.H * L.p1;
      int i0 = threadIdx.x;
      do {
        float v[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          const int i = min(i0 + u * step, n - 1);
          v[u] = P[i < n1 ? d.W1() + i : d.W2() + (i - n1)];
        }
        if (i0 == (int)threadIdx.x) ready();
#pragma unroll
        for (int u = 0; u < PER; ++u) {
          const int i = i0 + u * step;
          if (i < n1) {
            const int j = __umulhi((unsigned)i, L.f_inv);
            s1[i + j * (L.p1 - d.F)] = v[u];
          } else if (i < n) {
            const int c = __umulhi((unsigned)(i - n1), L.h_inv);
            s2[(i - n1) + c * (L.p2 - d.H)] = v[u];
          }
        }
        i0 += PER * step;
      } while (i0 < n);
      w1 = s1;
      w2 = s2;
      p1 = L.p1;
      p2 = L.p2;
    } else {
      ready();
      w1 = P + d.W1();
      w2 = P + d.W2();
      p1 = d.F;
      p2 = d.H;
    }
  }
};

// Forward of RR rows by one group of threads (t: thread within the group);
// row q's buffers start at xn + q * per_row.  Every thread of the block calls
// it; the first barrier also covers the staged weights.  Each dot product is
// one chain of fused multiply-adds in index order, as in the host twin.
template <int RR, bool STAGED>
__device__ __forceinline__ void mlp_rows_forward(const mlp_dims& d, const mlp_launch& L,
                                                 const mlp_weights<STAGED>& w, int t,
                                                 const float (&x)[RR], float mean, float stdv,
                                                 float b1, float b2, float* xn) {
  if (t < d.F)
#pragma unroll
    for (int q = 0; q < RR; ++q) xn[q * L.per_row + t] = (x[q] - mean) / stdv;
  __syncthreads();
  float* h = xn + d.F;
  if (t < d.H) {
    float a[RR];
#pragma unroll
    for (int q = 0; q < RR; ++q) a[q] = b1;
    const float* k = w.w1 + t * w.p1;
#pragma unroll 8
    for (int f = 0; f < d.F; ++f)
#pragma unroll
      for (int q = 0; q < RR; ++q) a[q] = fmaf(k[f], xn[q * L.per_row + f], a[q]);
#pragma unroll
    for (int q = 0; q < RR; ++q) h[q * L.per_row + t] = a[q] > 0.f ? a[q] : 0.f;
  }
  __syncthreads();
  if (t < d.C) {
    float a[RR];
#pragma unroll
    for (int q = 0; q < RR; ++q) a[q] = b2;
    const float* k = w.w2 + t * w.p2;
#pragma unroll 8
    for (int j = 0; j < d.H; ++j)
#pragma unroll
      for (int q = 0; q < RR; ++q) a[q] = fmaf(k[j], h[q * L.per_row + j], a[q]);
#pragma unroll
    for (int q = 0; q < RR; ++q) h[q * L.per_row + d.H + t] = a[q];
  }
  __syncthreads();
}

template <bool STAGED>
__global__ __launch_bounds__(256) void k_mlp_rows(mlp_dims d, mlp_launch L,
                                                const float* __restrict__ X,
                                                const int32_t* __restrict__ labels,
                                                const int32_t* __restrict__ rows, int B,
                                                const float* __restrict__ mean,
                                                const float* __restrict__ stdv,
                                                const float* __restrict__ P, float* __restrict__ XN,
                                                float* __restrict__ Hs, float* __restrict__ DL,
                                                float* __restrict__ DH, float* __restrict__ row_loss) {
  extern __shared__ float lds[];
  const int sub = threadIdx.x / L.tpr, t = threadIdx.x - sub * L.tpr;
  const int64_t b = (int64_t)blockIdx.x * L.groups + sub;
  const bool live = b < B;
  // batch row b is data row r (threads past the batch repeat its last row and
  // write nothing)
  const size_t bb = live ? (size_t)b : (size_t)(B - 1);
  const size_t r = rows ? (size_t)rows[bb] : bb;
  const float mu = t < d.F ? mean[t] : 0.f, sd = t < d.F ? stdv[t] : 1.f;
  const float b1 = t < d.H ? P[d.b1() + t] : 0.f, b2 = t < d.C ? P[d.b2() + t] : 0.f;
  // class t: its head and that head's first class
  int head = 0;
  while (head + 1 < d.n_heads && t >= d.head_off[head + 1]) ++head;
  const int o = d.head_off[head], k = d.head_off[head + 1] - o;
  float x[1] = {0.f};
  int lab = 0;
  const mlp_weights<STAGED> w(d, L, P, lds, [&] {
    if (t < d.F) x[0] = X[r * d.F + t];
    if (t < d.C) lab = labels[r * d.n_heads + head];
  });
  float* xn = lds + L.weights + sub * L.per_row;
  float* h = xn + d.F;
  float* logit = h + d.H;
  float* term = logit + d.C;  // exp(logit - m), then dlogits
  float* head_loss = term + d.C;
  mlp_rows_forward<1, STAGED>(d, L, w, t, x, mu, sd, b1, b2, xn);
  // per-head softmax cross-entropy, one class per thread: loss = log sum
  // exp(logits) - logit[y]; dlogits = (softmax - onehot(y)) / B
  float m = 0.f, e = 0.f;
  if (t < d.C) {
    m = logit[o];
    for (int c = 1; c < k; ++c) m = fmaxf(m, logit[o + c]);
    e = expf(logit[t] - m);
    term[t] = e;
  }
  __syncthreads();
  float g = 0.f;
  if (t < d.C) {
    float z = 0.f;
    for (int c = 0; c < k; ++c) z += term[o + c];
    const int y = o + min(max(lab, 0), k - 1);
    g = (e / z - (t == y ? 1.f : 0.f)) / (float)B;
    if (t == o) head_loss[head] = logf(z) + m - logit[y];
  }
  __syncthreads();
  if (t < d.C) term[t] = g;
  __syncthreads();
  if (!live) return;
  if (t == 0) {
    float loss = 0.f;
    for (int q = 0; q < d.n_heads; ++q) loss += head_loss[q];
    row_loss[b] = loss;
  }
  if (t < d.F) XN[(size_t)b * d.F + t] = xn[t];
  if (t < d.H) {
    // dh_j = relu'(h_j) * sum_c W2[c, j] dl_c
    float s = 0.f;
#pragma unroll 8
    for (int c = 0; c < d.C; ++c) s = fmaf(w.w2[c * w.p2 + t], term[c], s);
    Hs[(size_t)b * d.H + t] = h[t];
    DH[(size_t)b * d.H + t] = h[t] > 0.f ? s : 0.f;
  }
  if (t < d.C) DL[(size_t)b * d.C + t] = g;
}

// The parameters as two matrices G[a][b] = sum over batch rows r, in row
// order, of A[r][a] * B[r][b], B extended by a column of ones for the bias:
//   layer 1: A = DH (H columns), B = [XN | 1] (F + 1)  ->  W1, b1
//   layer 2: A = DL (C columns), B = [Hs | 1] (H + 1)  ->  W2, b2
// One wave per 8 x 8 tile of G, one parameter per thread, then its Adam
// update.  (fma(A, 1, g) rounds as g + A does, so a bias needs no code of its
// own.)  The chain of B dependent multiply-adds a parameter's row-order sum
// needs is short (256 rows: under 1 us); the time is the loads' latency, so
// each chunk of kMlpChunk rows is brought into LDS with all its loads in
// flight, transposed so that a thread reads four rows per LDS access.  Reading
// the operands from global memory inside the chain took 66 us for a 256-row
// batch of the 25-64-14 model, this takes 5.  With lr == 0 the gradient is only written to
// `grad` (no update).
constexpr int kMlpTile = 8, kMlpChunk = 256, kMlpPitch = kMlpChunk + 4;

struct mlp_tiles {
  int a1, b1, a2, b2;  // tiles of each matrix, down and across
  __host__ __device__ explicit mlp_tiles(const mlp_dims& d)
      : a1((d.H + kMlpTile - 1) / kMlpTile), b1((d.F + kMlpTile) / kMlpTile),
        a2((d.C + kMlpTile - 1) / kMlpTile), b2((d.H + kMlpTile) / kMlpTile) {}
  __host__ __device__ int total() const { return a1 * b1 + a2 * b2; }
};

__global__ __launch_bounds__(64) void k_mlp_params(mlp_dims d, int B, const float* __restrict__ XN,
                                                 const float* __restrict__ Hs,
                                                 const float* __restrict__ DL,
                                                 const float* __restrict__ DH, float* __restrict__ P,
                                                 float* __restrict__ M, float* __restrict__ V,
                                                 float* __restrict__ grad, float lr, float beta1,
                                                 float beta2, float eps, float c1, float c2,
                                                 const float* __restrict__ row_loss,
                                                 float* __restrict__ loss) {
  __shared__ __align__(16) float As[kMlpTile * kMlpPitch], Bs[kMlpTile * kMlpPitch];
  const int t = threadIdx.x;
  const mlp_tiles T(d);
  int tile = blockIdx.x;
  if (tile == T.total()) {  // the mean loss (launched only when it is asked for)
    float L = 0.f;
    for (int64_t r0 = 0; r0 < B; r0 += kMlpChunk) {
      __syncthreads();
      for (int i = t; i < kMlpChunk; i += 64) As[i] = row_loss[imin(r0 + i, B - 1)];
      __syncthreads();
      const int n = (int)imin(kMlpChunk, B - r0);
      for (int i = 0; i < n; ++i) L += As[i];
    }
    if (t == 0) *loss = L / (float)B;
    return;
  }
  const bool first = tile < T.a1 * T.b1;
  if (!first) tile -= T.a1 * T.b1;
  const int across = first ? T.b1 : T.b2;
  const int a0 = tile / across * kMlpTile, b0 = tile % across * kMlpTile;
  const int na = first ? d.H : d.C, nb = first ? d.F : d.H;  // columns (nb: without the ones)
  const float* A = first ? DH : DL;
  const float* Bm = first ? XN : Hs;
  const int a = a0 + t / kMlpTile, b = b0 + t % kMlpTile;
  const bool mine = a < na && b <= nb;
  const int i = first ? (b < nb ? d.W1() + a * nb + b : d.b1() + a)
                      : (b < nb ? d.W2() + a * nb + b : d.b2() + a);
  float p = 0.f, m0 = 0.f, v0 = 0.f;
  if (mine && lr != 0.f) { p = P[i]; m0 = M[i]; v0 = V[i]; }
  const int lc = t % kMlpTile, lr0 = t / kMlpTile;  // staging: column of the tile, first row
  const int ca = min(a0 + lc, na - 1), cb = min(b0 + lc, nb - 1);
  const bool ones = b0 + lc >= nb;
  float g = 0.f;
  for (int64_t r0 = 0; r0 < B; r0 += kMlpChunk) {
    const int n = (int)imin(kMlpChunk, B - r0);
    constexpr int PER = kMlpChunk / kMlpTile;
    float va[PER], vb[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const size_t r = imin(r0 + lr0 + u * kMlpTile, B - 1);
      va[u] = A[r * na + ca];
      vb[u] = Bm[r * nb + cb];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      As[lc * kMlpPitch + lr0 + u * kMlpTile] = va[u];
      Bs[lc * kMlpPitch + lr0 + u * kMlpTile] = ones ? 1.f : vb[u];
    }
    __syncthreads();
    const float* qa = As + (t / kMlpTile) * kMlpPitch;
    const float* qb = Bs + (t % kMlpTile) * kMlpPitch;
    int r = 0;
#pragma unroll 4
    for (; r + 4 <= n; r += 4) {
      const float4 x = *reinterpret_cast<const float4*>(qa + r);
      const float4 y = *reinterpret_cast<const float4*>(qb + r);
      g = fmaf(x.x, y.x, g);
      g = fmaf(x.y, y.y, g);
      g = fmaf(x.z, y.z, g);
      g = fmaf(x.w, y.w, g);
    }
    for (; r < n; ++r) g = fmaf(qa[r], qb[r], g);
  }
  if (!mine) return;
  if (grad) grad[i] = g;
  if (lr == 0.f) return;
  const float m = beta1 * m0 + (1.f - beta1) * g;
  const float v = beta2 * v0 + (1.f - beta2) * g * g;
  M[i] = m;
  V[i] = v;
  P[i] = p - lr * (m / c1) / (sqrtf(v / c2) + eps);
}

// Inference: a group of threads takes RR rows at a time, so that one read of a
// weight serves RR independent chains, from weights staged once per block.  Up to
// 16 waves per CU (64 of models whose weights are neither staged nor over 96 KiB) each row has a
// group and a block of its own, which reads the weights from the caches: the
// chip is not full, and staging, or four rows one after another, only adds its
// latency (25-64-14 model, through the binding: 256 rows 8.1 us against 9.9,
// 4096 8.3 and 9.0, 20000 23.8 and 16.3; 64-256-64 256 rows 9.5 and 18.3, 4096 63 and
// 23; 25-200-63, not staged, 256 rows 10 and 28, 4096 28 and 31, 20000 146 and 128).
// Rows of their own read the weights from the L2 again each: over 96 KiB that bounds
// them from 1024 rows on (64-256-64, 1024 rows 18 us both ways).
constexpr int kMlpForwardRows = 4;
constexpr int kMlpSingleWaves = 16, kMlpSingleWavesUnstaged = 64, kMlpLargeFloats = 24 * 1024;
template <int RR, bool STAGED>
__global__ __launch_bounds__(256) void k_mlp_forward(mlp_dims d, mlp_launch L, int B,
                                                   const float* __restrict__ X,
                                                   const float* __restrict__ mean,
                                                   const float* __restrict__ stdv,
                                                   const float* __restrict__ P,
                                                   float* __restrict__ logits,
                                                   int32_t* __restrict__ choice) {
  extern __shared__ float lds[];
  const int sub = threadIdx.x / L.tpr, t = threadIdx.x - sub * L.tpr;
  const float mu = t < d.F ? mean[t] : 0.f, sd = t < d.F ? stdv[t] : 1.f;
  const float b1 = t < d.H ? P[d.b1() + t] : 0.f, b2 = t < d.C ? P[d.b2() + t] : 0.f;
  const int64_t stride = (int64_t)gridDim.x * L.groups * RR;
  float x[RR] = {};
  auto fetch = [&](int64_t b) {  // rows past the batch repeat its last
    if (t < d.F)
#pragma unroll
      for (int q = 0; q < RR; ++q) x[q] = X[(size_t)imin(b + q, B - 1) * d.F + t];
  };
  const mlp_weights<STAGED> w(d, L, P, lds, [&] {
    fetch(((int64_t)blockIdx.x * L.groups + sub) * RR);
  });
  float* xn = lds + L.weights + sub * RR * L.per_row;
  const float* logit = xn + d.F + d.H;
  // uniform over the block: the loop runs on the block's first row
  for (int64_t b0 = (int64_t)blockIdx.x * L.groups * RR; b0 < B; b0 += stride) {
    const int64_t b = b0 + sub * RR;
    mlp_rows_forward<RR, STAGED>(d, L, w, t, x, mu, sd, b1, b2, xn);
    if (b0 + stride < B) fetch(b + stride);
#pragma unroll
    for (int q = 0; q < RR; ++q) {
      if (b + q >= B) break;
      const float* z = logit + q * L.per_row;
      if (logits && t < d.C) logits[(size_t)(b + q) * d.C + t] = z[t];
      if (choice && t < d.n_heads) {
        const int o = d.head_off[t], k = d.head_off[t + 1] - o;
        int best = 0;
        for (int c = 1; c < k; ++c)
          if (z[o + c] > z[o + best]) best = c;
        choice[(size_t)(b + q) * d.n_heads + t] = best;
      }
    }
    __syncthreads();  // the row buffers are rewritten by the next iteration
  }
}

static mlp_launch mlp_shape(const mlp_dims& d) {
  mlp_launch L;
  L.tpr = std::max(64, (std::max(d.H, std::max(d.F, d.C)) + 63) / 64 * 64);
  L.groups = std::max(1, 256 / L.tpr);
  L.p1 = d.F | 1;
  L.p2 = d.H | 1;
  L.f_inv = (uint32_t)(((uint64_t)1 << 32) / d.F + 1);
  L.h_inv = (uint32_t)(((uint64_t)1 << 32) / d.H + 1);
  const int w = d.H * L.p1 + d.C * L.p2;
  L.weights = w <= kMlpStagedFloats ? w : 0;
  L.per_row = d.F + d.H + 2 * d.C + kMlpMaxHeads;
  return L;
}

}  // namespace fx

using namespace fx;

struct fx_model {
  mlp_dims d;
  float* dP = nullptr;   // params, Adam moments, standardisation
  float* dM = nullptr;
  float* dV = nullptr;
  float* dMean = nullptr;
  float* dStd = nullptr;
  float* scratch = nullptr;  // XN, Hs, DL, DH, row_loss for `cap` rows
  int cap = 0;
  int32_t* perm = nullptr;  // fx_model_train's visiting order, `perm_cap` entries
  size_t perm_cap = 0;
  long step = 0;
  // Host twin for single queries.  Training updates the parameters on the
  // device only and marks the twin stale; it is refreshed (after the device
  // has finished) before anything reads it.  `version` counts every change
  // of the parameters or the standardisation, so cached picks can tell.
  mutable std::mutex twin_mu;
  mutable bool twin_stale = false;
  mutable std::vector<float> hP;
  std::vector<float> hMean, hStd;
  std::atomic<long> version{0};
};

namespace fx {
long model_version(const fx_model* m) { return m ? m->version.load() : 0; }
}  // namespace fx

// Bring the host twin of the parameters up to date (caller holds twin_mu).
static int refresh_twin(const fx_model* m) {
  if (!m->twin_stale) return FX_OK;
  if (int rc = hip_check(hipDeviceSynchronize(), "model twin refresh")) return rc;
  if (int rc = hip_check(hipMemcpy(m->hP.data(), m->dP, m->d.n_params() * sizeof(float),
                                   hipMemcpyDeviceToHost), "model twin refresh"))
    return rc;
  m->twin_stale = false;
  return FX_OK;
}

// Release paths cannot report errors: a failed hipFree here only means the
// context is already gone.
static void model_free(fx_model* m) {
  (void)hipFree(m->dP);
  (void)hipFree(m->dM);
  (void)hipFree(m->dV);
  (void)hipFree(m->dMean);
  (void)hipFree(m->dStd);
  (void)hipFree(m->scratch);
  (void)hipFree(m->perm);
}

static int ensure_scratch(fx_model* m, int B) {
  if (B <= m->cap) return FX_OK;
  (void)hipFree(m->scratch);
  m->scratch = nullptr;
  const mlp_dims& d = m->d;
  const size_t per_row = (size_t)d.F + 2 * d.H + d.C + 1;
  if (int rc = hip_check(hipMalloc((void**)&m->scratch, per_row * B * sizeof(float)), "hipMalloc")) {
    m->cap = 0;
    return rc;
  }
  m->cap = B;
  return FX_OK;
}

extern "C" {

int fx_model_create(int32_t n_features, int32_t hidden, const int32_t* head_sizes, int32_t n_heads,
                    fx_model** out) {
  if (!out || !head_sizes) return fail(FX_E_ARG, "NULL argument");
  *out = nullptr;
  if (n_features <= 0 || n_features > kMlpMaxF || hidden <= 0 || hidden > kMlpMaxH ||
      n_heads <= 0 || n_heads > kMlpMaxHeads)
    return fail(FX_E_ARG, "model dimensions out of range (F <= %d, H <= %d, heads <= %d)", kMlpMaxF,
                kMlpMaxH, kMlpMaxHeads);
  mlp_dims d{};
  d.F = n_features;
  d.H = hidden;
  d.n_heads = n_heads;
  d.head_off[0] = 0;
  for (int q = 0; q < n_heads; ++q) {
    if (head_sizes[q] < 2) return fail(FX_E_ARG, "head %d needs at least two classes", q);
    d.head_off[q + 1] = d.head_off[q] + head_sizes[q];
  }
  d.C = d.head_off[n_heads];
  if (d.C > kMlpMaxC) return fail(FX_E_ARG, "too many classes (%d)", d.C);
  fx_model* m = new (std::nothrow) fx_model;
  if (!m) return fail(FX_E_ARG, "out of host memory");
  m->d = d;
  const size_t np = d.n_params();
  hipError_t e = hipSuccess;
  auto alloc = [&](float** p, size_t n) {
    if (e == hipSuccess) e = hipMalloc((void**)p, n * sizeof(float));
  };
  alloc(&m->dP, np);
  alloc(&m->dM, np);
  alloc(&m->dV, np);
  alloc(&m->dMean, d.F);
  alloc(&m->dStd, d.F);
  if (e == hipSuccess) e = hipMemset(m->dP, 0, np * sizeof(float));
  if (e == hipSuccess) e = hipMemset(m->dM, 0, np * sizeof(float));
  if (e == hipSuccess) e = hipMemset(m->dV, 0, np * sizeof(float));
  m->hP.assign(np, 0.f);
  m->hMean.assign(d.F, 0.f);
  m->hStd.assign(d.F, 1.f);
  if (e == hipSuccess)
    e = hipMemcpy(m->dMean, m->hMean.data(), d.F * sizeof(float), hipMemcpyHostToDevice);
  if (e == hipSuccess)
    e = hipMemcpy(m->dStd, m->hStd.data(), d.F * sizeof(float), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    int rc = hip_check(e, "fx_model_create");
    model_free(m);
    delete m;
    return rc;
  }
  *out = m;
  return FX_OK;
}

int32_t fx_model_num_params(const fx_model* m) { return m ? m->d.n_params() : 0; }

int fx_model_set(fx_model* m, const float* params, const float* mean, const float* stdv) {
  if (!m) return fail(FX_E_ARG, "NULL model");
  const mlp_dims& d = m->d;
  if (stdv)
    for (int f = 0; f < d.F; ++f)
      if (!(stdv[f] > 0.f)) return fail(FX_E_ARG, "standard deviation %d is not positive", f);
  std::lock_guard<std::mutex> g(m->twin_mu);
  // only the arrays passed are written; the others keep their current values
  // on the device (the host twin of the parameters may be stale then, and is
  // refreshed when next read)
  hipError_t e = hipSuccess;
  if (params) {
    e = hipDeviceSynchronize();  // queued training steps finish before the overwrite
    m->hP.assign(params, params + d.n_params());
    m->twin_stale = false;
    if (e == hipSuccess)
      e = hipMemcpy(m->dP, m->hP.data(), d.n_params() * sizeof(float), hipMemcpyHostToDevice);
    // a new starting point resets Adam
    if (e == hipSuccess) e = hipMemset(m->dM, 0, d.n_params() * sizeof(float));
    if (e == hipSuccess) e = hipMemset(m->dV, 0, d.n_params() * sizeof(float));
    m->step = 0;
  }
  if (mean) {
    m->hMean.assign(mean, mean + d.F);
    if (e == hipSuccess)
      e = hipMemcpy(m->dMean, m->hMean.data(), d.F * sizeof(float), hipMemcpyHostToDevice);
  }
  if (stdv) {
    m->hStd.assign(stdv, stdv + d.F);
    if (e == hipSuccess)
      e = hipMemcpy(m->dStd, m->hStd.data(), d.F * sizeof(float), hipMemcpyHostToDevice);
  }
  m->version++;
  return hip_check(e, "fx_model_set");
}

int fx_model_get(fx_model* m, float* params, float* mean, float* stdv) {
  if (!m) return fail(FX_E_ARG, "NULL model");
  const mlp_dims& d = m->d;
  std::lock_guard<std::mutex> g(m->twin_mu);
  m->twin_stale = true;  // read the device copy even if nothing was trained
  if (int rc = refresh_twin(m)) return rc;
  if (params) memcpy(params, m->hP.data(), d.n_params() * sizeof(float));
  if (mean) memcpy(mean, m->hMean.data(), d.F * sizeof(float));
  if (stdv) memcpy(stdv, m->hStd.data(), d.F * sizeof(float));
  return FX_OK;
}

// Gradient (lr = 0) or one Adam step over a batch of B rows in device memory.
// `rows` (device, may be NULL) lists the B data rows of the batch.
static int model_step(fx_model* m, const float* X, const int32_t* labels, const int32_t* rows,
                      int32_t B, float lr, float beta1, float beta2, float eps, float* d_loss,
                      float* d_grad, hipStream_t st) {
  if (!m || !X || !labels || B <= 0) return fail(FX_E_ARG, "bad arguments");
  if (int rc = ensure_scratch(m, B)) return rc;
  const mlp_dims& d = m->d;
  float* XN = m->scratch;
  float* Hs = XN + (size_t)B * d.F;
  float* DL = Hs + (size_t)B * d.H;
  float* DH = DL + (size_t)B * d.C;
  float* RL = DH + (size_t)B * d.H;
  const mlp_launch L = mlp_shape(d);
  const dim3 grid((B - 1) / L.groups + 1), block(L.tpr * L.groups);
  const size_t lds = sizeof(float) * (L.weights + (size_t)L.groups * L.per_row);
  auto rows_kernel = L.weights ? k_mlp_rows<true> : k_mlp_rows<false>;
  hipLaunchKernelGGL(rows_kernel, grid, block, lds, st, d, L, X, labels, rows, (int)B, m->dMean,
                     m->dStd, m->dP, XN, Hs, DL, DH, RL);
  double c1 = 1.0, c2 = 1.0;
  if (lr != 0.f) {
    m->step += 1;
    c1 = 1.0 - pow((double)beta1, (double)m->step);
    c2 = 1.0 - pow((double)beta2, (double)m->step);
  }
  hipLaunchKernelGGL(k_mlp_params, dim3(mlp_tiles(d).total() + (d_loss ? 1 : 0)), dim3(64), 0, st,
                     d, (int)B, XN, Hs, DL, DH, m->dP, m->dM, m->dV, d_grad, lr, beta1, beta2, eps,
                     (float)c1, (float)c2, RL, d_loss);
  if (lr != 0.f) {  // the parameters change on the device
    std::lock_guard<std::mutex> g(m->twin_mu);
    m->twin_stale = true;
    m->version++;
  }
  return hip_check(hipGetLastError(), "k_mlp launch");
}

int fx_model_train_step(fx_model* m, const float* d_X, const int32_t* d_labels, int32_t batch,
                        float lr, float* d_loss, void* stream) {
  if (!(lr > 0.f)) return fail(FX_E_ARG, "learning rate must be positive");
  return model_step(m, d_X, d_labels, nullptr, batch, lr, 0.9f, 0.999f, 1e-8f, d_loss, nullptr,
                    S(stream));
}

int fx_model_train(fx_model* m, const float* d_X, const int32_t* d_labels, int32_t n,
                   int32_t epochs, int32_t batch, float lr, const int32_t* perm,
                   float* d_losses, void* stream) {
  if (!m || !d_X || !d_labels || n <= 0 || epochs < 0 || batch <= 0)
    return fail(FX_E_ARG, "bad arguments");
  if (!(lr > 0.f)) return fail(FX_E_ARG, "learning rate must be positive");
  if (epochs == 0) return FX_OK;
  const size_t total = (size_t)epochs * n;
  if (perm) {  // every epoch's order must be a permutation of 0..n-1
    std::vector<uint8_t> seen(n);
    for (int32_t e = 0; e < epochs; ++e) {
      std::fill(seen.begin(), seen.end(), 0);
      for (int32_t i = 0; i < n; ++i) {
        const int32_t r = perm[(size_t)e * n + i];
        if (r < 0 || r >= n || seen[r]) return fail(FX_E_ARG, "epoch %d order is not a permutation", e);
        seen[r] = 1;
      }
    }
  }
  hipStream_t st = S(stream);
  if (total > m->perm_cap) {
    (void)hipFree(m->perm);
    m->perm = nullptr;
    m->perm_cap = 0;
    if (int rc = hip_check(hipMalloc((void**)&m->perm, total * sizeof(int32_t)), "hipMalloc"))
      return rc;
    m->perm_cap = total;
  }
  std::vector<int32_t> natural;
  const int32_t* src = perm;
  if (!src) {
    natural.resize(total);
    for (size_t i = 0; i < total; ++i) natural[i] = (int32_t)(i % (size_t)n);
    src = natural.data();
  }
  // The order buffer belongs to the model: the copy is queued behind the
  // stream's earlier work, and waited for before the host array can go.
  if (int rc = hip_check(hipMemcpyAsync(m->perm, src, total * sizeof(int32_t),
                                        hipMemcpyHostToDevice, st), "hipMemcpyAsync"))
    return rc;
  if (int rc = hip_check(hipStreamSynchronize(st), "hipStreamSynchronize")) return rc;
  for (int32_t e = 0; e < epochs; ++e)
    for (int32_t s = 0; s < n; s += batch) {
      const int32_t b = std::min(batch, n - s);
      const bool last = s + b >= n;
      if (int rc = model_step(m, d_X, d_labels, m->perm + (size_t)e * n + s, b, lr, 0.9f, 0.999f,
                              1e-8f, last && d_losses ? d_losses + e : nullptr, nullptr, st))
        return rc;
    }
  return FX_OK;
}

int fx_model_grad(fx_model* m, const float* d_X, const int32_t* d_labels, int32_t batch,
                  float* d_grad, float* d_loss, void* stream) {
  if (!d_grad) return fail(FX_E_ARG, "NULL gradient output");
  return model_step(m, d_X, d_labels, nullptr, batch, 0.f, 0.9f, 0.999f, 1e-8f, d_loss, d_grad,
                    S(stream));
}

int fx_model_forward(const fx_model* m, const float* d_X, int32_t batch, float* d_logits,
                     int32_t* d_choice, void* stream) {
  if (!m || !d_X || batch < 0 || (!d_logits && !d_choice)) return fail(FX_E_ARG, "bad arguments");
  if (batch == 0) return FX_OK;
  const mlp_dims& d = m->d;
  mlp_launch L = mlp_shape(d);
  const bool many = !L.weights && d.H * L.p1 + d.C * L.p2 <= kMlpLargeFloats;
  const int64_t single = (int64_t)device_cus() * (many ? kMlpSingleWavesUnstaged : kMlpSingleWaves);
  if ((int64_t)batch * (L.tpr / 64) <= single) {
    L.groups = 1;
    L.weights = 0;
    hipLaunchKernelGGL((k_mlp_forward<1, false>), dim3(batch), dim3(L.tpr), sizeof(float) * L.per_row, S(stream),
                       d, L, (int)batch, d_X, m->dMean, m->dStd, m->dP, d_logits, d_choice);
    return hip_check(hipGetLastError(), "k_mlp_forward launch");
  }
  const int per_block = L.groups * kMlpForwardRows;
  const size_t lds = sizeof(float) * (L.weights + (size_t)per_block * L.per_row);
  // each block stages the weights once and loops over its rows
  const int grid = std::min((batch - 1) / per_block + 1, 8 * device_cus());
  auto kernel = L.weights ? k_mlp_forward<kMlpForwardRows, true> : k_mlp_forward<kMlpForwardRows, false>;
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(L.tpr * L.groups), lds, S(stream), d, L, (int)batch,
                     d_X, m->dMean, m->dStd, m->dP, d_logits, d_choice);
  return hip_check(hipGetLastError(), "k_mlp_forward launch");
}

// Host twin of the predict kernel for one feature row (no GPU involved): the
// same arithmetic in the same order, FP32 with fused multiply-adds.
int fx_model_choose(const fx_model* m, const float* x, int32_t* choice) {
  if (!m || !x || !choice) return fail(FX_E_ARG, "NULL argument");
  const mlp_dims& d = m->d;
  std::lock_guard<std::mutex> g(m->twin_mu);
  if (int rc = refresh_twin(m)) return rc;
  const float* P = m->hP.data();
  float xn[kMlpMaxF], h[kMlpMaxH], logit[kMlpMaxC];
  for (int f = 0; f < d.F; ++f) xn[f] = (x[f] - m->hMean[f]) / m->hStd[f];
  for (int j = 0; j < d.H; ++j) {
    float a = P[d.b1() + j];
    for (int f = 0; f < d.F; ++f) a = fmaf(P[d.W1() + j * d.F + f], xn[f], a);
    h[j] = a > 0.f ? a : 0.f;
  }
  for (int c = 0; c < d.C; ++c) {
    float a = P[d.b2() + c];
    for (int j = 0; j < d.H; ++j) a = fmaf(P[d.W2() + c * d.H + j], h[j], a);
    logit[c] = a;
  }
  for (int q = 0; q < d.n_heads; ++q) {
    const int o = d.head_off[q], k = d.head_off[q + 1] - o;
    int best = 0;
    for (int c = 1; c < k; ++c)
      if (logit[o + c] > logit[o + best]) best = c;
    choice[q] = best;
  }
  return FX_OK;
}

void fx_model_destroy(fx_model* m) {
  if (!m) return;
  (void)hipDeviceSynchronize();  // queued work may still use the buffers
  model_free(m);
  delete m;
}

}  // extern "C"

// linreg.hip -- one gradient-descent step of MC-Linear regression with the mean-squared
// error, the paper's precision experiment (Section 2.4): a single MC-Linear layer
// without bias fitted by gradient descent to y = X W*^T.
//
// The step (in stream order, all on the device):
//   1. yhat = MC-Linear(X, W)                   MM-MCN order (Section 2.3)
//   2. r    = Grow-ExpN(yhat, -y)               the MC residual, in place of yhat
//   3. G    = r^T X                             K-split product, default slice count
//   4. RR   = r . r                             K-split product, default slice count
//   5. per weight j: g = ScalingN(G_j, fl(2/n)); the gradient is g's leading component
//      (the paper keeps the gradient of an MC value as the plain gradient of its
//      leading component, Section 2.1); W_j = Grow-ExpN(W_j, fl(-lr * grad));
//      loss = ScalingN(RR, fl(1/n)), the mean-squared error at the weights before the
//      update.
// fl(2/n), fl(1/n) and fl(-lr) are the component-format roundings of the binary64
// quotient or value (one rounding each, done on the host); fl(-lr * grad) is one
// rounding of the product in the component format.
//
// The step is launch- and latency-bound (three dependent launches for n <= 16447 and
// d <= 16): 1 and 2 are one kernel with a sample a lane, 3 and 4 are one launch with every
// sum's slices side by side (splitk.hip: sk_chain_kernel).  n = 10000, d = 2, a step of
// binary32 nc = 2 / binary16 nc = 3: 39 / 84 us as five launches of the general kernels, now
// 19.9 / 21.3 us (replayed from a graph 19.6 / 20.9; the kernels of the first take 2.9, 10.4
// and 3.2 us).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mcf_arith.hpp"
#include "mcf_internal.hpp"
#include "mm_steps.hpp"

namespace mcf {

namespace {

// r_i = Grow-ExpN(MC-Linear(X_i, W), -y_i) for d <= LR_MAX_D features, one sample a lane (a
// chain of d steps: a few samples' worth of a wavefront's time, where the product kernel
// and a launch of its own for Grow-ExpN cost 9 us).
constexpr int64_t LR_MAX_D = 16;

template <typename T, int NC>
__global__ __launch_bounds__(256) void lr_residual_kernel(const T *__restrict__ X, const T *__restrict__ y_neg,
                                                          const T *__restrict__ W, T *__restrict__ R, int64_t n, int d) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  T acc[NC], r[NC];
  for (int j = 0; j < d; ++j) {
    T w[NC], t[NC], h[NC + 1];
#pragma unroll
    for (int c = 0; c < NC; ++c) w[c] = W[c * d + j];
    scaling_terms<T, NC>(w, X[i * d + j], h);
    compact_nz<T, NC + 1, NC>(h, t);
    if (j == 0) {
      nonfinite_tail<T, NC>(t);
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[c] = t[c];
    } else {
      add_terms<T, NC>(acc, t, h);
      compact_nz<T, NC + 1, NC>(h, acc);
    }
  }
  grow_expn<T, NC>(acc, y_neg[i], r);
#pragma unroll
  for (int c = 0; c < NC; ++c) R[c * n + i] = r[c];
}

// G: planes g_plane apart.  RR: parts components of r's products with itself, part p at
// RR + p, planes rr_plane apart; they are added left to right.
template <typename T, int NC>
__global__ void lr_update_kernel(const T *G, int64_t g_plane, const T *RR, int64_t rr_plane, int parts, T *W, int64_t d,
                                 T s2n, T s1n, T neg_lr, T *loss) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j < d) {
    T g[NC], gs[NC], w[NC], wn[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      g[c] = G[c * g_plane + j];
      w[c] = W[c * d + j];
    }
    scaling_n<T, NC, NC>(g, s2n, gs);
    const T step = neg_lr * gs[0];  // one rounding in the component format
    grow_expn<T, NC>(w, step, wn);
#pragma unroll
    for (int c = 0; c < NC; ++c) W[c * d + j] = wn[c];
  }
  if (j == d && loss != nullptr) {
    T rr[NC], l[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) rr[c] = RR[c * rr_plane];
    for (int p = 1; p < parts; ++p) {
      T part[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) part[c] = RR[c * rr_plane + p];
      add_mcn<T, NC>(rr, part, rr);
    }
    scaling_n<T, NC, NC>(rr, s1n, l);
#pragma unroll
    for (int c = 0; c < NC; ++c) loss[c] = l[c];
  }
}

template <typename T, int NC>
hipError_t lr_step(int dtype, int64_t n, int64_t d, const T *X, const T *y_neg, T *W, T s2n, T s1n, T neg_lr, T *R, T *G,
                   T *RR, void *SK, T *loss, hipStream_t s) {
  hipError_t e;
  if (d <= LR_MAX_D) {
    hipLaunchKernelGGL((lr_residual_kernel<T, NC>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, X, y_neg, W, R, n,
                       (int)d);
    e = hipGetLastError();
  } else {
    e = launch_matmul(dtype, NC, n, 1, d, X, 0, W, 1, 1, nullptr, R, s);
    if (e != hipSuccess) return e;
    e = launch_elementwise(dtype, EW_ADD, NC, NC, n, R, 1, y_neg, 0, R, s);
  }
  if (e != hipSuccess) return e;
  // G = r^T X and RR = r . r.  With one slice count of at most one group for both, all of
  // their chains run side by side in one launch; [G | RR's parts] takes G's and RR's space
  // (nc nc components more than G's, at most 128 bytes).
  const int64_t S = splitk_default_slices(1, d, n), S1 = splitk_default_slices(1, 1, n);
  const bool both = S == S1 && splitk_roots(S) == 0;
  if (both) {
    e = launch_linreg_sums(dtype, NC, n, d, X, R, S, G, s);
  } else {
    e = launch_matmul_splitk(dtype, NC, 1, d, n, R, 1, X, 0, S, SK, G, s);
    if (e != hipSuccess) return e;
    e = launch_matmul_splitk(dtype, NC, 1, 1, n, R, 1, R, 1, S1, SK, RR, s);
  }
  if (e != hipSuccess) return e;
  // (lane d takes the loss)
  const dim3 grid((unsigned)((d + 1 + 255) / 256)), block(256);
  if (both)
    hipLaunchKernelGGL((lr_update_kernel<T, NC>), grid, block, 0, s, G, d + NC, G + d, d + NC, NC, W, d, s2n, s1n, neg_lr,
                       loss);
  else
    hipLaunchKernelGGL((lr_update_kernel<T, NC>), grid, block, 0, s, G, d, RR, (int64_t)1, 1, W, d, s2n, s1n, neg_lr, loss);
  return hipGetLastError();
}

template <typename T>
hipError_t lr_step_nc(int nc, int dtype, int64_t n, int64_t d, const T *X, const T *y_neg, T *W, T s2n, T s1n, T neg_lr,
                      T *R, T *G, T *RR, void *SK, T *loss, hipStream_t s) {
  switch (nc) {
    case 1: return lr_step<T, 1>(dtype, n, d, X, y_neg, W, s2n, s1n, neg_lr, R, G, RR, SK, loss, s);
    case 2: return lr_step<T, 2>(dtype, n, d, X, y_neg, W, s2n, s1n, neg_lr, R, G, RR, SK, loss, s);
    case 3: return lr_step<T, 3>(dtype, n, d, X, y_neg, W, s2n, s1n, neg_lr, R, G, RR, SK, loss, s);
    case 4: return lr_step<T, 4>(dtype, n, d, X, y_neg, W, s2n, s1n, neg_lr, R, G, RR, SK, loss, s);
  }
  return hipErrorInvalidValue;
}

int64_t align256(int64_t x) { return (x + 255) / 256 * 256; }

struct LrLayout {
  int64_t r, g, rr, sk, total;
};

LrLayout lr_layout(int dtype, int nc, int64_t n, int64_t d) {
  const int64_t es = dtype == 0 ? 2 : (dtype == 2 ? 8 : 4);
  LrLayout L;
  L.r = 0;
  L.g = align256(nc * n * es);
  L.rr = L.g + align256(nc * d * es);
  L.sk = L.rr + align256(nc * es);
  // K-split workspaces of r^T X (M = 1, N = d, MC x plain) and r . r (M = N = 1, MC x MC)
  const int64_t w1 = splitk_roots(splitk_default_slices(1, d, n)) * nc * d * es;
  const int64_t w2 = splitk_roots(splitk_default_slices(1, 1, n)) * nc * nc * es;
  L.total = L.sk + align256(w1 > w2 ? w1 : w2);
  return L;
}

}  // namespace

int64_t linreg_workspace_bytes(int dtype, int nc, int64_t n, int64_t d) { return lr_layout(dtype, nc, n, d).total; }

hipError_t launch_linreg_step(int dtype, int nc, int64_t n, int64_t d, const void *X, const void *y_neg, void *W,
                              double s2n, double s1n, double neg_lr, void *ws, void *loss, hipStream_t s) {
  const LrLayout L = lr_layout(dtype, nc, n, d);
  char *w = (char *)ws;
  void *R = w + L.r, *G = w + L.g, *RR = w + L.rr, *SK = w + L.sk;
  if (dtype == 0) {
    using H = _Float16;
    return lr_step_nc<H>(nc, dtype, n, d, (const H *)X, (const H *)y_neg, (H *)W, (H)(float)s2n, (H)(float)s1n,
                         (H)(float)neg_lr, (H *)R, (H *)G, (H *)RR, SK, (H *)loss, s);
  }
  if (dtype == 2)
    return lr_step_nc<double>(nc, dtype, n, d, (const double *)X, (const double *)y_neg, (double *)W, s2n, s1n, neg_lr,
                              (double *)R, (double *)G, (double *)RR, SK, (double *)loss, s);
  return lr_step_nc<float>(nc, dtype, n, d, (const float *)X, (const float *)y_neg, (float *)W, (float)s2n, (float)s1n,
                           (float)neg_lr, (float *)R, (float *)G, (float *)RR, SK, (float *)loss, s);
}

}  // namespace mcf

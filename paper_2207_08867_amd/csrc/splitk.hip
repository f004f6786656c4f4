// splitk.hip -- K-split MC matrix product on gfx950 VALU, for reductions that are
// long compared with the number of outputs (Dot-MCN, MV-MCN, small products).
//
// The function computed (fixed by the slice count S alone, not by the launch):
// the reduction steps are dealt round-robin to S slices, slice s taking
// k = s, s + S, s + 2S, ...; each slice is summed in MM-MCN order (ScalingN of its
// first term, then Add-MCN of each further ScalingN term); the S slice sums are then
// combined by a pairwise Add-MCN tree -- at each level entry q of the next level is
// Add-MCN(entry 2q, entry 2q+1) and an odd last entry moves up unchanged.  This is
// the log-depth accumulation that Section 2.2 of the paper names as the cost of an
// accurate N-term MC sum.  MC x MC products are taken by linearity over B's
// components, one K-split product per component, combined left to right.
//
// Launch: a 256-lane workgroup holds 256/KS outputs x KS consecutive slices (KS a
// power of two); lane (output o, slice s) reads A[i][k] and B[k][j] for its own k,
// so the lanes of a slice group read consecutive k.  The first log2(KS) tree levels
// run inside the workgroup (strides < 64 by lane exchange inside a wavefront, 64 and
// 128 through LDS); when S > KS the G = ceil(S/KS) group results go to a workspace
// and a second kernel runs all further levels in one launch: each of its lanes takes an
// aligned block of R consecutive roots (R = 1, 4 or 16, the smallest with G <= 256 R)
// and runs the first log2(R) of those levels in registers, and the lanes then run the
// last levels as in the first kernel.  Because every group and block is an aligned
// block of the level below, a pair of the tree never straddles two of them: the
// result equals the tree's definition for every launch shape.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "mcf_arith.hpp"
#include "mcf_internal.hpp"
#include "mm_steps.hpp"
#include "seq.hpp"

namespace mcf {

constexpr int SK_THREADS = 256;
constexpr int SK_UNROLL = 4;

// Lane exchange inside a wavefront: the value of lane (l + d), for d < 64.  binary16
// values travel as binary32 (exact both ways).
__device__ __forceinline__ float lane_down(float v, int d) { return __shfl_down(v, (unsigned)d, 64); }
__device__ __forceinline__ _Float16 lane_down(_Float16 v, int d) {
  return (_Float16)__shfl_down((float)v, (unsigned)d, 64);
}
__device__ __forceinline__ double lane_down(double v, int d) { return __shfl_down(v, (unsigned)d, 64); }

// Pairwise Add-MCN tree over groups of W lanes (W a power of two, W <= 256): lane q
// of a group holds leaf q, and leaves q >= count are absent.  At stride d the entry of
// lane q (q a multiple of 2d) becomes Add-MCN(entry q, entry q + d) when q + d <
// count, and is unchanged otherwise.  Afterwards lane 0 of each group holds the root.
// Every lane of the workgroup must call this (it contains barriers and exchanges).
template <typename T, int NC, int NP, int APOL>
__device__ __forceinline__ void group_tree(T (&acc)[NP][NC], int q, int W, int count, T (*lds)[NP * NC]) {
  for (int d = 1; d < W; d <<= 1) {
    T other[NP][NC];
    if (d < 64) {
#pragma unroll
      for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int c = 0; c < NC; ++c) other[p][c] = lane_down(acc[p][c], d);
    } else {
      if ((q & (2 * d - 1)) == d) {
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
          for (int c = 0; c < NC; ++c) lds[threadIdx.x][p * NC + c] = acc[p][c];
      }
      __syncthreads();
      if ((q & (2 * d - 1)) == 0 && q + d < count) {
#pragma unroll
        for (int p = 0; p < NP; ++p)
#pragma unroll
          for (int c = 0; c < NC; ++c) other[p][c] = lds[threadIdx.x + d][p * NC + c];
      }
      __syncthreads();
    }
    if ((q & (2 * d - 1)) == 0 && q + d < count) {
#pragma unroll
      for (int p = 0; p < NP; ++p) mm_add<T, NC, APOL>(acc[p], other[p], acc[p]);
    }
  }
}

// Combine the per-component products of B left to right and store one output
// (zero components as +0, Simple-Renorm's padding).
template <typename T, int NC, int NP, int APOL>
__device__ __forceinline__ void sk_store(const T (&acc)[NP][NC], T *__restrict__ C, int64_t MN, int64_t o) {
  T r[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) r[c] = acc[0][c];
#pragma unroll
  for (int p = 1; p < NP; ++p) mm_add<T, NC, APOL>(r, acc[p], r);
#pragma unroll
  for (int c = 0; c < NC; ++c) C[c * MN + o] = (r[c] != T(0)) ? r[c] : T(0);
}

// One MM-MCN term into the accumulators: acc[p] = Add-MCN(acc[p], ScalingN(mc, v_p)).
// FIRST: acc[p] = ScalingN(mc, v_p).
template <typename T, int NC, bool AMC, bool BMC, int SPOL, int APOL, bool FIRST>
__device__ __forceinline__ void sk_term(T (&acc)[(AMC && BMC) ? NC : 1][NC], const T (&a)[AMC ? NC : 1],
                                        const T (&b)[BMC ? NC : 1]) {
  constexpr int NP = (AMC && BMC) ? NC : 1;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const T v = AMC ? b[BMC ? p : 0] : a[0];
    T h[NC + 1];
    if constexpr (AMC)
      scaling_terms<T, NC>(a, v, h);
    else
      scaling_terms<T, NC>(b, v, h);
    if constexpr (FIRST) {
      if (__builtin_expect(sr_try<T, NC, SPOL>(h, acc[p], v == T(0)), 0)) compact_nz<T, NC + 1, NC>(h, acc[p]);
      nonfinite_tail<T, NC>(acc[p]);
    } else {
      T term[NC];
      if (__builtin_expect(sr_try<T, NC, SPOL>(h, term, v == T(0)), 0)) compact_nz<T, NC + 1, NC>(h, term);
      add_terms<T, NC>(acc[p], term, h);
      if (__builtin_expect(sr_try<T, NC, APOL>(h, acc[p]), 0)) compact_nz<T, NC + 1, NC>(h, acc[p]);
    }
  }
}

// Phase 1: slice sums and the in-workgroup tree levels.  A: [NA][M][K], B: [NB][K][N].
// G == 1: the result goes to C [NC][M*N].  G > 1: the group roots go to
// W [G][NP][NC][M*N].
template <typename T, int NC, bool AMC, bool BMC, int SPOL, int APOL>
__global__ __launch_bounds__(SK_THREADS) void sk_kernel(const T *__restrict__ A, const T *__restrict__ B,
                                                        T *__restrict__ C, T *__restrict__ W, int64_t M, int64_t N,
                                                        int64_t K, int64_t S, int KS, int G) {
  constexpr int NA = AMC ? NC : 1;
  constexpr int NB = BMC ? NC : 1;
  constexpr int NP = (AMC && BMC) ? NC : 1;
  __shared__ T lds[SK_THREADS][NP * NC];

  const int64_t MN = M * N;
  const int q = threadIdx.x & (KS - 1);
  const int64_t o = (int64_t)blockIdx.x * (SK_THREADS / KS) + threadIdx.x / KS;
  const int64_t s = (int64_t)blockIdx.y * KS + q;
  const int64_t i = o / N, j = o % N;

  T acc[NP][NC];
#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[p][c] = T(0);

  if (o < MN && s < S) {
    const T *Ai = A + i * K;
    const T *Bj = B + j;
    auto load = [&](int64_t k, T (&a)[NA], T (&b)[NB]) {
#pragma unroll
      for (int c = 0; c < NA; ++c) a[c] = Ai[c * M * K + k];
#pragma unroll
      for (int c = 0; c < NB; ++c) b[c] = Bj[c * K * N + k * N];
    };
    int64_t k = s;
    {
      T a[NA], b[NB];
      load(k, a, b);
      sk_term<T, NC, AMC, BMC, SPOL, APOL, true>(acc, a, b);
      k += S;
    }
    // Loads of SK_UNROLL steps are issued before their arithmetic.
    for (; k + (SK_UNROLL - 1) * S < K; k += SK_UNROLL * S) {
      T a[SK_UNROLL][NA], b[SK_UNROLL][NB];
#pragma unroll
      for (int u = 0; u < SK_UNROLL; ++u) load(k + u * S, a[u], b[u]);
#pragma unroll
      for (int u = 0; u < SK_UNROLL; ++u) sk_term<T, NC, AMC, BMC, SPOL, APOL, false>(acc, a[u], b[u]);
    }
    for (; k < K; k += S) {
      T a[NA], b[NB];
      load(k, a, b);
      sk_term<T, NC, AMC, BMC, SPOL, APOL, false>(acc, a, b);
    }
  }

  const int64_t left = S - (int64_t)blockIdx.y * KS;
  const int count = left < KS ? (int)left : KS;
  group_tree<T, NC, NP, APOL>(acc, q, KS, count, lds);

  if (q == 0 && o < MN) {
    if (G == 1) {
      sk_store<T, NC, NP, APOL>(acc, C, MN, o);
    } else {
#pragma unroll
      for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int c = 0; c < NC; ++c) W[(((int64_t)blockIdx.y * NP + p) * NC + c) * MN + o] = acc[p][c];
    }
  }
}

// Phase 1 for few wavefronts, where a slice's chain of dependent steps sets the time (16 us
// for the 64 steps of a binary32 nc = 2 reduction over 10000 values, whatever else the
// chip does): U steps at a time as one straight line (seq.hpp), the next U steps' loads
// in flight meanwhile, and for MC x MC 256 lanes for each component of B (np), whose
// products are combined at the end.  The same slices, tree and results.
// Columns from N1 on are not in B but in B2, a column after the other.
template <typename T, int NC, int ROLE>
__global__ __attribute__((amdgpu_flat_work_group_size(SK_THREADS, ROLE == SEQ_AMC ? SK_THREADS * NC : SK_THREADS)))
void sk_chain_kernel(const T *__restrict__ A, const T *__restrict__ B, T *__restrict__ C, T *__restrict__ W, int64_t M,
                     int64_t N, int64_t K, int64_t S, int KS, int G, int np, const T *__restrict__ B2, int64_t N1) {
  constexpr int U = seq_unroll<T, NC>();
  extern __shared__ __align__(16) char chain_lds[];
  T(*lds)[NC] = reinterpret_cast<T(*)[NC]>(chain_lds);

  const int64_t MN = M * N;
  const int lane = threadIdx.x & (SK_THREADS - 1), p = threadIdx.x / SK_THREADS;
  const int q = lane & (KS - 1);
  const int64_t o = (int64_t)blockIdx.x * (SK_THREADS / KS) + lane / KS;
  const int64_t s = (int64_t)blockIdx.y * KS + q;
  const bool valid = o < MN && s < S;

  T acc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) acc[c] = T(0);
  if (valid) {
    const int64_t i = o / N, j = o - i * N;
    const int64_t bn = j < N1 ? N1 : 1;
    const T *Ai = A + i * K, *Bj = (j < N1 ? B + j : B2 + (j - N1) * K) + (ROLE == SEQ_AMC ? p * K * N1 : 0);
    const T *xs = ROLE == SEQ_AMC ? Ai : Bj, *vs = ROLE == SEQ_AMC ? Bj : Ai;
    const int64_t xk = ROLE == SEQ_AMC ? 1 : bn, vk = ROLE == SEQ_AMC ? bn : 1;
    const int64_t x_plane = ROLE == SEQ_AMC ? M * K : K * N1;
    using Ops = SeqOps<T, NC, ROLE, U>;
    // steps beyond K are zeros, which leave the accumulator as it is
    auto one = [&](int64_t k, T(&x)[NC], T &v) {
      const bool in = k < K;
      const int64_t kk = in ? k : 0;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        x[c] = xs[c * x_plane + kk * xk];
        x[c] = in ? x[c] : T(0);
      }
      v = vs[kk * vk];
      v = in ? v : T(0);
    };
    auto read = [&](Ops &ops, int64_t k) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        T x[NC];
        one(k + u * S, x, ops.v[u]);
#pragma unroll
        for (int c = 0; c < NC; ++c) ops.x[c][u] = x[c];
      }
    };
    // (binary64: a count in place of a lane mask costs 256 x 1024 nc = 3, plain A 12.9 -> 14.2 us)
    constexpr int LIMIT = sizeof(T) == 4 && NC <= 3 ? 2 : 1;
    std::conditional_t<LIMIT == 1, bool, int> fails = 0;
    auto steps = [&](const Ops &ops, int64_t k) {
      seq_steps<T, NC, ROLE, U, LIMIT, sizeof(T) == 2 && NC == 3>(
          ops, acc, fails, true, k == s,
          [&](Ops &o2) {
            int64_t at = k;
            asm volatile("" : "+v"(at));
            read(o2, at);
          },
          [&](int u, T(&x)[NC], T &v) { one(k + u * S, x, v); });
    };
    Ops o0, o1;
    read(o0, s);
    for (int64_t k = s; k < K; k += 2 * U * S) {
      read(o1, k + U * S);
      steps(o0, k);
      if (k + U * S >= K) break;
      read(o0, k + 2 * U * S);
      steps(o1, k + U * S);
    }
  }

  constexpr int APOL = sizeof(T) >= 4 ? SR_FULL : SR_SELECT;
  const int64_t left = S - (int64_t)blockIdx.y * KS;
  const int count = left < KS ? (int)left : KS;
  T(&acc1)[1][NC] = *reinterpret_cast<T(*)[1][NC]>(&acc);
  group_tree<T, NC, 1, APOL>(acc1, q, KS, count, lds);

  if (G > 1) {
    if (q == 0 && o < MN) {
#pragma unroll
      for (int c = 0; c < NC; ++c) W[(((int64_t)blockIdx.y * np + p) * NC + c) * MN + o] = acc[c];
    }
    return;
  }
  if (np > 1) {
    if (q == 0 && p > 0) {
#pragma unroll
      for (int c = 0; c < NC; ++c) lds[threadIdx.x][c] = acc[c];
    }
    __syncthreads();
  }
  if (q == 0 && p == 0 && o < MN) {
    for (int r = 1; r < np; ++r) {
      T part[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) part[c] = lds[r * SK_THREADS + lane][c];
      mm_add<T, NC, APOL>(acc, part, acc);
    }
    sk_store<T, NC, 1, APOL>(acc1, C, MN, o);
  }
}

// Phase 2: the tree levels above the G group roots of each output in W, in one launch.
// Lane q of an output's GW-lane group takes roots q R .. q R + R - 1 (those below G)
// and folds them in tree order in registers: entry j is pushed after one Add-MCN with
// each completed left neighbour (one per trailing one bit of j), and what is left
// when fewer than R are present combines lowest level first -- an unpaired right
// entry moves up until it meets its left partner, as the tree's rule has it.  The
// lanes then run the last levels as a group tree over ceil(G / R) entries.
template <int R>
struct log2_of {
  static constexpr int value = R <= 1 ? 0 : 1 + log2_of<R / 2>::value;
};
template <>
struct log2_of<1> {
  static constexpr int value = 0;
};

template <typename T, int NC, int NP, int APOL, int R>
__global__ __launch_bounds__(SK_THREADS) void sk_reduce_kernel(const T *__restrict__ W, T *__restrict__ C, int64_t MN,
                                                               int G, int GW) {
  constexpr int L = log2_of<R>::value;
  __shared__ T lds[SK_THREADS][NP * NC];
  const int q = threadIdx.x & (GW - 1);
  const int64_t o = (int64_t)blockIdx.x * (SK_THREADS / GW) + threadIdx.x / GW;
  const int first = q * R;
  const int n = (o < MN && first < G) ? (G - first < R ? G - first : R) : 0;
  // Loads stay in bounds for absent entries (the last root of the last output) so that
  // they can all be issued before the arithmetic; absent entries are never used.
  const int64_t ol = o < MN ? o : MN - 1;
  T stk[L + 1][NP][NC];
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int64_t e = first + j < G ? first + j : G - 1;
    T v[NP][NC];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int c = 0; c < NC; ++c) v[p][c] = W[((e * NP + p) * NC + c) * MN + ol];
    if (j < n) {
      int l = 0;
#pragma unroll
      for (; l < L && ((j >> l) & 1); ++l) {
#pragma unroll
        for (int p = 0; p < NP; ++p) mm_add<T, NC, APOL>(stk[l][p], v[p], v[p]);
      }
#pragma unroll
      for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int c = 0; c < NC; ++c) stk[l][p][c] = v[p][c];
    }
  }
  T acc[NP][NC];
#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[p][c] = T(0);
  bool have = false;
#pragma unroll
  for (int l = 0; l <= L; ++l) {
    if ((n >> l) & 1) {
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        if (have) {
          mm_add<T, NC, APOL>(stk[l][p], acc[p], acc[p]);
        } else {
#pragma unroll
          for (int c = 0; c < NC; ++c) acc[p][c] = stk[l][p][c];
        }
      }
      have = true;
    }
  }
  group_tree<T, NC, NP, APOL>(acc, q, GW, (G + R - 1) / R, lds);
  if (q == 0 && o < MN) sk_store<T, NC, NP, APOL>(acc, C, MN, o);
}

static int pow2_at_least(int64_t v) {
  int p = 1;
  while (p < v) p <<= 1;
  return p;
}

int64_t splitk_default_slices(int64_t M, int64_t N, int64_t K) {
  const int64_t MN = M * N;
  if (MN <= 0 || K <= 0) return 1;
  int64_t s = ((int64_t)SPLITK_TARGET_LANES + MN - 1) / MN;
  const int64_t by_k = K / SPLITK_MIN_STEPS > 1 ? K / SPLITK_MIN_STEPS : 1;
  if (s > by_k) s = by_k;
  if (s > SPLITK_MAX_SLICES) s = SPLITK_MAX_SLICES;
  return s < 1 ? 1 : s;
}

void splitk_shape(int64_t S, int *KS, int *G) {
  const int ks = pow2_at_least(S < SK_THREADS ? S : SK_THREADS);
  *KS = ks;
  *G = (int)((S + ks - 1) / ks);
}

int64_t splitk_roots(int64_t S) {
  int KS, G;
  splitk_shape(S, &KS, &G);
  return G == 1 ? 0 : G;
}

template <typename T, int NC, int NP, int APOL, int R>
static void sk_reduce_launch(const T *W, T *C, int64_t MN, int G, hipStream_t s) {
  const int lanes = (G + R - 1) / R;
  const int GW = pow2_at_least(lanes);
  dim3 grid((unsigned)((MN + (SK_THREADS / GW) - 1) / (SK_THREADS / GW)));
  hipLaunchKernelGGL((sk_reduce_kernel<T, NC, NP, APOL, R>), grid, dim3(SK_THREADS), 0, s, W, C, MN, G, GW);
}

// Up to how many blocks of 256 chains (for each component of B when both operands are MC)
// the chains' latency is what counts, and sk_chain_kernel the faster one; on larger grids
// sk_kernel's higher occupancy keeps more loads in flight.  The block count alone separates
// the two: matrix-vector products with 13 row counts from 1 to 6000 and 9 lengths from 512 to
// 8192, each kernel's time at the last size below a limit and the first above (sk_kernel ->
// sk_chain_kernel, us; in brackets the blocks):
//   MC x MC    f32 nc 2 1536 x 4096 (384) 18.6 -> 15.8, 3000 x 2463 (750) 20.7 -> 26.5; nc 3
//              880 x 4096 (220) 39.2 -> 34.4, 1536 x 2463 (384) 39.6 -> 61.9; nc 4 500 x 8192 (250)
//              82 -> 52, 880 x 4321 (440) 85 -> 94; f64 nc 2 500 x 8192 (250) 20.5 -> 17.7,
//              1536 x 2463 (384) 22.3 -> 29.3; nc 3 880 x 4096 (220) 47.9 -> 38.0, 1536 x 2463 58.1 -> 66.8
//              f16 nc 2 6000 x 4096 (1500) 54 -> 47, nc 3 3000 x 8192 (1500) 137 -> 138
//   MC, plain  f32 nc 3 500 x 8192 (250) 21.0 -> 14.1, 1536 x 4321 (768) 19.8 -> 24.4; f64 nc 3
//              880 x 4096 (220) 20.3 -> 16.2, 1536 x 2463 (384) 23.5 -> 25.3
//   plain, MC  f32 nc 3 880 x 4321 (440) 18.2 -> 16.5, 3000 x 2463 (750) 19.0 -> 21.1; f64 nc 3
//              500 x 8192 (250) 19.2 -> 15.7, 1536 x 2463 (384) 23.0 -> 24.7
// nc = 1 (two operations a step) gains nothing, nor does binary16 nc = 2 with one MC operand;
// binary32 nc = 4 with one MC operand loses (22 -> 30 us at 16 slices of 64 steps): the
// components beyond what a binary64 value fills are zero or nearly, and its short slices
// start with many general steps.  And where a few of few slices have one step more than the
// others' whole groups (binary32, one MC operand: 64 x 577, nc = 3, 9 slices 15.2 -> 17.3 us;
// 64 x 576 14.7 -> 10.6, 64 x 608 15.3 -> 13.0), those lanes wait by themselves.
static bool sk_chain_wanted(int size, int nc, bool a_mc, bool b_mc, int64_t blocks, int64_t K, int64_t S) {
  const bool both = a_mc && b_mc;
  if (nc == 1 || (size == 4 && nc == 4 && !both)) return false;
  if (size == 2) return both ? blocks * nc <= 4096 : (nc >= 3 && blocks <= 512);
  if (size == 8) return blocks <= 256;
  if (both) return blocks <= (nc == 2 ? 384 : 256);
  if (S <= 24 && K / S % 8 == 0 && K % S != 0 && 4 * (K % S) < S) return false;
  return blocks <= (a_mc ? 256 : 512);
}

template <typename T, int NC, bool AMC, bool BMC>
static hipError_t sk_launch(int64_t M, int64_t N, int64_t K, const void *A, const void *B, int64_t S, void *W, void *C,
                            hipStream_t s) {
  constexpr int NP = (AMC && BMC) ? NC : 1;
  // Simple-Renorm fast-path policies as in the sequential product (they change speed only)
  constexpr int SPOL = sizeof(T) >= 4 ? SR_FULL : (NC == 2 ? SR_NET : SR_HEAD);
  constexpr int APOL = sizeof(T) >= 4 ? SR_FULL : SR_SELECT;
  const int64_t MN = M * N;
  int KS, G;
  splitk_shape(S, &KS, &G);
  // S <= SPLITK_MAX_SLICES = 2^20 gives G <= 4096 = 16 x 256 group roots.
  if (G > 16 * SK_THREADS) return hipErrorInvalidValue;
  dim3 grid((unsigned)((MN + (SK_THREADS / KS) - 1) / (SK_THREADS / KS)), (unsigned)G);
  if (sk_chain_wanted(sizeof(T), NC, AMC, BMC, (int64_t)grid.x * G, K, S)) {
    constexpr int ROLE = AMC ? SEQ_AMC : SEQ_BMC;
    hipLaunchKernelGGL((sk_chain_kernel<T, NC, ROLE>), grid, dim3(SK_THREADS * NP), SK_THREADS * NP * NC * sizeof(T), s,
                       (const T *)A, (const T *)B, (T *)C, (T *)W, M, N, K, S, KS, G, NP, (const T *)nullptr, N);
  } else {
    hipLaunchKernelGGL((sk_kernel<T, NC, AMC, BMC, SPOL, APOL>), grid, dim3(SK_THREADS), 0, s, (const T *)A,
                       (const T *)B, (T *)C, (T *)W, M, N, K, S, KS, G);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || G == 1) return e;
  // W: the G group roots.
  if (G <= SK_THREADS)
    sk_reduce_launch<T, NC, NP, APOL, 1>((const T *)W, (T *)C, MN, G, s);
  else if (G <= 4 * SK_THREADS)
    sk_reduce_launch<T, NC, NP, APOL, 4>((const T *)W, (T *)C, MN, G, s);
  else
    sk_reduce_launch<T, NC, NP, APOL, 16>((const T *)W, (T *)C, MN, G, s);
  return hipGetLastError();
}

template <typename T, int NC>
static hipError_t sk_kinds(int64_t M, int64_t N, int64_t K, const void *A, int a_mc, const void *B, int b_mc,
                           int64_t S, void *W, void *C, hipStream_t s) {
  if (a_mc && b_mc) return sk_launch<T, NC, true, true>(M, N, K, A, B, S, W, C, s);
  if (a_mc) return sk_launch<T, NC, true, false>(M, N, K, A, B, S, W, C, s);
  return sk_launch<T, NC, false, true>(M, N, K, A, B, S, W, C, s);
}

template <typename T>
static hipError_t sk_dispatch(int nc, int64_t M, int64_t N, int64_t K, const void *A, int a_mc, const void *B,
                              int b_mc, int64_t S, void *W, void *C, hipStream_t s) {
  switch (nc) {
    case 1: return sk_kinds<T, 1>(M, N, K, A, a_mc, B, b_mc, S, W, C, s);
    case 2: return sk_kinds<T, 2>(M, N, K, A, a_mc, B, b_mc, S, W, C, s);
    case 3: return sk_kinds<T, 3>(M, N, K, A, a_mc, B, b_mc, S, W, C, s);
    case 4: return sk_kinds<T, 4>(M, N, K, A, a_mc, B, b_mc, S, W, C, s);
  }
  return hipErrorInvalidValue;
}

// The sums of one linear-regression step in one launch: C = r^T [X | r^(0) | r^(1) | ...],
// [nc][d + nc], the K-split products of the MC residual r [nc][n] with the columns of X
// [n][d] and with its own components, S <= 256 slices (one group: no workspace).
template <typename T, int NC>
static hipError_t lr_sums(int64_t n, int64_t d, const void *X, const void *R, int64_t S, void *C, hipStream_t s) {
  int KS, G;
  splitk_shape(S, &KS, &G);
  if (G != 1) return hipErrorInvalidValue;
  const unsigned per = SK_THREADS / KS, blocks = (unsigned)((d + NC + per - 1) / per);
  hipLaunchKernelGGL((sk_chain_kernel<T, NC, SEQ_AMC>), dim3(blocks), dim3(SK_THREADS), SK_THREADS * NC * sizeof(T), s,
                     (const T *)R, (const T *)X, (T *)C, (T *)nullptr, (int64_t)1, d + NC, n, S, KS, G, 1, (const T *)R,
                     d);
  return hipGetLastError();
}

template <typename T>
static hipError_t lr_sums_nc(int nc, int64_t n, int64_t d, const void *X, const void *R, int64_t S, void *C,
                             hipStream_t s) {
  switch (nc) {
    case 1: return lr_sums<T, 1>(n, d, X, R, S, C, s);
    case 2: return lr_sums<T, 2>(n, d, X, R, S, C, s);
    case 3: return lr_sums<T, 3>(n, d, X, R, S, C, s);
    case 4: return lr_sums<T, 4>(n, d, X, R, S, C, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_linreg_sums(int dtype, int nc, int64_t n, int64_t d, const void *X, const void *R, int64_t S, void *C,
                              hipStream_t s) {
  if (dtype == 0) return lr_sums_nc<_Float16>(nc, n, d, X, R, S, C, s);
  if (dtype == 2) return lr_sums_nc<double>(nc, n, d, X, R, S, C, s);
  return lr_sums_nc<float>(nc, n, d, X, R, S, C, s);
}

hipError_t launch_matmul_splitk(int dtype, int nc, int64_t M, int64_t N, int64_t K, const void *A, int a_mc,
                                const void *B, int b_mc, int64_t S, void *W, void *C, hipStream_t stream) {
  if (dtype == 0) return sk_dispatch<_Float16>(nc, M, N, K, A, a_mc, B, b_mc, S, W, C, stream);
  if (dtype == 2) return sk_dispatch<double>(nc, M, N, K, A, a_mc, B, b_mc, S, W, C, stream);
  return sk_dispatch<float>(nc, M, N, K, A, a_mc, B, b_mc, S, W, C, stream);
}

// Static scratch of the allocation-free K-split entry point: the partial tree roots
// of one call live here instead of in a caller workspace.  Each device holds its own
// copy for the life of the process.  In host code `scratch` names a host-side
// stand-in, not device memory: the device address is looked up once per device with
// hipGetSymbolAddress and only that address is ever passed to a kernel.
__device__ __align__(256) unsigned char scratch[SPLITK_SCRATCH_BYTES];

namespace {
constexpr int SCRATCH_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[SCRATCH_MAX_DEVICES] = {};
}  // namespace

// Device address of `scratch` on the device that runs `stream` (the current device
// for the null stream); the lookup runs with that device current, once per device.
hipError_t splitk_scratch(hipStream_t stream, void **ptr) {
  int dev = 0, cur = 0;
  hipError_t e = hipGetDevice(&cur);
  if (e != hipSuccess) return e;
  dev = cur;
  if (stream != nullptr) {
    e = hipStreamGetDevice(stream, &dev);
    if (e != hipSuccess) return e;
  }
  if (dev < 0 || dev >= SCRATCH_MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    if (dev != cur && (e = hipSetDevice(dev)) != hipSuccess) return e;
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (dev != cur) {
      const hipError_t r = hipSetDevice(cur);
      if (e == hipSuccess) e = r;
    }
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace mcf

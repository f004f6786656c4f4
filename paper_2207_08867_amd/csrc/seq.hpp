// seq.hpp -- the sequential MC product (MM-MCN) for grids of few wavefronts.
//
// Every output is a chain of K dependent Add-MCN steps that its definition forbids to
// split, so with few outputs the time is K times the latency of one step.  What the
// chain itself needs is short: component c of the next accumulator waits for one or two
// additions on component c of this one, and everything else (the products, the error
// terms) can run ahead.  mm_kernel (matmul.hip) cannot use that: it tests Simple-Renorm's
// common case and branches after every ScalingN and Add-MCN, and nothing is scheduled
// across a branch, so each step pays its whole operation chain, its LDS reads and two
// branches (about 450 clocks at nc = 2, one wavefront per SIMD).  Here
//   * U steps run as one straight line on the assumption that every Simple-Renorm keeps
//     its leading nc terms; one test per U steps covers all of them, and a lane that
//     fails restores its accumulator and redoes the U steps with the general algorithm;
//   * the operands of the next U steps are read from LDS (16 bytes at a time: both tiles
//     are stored with k contiguous) before the current U steps run;
//   * the tiles are double-buffered: one barrier per 128 / sizeof(T) steps;
//   * MC x MC: the nc products A B^(p) are independent chains, so each has wavefronts of
//     its own (a workgroup of 256 nc lanes) and they are combined at the end;
//   * the workgroup's 256 outputs form a TY x TX block whose shape is chosen at launch to
//     waste the fewest lanes on the edges (N = 50 in 16 columns wastes 22%, in 8 columns
//     11%).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "mcf_arith.hpp"
#include "mcf_internal.hpp"
#include "mm_steps.hpp"

namespace mcf {

constexpr int SEQ_ROW_BYTES = 128;                 // a tile row: 128 / sizeof(T) steps of one row or column
constexpr int SEQ_STRIDE = SEQ_ROW_BYTES + 16;     // in LDS, padded: 16-byte reads of 8 rows meet no bank twice
constexpr int SEQ_VECS = SEQ_ROW_BYTES / 16;       // 16-byte pieces of a tile row
constexpr int SEQ_LANES = 256;                     // outputs per workgroup

// Which operand is MC.  SEQ_PLAIN: neither; the term of step k is the exact product
// (p, e, 0, ...) of two plain values -- what ScalingN of (x, 0, ..., 0) by v returns.
enum SeqRole { SEQ_AMC = 0, SEQ_BMC = 1, SEQ_PLAIN = 2 };

template <typename T>
struct SeqArgs {
  const T *A, *B, *y;
  T *C;
  int64_t M, N, K;
  int64_t a_plane, b_plane, c_plane, y_plane, y_ld;
  int64_t a_ld, b_ld;  // rows of A and B as stored (see AT / BT)
  int64_t B2, bb0, a_s1, a_s2, b_s1, b_s2;
  int np;     // planes of the plain side, each a product of its own (MC x MC: nc), else 1
  int tx_log; // TX = 1 << tx_log columns by 256 / TX rows per workgroup
  uint32_t tile0;  // the launch's first tile
  int vec_a, vec_b;  // 16-byte loads are aligned and never cross an edge
  int mode;   // epilogue, as MmArgs
  T alpha, beta;
  // When last is given, column N - 1 of B is not stored: it holds ones, and that column
  // of the result goes to `last` (nc planes of M).
  T *last;
};

typedef unsigned int seq_u32x4 __attribute__((ext_vector_type(4)));

// The smallest of a set of values' magnitudes, for a test whether one of them is zero.
// binary64 compares the high words' bits (in order like the magnitudes), so a magnitude
// below 2^-1042 counts as zero too: the redo that follows gives the same result.
template <typename T>
struct SeqLow {
  float v = 1.0f;
  __device__ __forceinline__ void add(T h) { v = __builtin_fminf(v, __builtin_fabsf((float)h)); }
  __device__ __forceinline__ bool zero() const { return v == 0.0f; }
};
template <>
struct SeqLow<double> {
  unsigned v = ~0u;
  __device__ __forceinline__ void add(double h) {
    const unsigned m = (unsigned)((unsigned long long)__double_as_longlong(h) >> 32) << 1;
    v = m < v ? m : v;
  }
  __device__ __forceinline__ bool zero() const { return v == 0; }
};

// Steps per test (16-byte multiples; nc = 4 would spill its two sets of operands at 8).
template <typename T, int NC>
constexpr int seq_unroll() {
  return sizeof(T) == 2 ? 8 : (sizeof(T) == 4 && NC <= 3 ? 8 : 4);
}

// The U = VW * NV operand values of consecutive steps of one LDS row.
template <typename T, int U>
__device__ __forceinline__ void seq_read(const char *row, T (&out)[U]) {
  constexpr int VW = 16 / (int)sizeof(T);
  static_assert(U % VW == 0, "");
#pragma unroll
  for (int i = 0; i < U / VW; ++i) {
    const seq_u32x4 r = *reinterpret_cast<const seq_u32x4 *>(row + 16 * i);
    __builtin_memcpy(&out[i * VW], &r, 16);
  }
}

template <typename T, int NC, int ROLE, int U>
struct SeqOps {
  static constexpr int NX = ROLE == SEQ_PLAIN ? 1 : NC;
  T x[NX][U], v[U];
};

// The term of one step in full (Simple-Renorm by the general compaction).
template <typename T, int NC, int ROLE>
__device__ __forceinline__ void seq_term_general(const T (&x)[ROLE == SEQ_PLAIN ? 1 : NC], T v, T (&t)[NC]) {
  if constexpr (ROLE == SEQ_PLAIN) {
    plain_term<T, NC>(x[0], v, t);
  } else {
    T h[NC + 1];
    scaling_terms<T, NC>(x, v, h);
    compact_nz<T, NC + 1, NC>(h, t);
  }
}

// U steps on the assumption that every Simple-Renorm keeps its first nc terms; true when
// that may fail for a lane.  Two tests:
//   STRICT = false: no kept term is zero (one running minimum of magnitudes, and one
//     branch per U steps).  Enough for dense binary32 and binary64 values.
//   STRICT: kept_invalid's, which accepts zeros that trail: binary16, whose low terms fall
//     below its subnormal grid, and values with zero low components or plain factors.
// nc = 1 needs no test: a zero sum or product is exact.
template <typename T, int NC, int ROLE, int U, bool STRICT>
__device__ __forceinline__ bool seq_group(const SeqOps<T, NC, ROLE, U> &o, T (&acc)[NC]) {
  SeqLow<T> low;
  uint64_t bad = 0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    T t[NC], s[NC], last;
    const T v = o.v[u];
    if constexpr (ROLE == SEQ_PLAIN) {
      const T x[1] = {o.x[0][u]};
      seq_term_general<T, NC, ROLE>(x, v, t);
    } else {
      T x[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) x[c] = o.x[c][u];
      scaling_kept<T, NC, false, false>(x, v, t, last);
      if constexpr (NC > 1 && STRICT) bad |= kept_invalid_mask<T, NC, false, sizeof(T) == 2>(t, last);
      if constexpr (NC > 1 && !STRICT) {
#pragma unroll
        for (int c = 0; c < NC; ++c) low.add(t[c]);
      }
    }
    add_kept<T, NC>(acc, t, s, last);
    if constexpr (NC > 1 && STRICT) bad |= kept_invalid_mask<T, NC, false>(s, last);
    if constexpr (NC > 1 && !STRICT) {
#pragma unroll
      for (int c = 0; c < NC; ++c) low.add(s[c]);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = s[c];
  }
  if constexpr (NC == 1) return false;
  if constexpr (STRICT) return (bad >> (threadIdx.x & 63)) & 1;
  return low.zero();
}

// One step by the general algorithm.
template <typename T, int NC, int ROLE>
__device__ __forceinline__ void seq_general(const T (&x)[ROLE == SEQ_PLAIN ? 1 : NC], T v, T (&acc)[NC]) {
  T t[NC], h[NC + 1];
  seq_term_general<T, NC, ROLE>(x, v, t);
  add_terms<T, NC>(acc, t, h);
  compact_nz<T, NC + 1, NC>(h, acc);
}

// U steps into acc: the straight line, then the general algorithm for lanes that fail.
// again(o2) reads the operands again (binary32 and binary64, for the strict test), from
// somewhere the compiler cannot know, or it would keep the terms of the first attempt in
// registers; one(u, x, v) reads those of step u (HELD: the general algorithm takes the
// group's operands from registers, where a read is a trip to memory).  valid: the lane's
// result is wanted; first: these are the first steps of the reduction.
// fails: the wavefront's state, how many of its groups failed the first test.  After LIMIT
// it stays with the strict test: two, since what fails again is a property of its data, and
// one alone is a term that came out zero by chance; a wavefront that left the first test
// for it would be the slowest of the grid (256^2 x 256 binary32 nc = 3, plain A: 43 us when the
// first failure counted, 31 us now).  With LIMIT = 1 a bool, tested as one: it stays a lane mask.
template <typename T, int NC, int ROLE, int U, int LIMIT, bool HELD = false, typename Fails, typename Again, typename One>
__device__ __forceinline__ void seq_steps(const SeqOps<T, NC, ROLE, U> &o, T (&acc)[NC], Fails &fails, bool valid,
                                          bool first, const Again &again, const One &one) {
  constexpr int NX = SeqOps<T, NC, ROLE, U>::NX;
  T saved[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) saved[c] = acc[c];
  bool bad;
  if constexpr (sizeof(T) == 2) {
    bad = seq_group<T, NC, ROLE, U, true>(o, acc);
  } else {
    if (LIMIT == 1 ? !fails : fails < LIMIT) {
      bad = seq_group<T, NC, ROLE, U, false>(o, acc);
      if (__builtin_expect(NC == 1 || !__any(bad && valid), 1)) return;
      // (not counted: the first steps of plain factors, whose accumulator has no third
      // component yet)
      const bool counted = ROLE != SEQ_PLAIN || !first;
      if constexpr (LIMIT == 1)
        fails = counted;
      else
        fails += counted;
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[c] = saved[c];
    }
    SeqOps<T, NC, ROLE, U> o2;
    again(o2);
    bad = seq_group<T, NC, ROLE, U, true>(o2, acc);
  }
  if (NC > 1 && __builtin_expect(bad && valid, 0)) {
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = saved[c];
    if constexpr (HELD) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        T x[NX];
#pragma unroll
        for (int c = 0; c < NX; ++c) x[c] = o.x[c][u];
        seq_general<T, NC, ROLE>(x, o.v[u], acc);
      }
    } else {
#pragma unroll 1
      for (int u = 0; u < U; ++u) {
        T x[NX], v;
        one(u, x, v);
        seq_general<T, NC, ROLE>(x, v, acc);
      }
    }
  }
}

// One lane's piece of a plane's tile: 16 bytes along the contiguous dimension of an
// operand stored [rows][K] (KC) or [K][rows].
// ANY: rows of ragged sizes.  A piece is one 16-byte load wherever 16 bytes from its start lie
// inside the matrix, at any alignment (the ISA allows it).  binary16 only: a load per element
// costs it eight a piece (711 x 1803 x 196 nc = 1 48 us against 26), binary32 and binary64,
// with four and two, gain nothing.
template <typename T, bool KC, bool ANY>
struct SeqPiece {
  static constexpr int VW = 16 / (int)sizeof(T);
  int row, k, rows;  // first tile row and step of the piece; rows of it inside the operand
  bool active;
  bool spare;      // ANY: elements of the next stored row follow this one's, VW or more (!KC: if there is one)
  int64_t offset;  // of the piece from the operand's plane
  __device__ __forceinline__ SeqPiece(int lane, int rows_log, int64_t r0, int64_t limit, int64_t ld) {
    if constexpr (KC) {
      row = lane / SEQ_VECS;
      k = (lane % SEQ_VECS) * VW;
    } else {
      row = (lane & ((1 << rows_log) / VW - 1)) * VW;
      k = lane / ((1 << rows_log) / VW);
    }
    active = lane < (SEQ_VECS << rows_log);
    const int64_t left = limit - (r0 + row);
    const int most = KC ? 1 : VW;
    rows = !active || left <= 0 ? 0 : (left < most ? (int)left : most);
    spare = ld >= VW && (!KC || left > 1);
    offset = KC ? (r0 + row) * ld + k : (int64_t)k * ld + r0 + row;
  }
  // The piece at src, k_left steps before the end of the reduction, zeros outside the
  // operand (ANY: any values for rows outside it, whose outputs are not wanted).  vec: a
  // 16-byte load is aligned wherever it lies inside the operand.  one: the element that
  // holds one instead (VW: none).
  __device__ __forceinline__ seq_u32x4 load(const T *src, int64_t k_left, bool vec, int one) const {
    const int64_t left = k_left - k;
    const int n = rows == 0 || left <= 0 ? 0 : (KC ? (left < VW ? (int)left : VW) : rows);
    seq_u32x4 r = {0, 0, 0, 0};
    if (ANY ? n == VW || (n > 0 && spare && (KC || left > 1)) : vec && n == VW) {
      if constexpr (ANY) {
        __builtin_memcpy(&r, src, 16);
        if ((KC && n < VW) || (!KC && one < VW)) {
          T e[VW];
          __builtin_memcpy(e, &r, 16);
#pragma unroll
          for (int i = 0; i < VW; ++i) e[i] = KC ? (i < n ? e[i] : T(0)) : (i == one ? T(1) : e[i]);
          __builtin_memcpy(&r, e, 16);
        }
      } else {
        r = *reinterpret_cast<const seq_u32x4 *>(src);
      }
    } else if (n > 0 || (!KC && one < VW)) {
      T e[VW];
#pragma unroll
      for (int i = 0; i < VW; ++i) e[i] = i < n ? src[i] : T(0);
      if constexpr (!KC) {
#pragma unroll
        for (int i = 0; i < VW; ++i) e[i] = i == one && left > 0 ? T(1) : e[i];
      }
      __builtin_memcpy(&r, e, 16);
    }
    return r;
  }
  // to: the plane's tile in LDS
  __device__ __forceinline__ void store(char *to, const seq_u32x4 &r) const {
    if (!active) return;
    char *at = to + row * SEQ_STRIDE + k * (int)sizeof(T);
    if constexpr (KC) {
      *reinterpret_cast<seq_u32x4 *>(at) = r;
    } else {
      T e[VW];
      __builtin_memcpy(e, &r, 16);
#pragma unroll
      for (int i = 0; i < VW; ++i) *reinterpret_cast<T *>(at + i * SEQ_STRIDE) = e[i];
    }
  }
};

// AT: A is stored [K][M] (rows a_ld apart) instead of [M][K]; BT: B is stored [N][K]
// instead of [K][N].
template <typename T, int NC, int ROLE, bool AT, bool BT, bool ANY>
__global__ __attribute__((amdgpu_flat_work_group_size(SEQ_LANES, ROLE == SEQ_AMC ? SEQ_LANES * NC : SEQ_LANES))) void
seq_kernel(const SeqArgs<T> g) {
  constexpr int VW = 16 / (int)sizeof(T);
  constexpr int KT = SEQ_ROW_BYTES / (int)sizeof(T);
  constexpr int U = seq_unroll<T, NC>();
  constexpr int NA = ROLE == SEQ_AMC ? NC : 1;
  constexpr int NX = ROLE == SEQ_PLAIN ? 1 : NC;
  const int nb = ROLE == SEQ_BMC ? NC : g.np;
  extern __shared__ __align__(16) char lds[];

  const int tx_log = g.tx_log, ty_log = 8 - g.tx_log;
  const int BN = 1 << tx_log, BM = 1 << ty_log;
  const int lane = threadIdx.x & (SEQ_LANES - 1), p = threadIdx.x / SEQ_LANES;
  const int tx = lane & (BN - 1), ty = lane >> tx_log;
  const uint32_t gx = (uint32_t)((g.N + BN - 1) >> tx_log);
  const uint32_t tile = g.tile0 + blockIdx.x;
  const int64_t m0 = (int64_t)(tile / gx) << ty_log, n0 = (int64_t)(tile % gx) << tx_log;
  const T *A = g.A, *B = g.B;
  const int64_t bb = g.bb0 + blockIdx.y;
  if (bb != 0) {
    const int64_t i1 = bb / g.B2, i2 = bb - i1 * g.B2;
    A += i1 * g.a_s1 + i2 * g.a_s2;
    B += i1 * g.b_s1 + i2 * g.b_s2;
  }
  const int64_t K = g.K, n_stored = g.last ? g.N - 1 : g.N;

  // Staging.  A tile holds NA planes of BM rows of A and nb planes of BN columns of B.
  // A plane's tile is at most 32 rows = 256 pieces of 16 bytes along the operand's
  // contiguous dimension, one per lane of a 256-lane group; group p stages the planes of
  // A that are p modulo np, and plane p of B (every plane when np is 1).
  constexpr int NBS = ROLE == SEQ_BMC ? NC : 1;
  const SeqPiece<T, !AT, ANY> pa(lane, ty_log, m0, g.M, g.a_ld);
  const SeqPiece<T, BT, ANY> pb(lane, tx_log, n0, n_stored, g.b_ld);
  // column of ones: element `one` of this lane's piece of B
  const int one = !BT && g.last != nullptr && pb.active && n_stored >= n0 + pb.row && n_stored < n0 + pb.row + VW
                      ? (int)(n_stored - n0) - pb.row
                      : VW;
  const T *src_a = A + pa.offset, *src_b = B + pb.offset + (ROLE == SEQ_BMC ? 0 : p * g.b_plane);
  const int buf_bytes = (NA * BM + nb * BN) * SEQ_STRIDE;
  const int b_tile = NA * BM * SEQ_STRIDE + (ROLE == SEQ_BMC ? 0 : p * BN * SEQ_STRIDE);
  seq_u32x4 reg_a[NA], reg_b[NBS];
  auto fetch = [&](int64_t k0) {
#pragma unroll
    for (int c = 0; c < NA; ++c)
      if (g.np == 1 || c % g.np == p) reg_a[c] = pa.load(src_a + c * g.a_plane, K - k0, g.vec_a, VW);
#pragma unroll
    for (int c = 0; c < NBS; ++c) reg_b[c] = pb.load(src_b + c * g.b_plane, K - k0, g.vec_b, one);
    src_a += AT ? (int64_t)KT * g.a_ld : (int64_t)KT;
    src_b += BT ? (int64_t)KT : (int64_t)KT * g.b_ld;
  };
  auto store = [&](int buf) {
    char *to = lds + buf * buf_bytes;
#pragma unroll
    for (int c = 0; c < NA; ++c)
      if (g.np == 1 || c % g.np == p) pa.store(to + c * BM * SEQ_STRIDE, reg_a[c]);
#pragma unroll
    for (int c = 0; c < NBS; ++c) pb.store(to + b_tile + c * BN * SEQ_STRIDE, reg_b[c]);
  };

  // LDS rows of this lane: the MC side's planes (xs, x_step apart) and its plain factor.
  const int row_a = ty, row_b = (NA << ty_log) + tx;
  const int xs = (ROLE == SEQ_BMC ? row_b : row_a) * SEQ_STRIDE;
  const int x_step = (ROLE == SEQ_BMC ? BN : BM) * SEQ_STRIDE;
  const int vs = (ROLE == SEQ_BMC ? row_a : row_b + (p << tx_log)) * SEQ_STRIDE;
  const int64_t gm = m0 + ty, gn = n0 + tx;
  const bool valid = gm < g.M && gn < g.N;

  T acc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) acc[c] = T(0);  // Add-MCN(0, t) = t for the first term

  if (K > 0) {
    fetch(0);
    store(0);
  }
  __syncthreads();
  int buf = 0;
  constexpr int LIMIT = sizeof(T) == 4 && NC == 4 ? 1 : 2;  // (nc = 4: what fails first is an empty fourth component)
  std::conditional_t<LIMIT == 1, bool, int> fails = 0;
  for (int64_t k0 = 0; k0 < K; k0 += KT, buf ^= 1) {
    const bool more = k0 + KT < K;
    if (more) fetch(k0 + KT);
    const int kt = (int)(K - k0 < KT ? K - k0 : KT);
    const char *from = lds + buf * buf_bytes;
    using Ops = SeqOps<T, NC, ROLE, U>;
    auto read = [&](Ops &o, int kk) {
      const char *at = from + kk * (int)sizeof(T);
#pragma unroll
      for (int c = 0; c < NX; ++c) seq_read<T, U>(at + xs + c * x_step, o.x[c]);
      seq_read<T, U>(at + vs, o.v);
    };
    auto steps = [&](const Ops &o, int kk) {
      seq_steps<T, NC, ROLE, U, LIMIT>(
          o, acc, fails, valid, k0 + kk == 0,
          [&](Ops &o2) {
            int at = kk;
            asm volatile("" : "+s"(at));
            read(o2, at);
          },
          [&](int u, T(&x)[NX], T &v) {
            const char *at = from + (kk + u) * (int)sizeof(T);
#pragma unroll
            for (int c = 0; c < NX; ++c) x[c] = *reinterpret_cast<const T *>(at + xs + c * x_step);
            v = *reinterpret_cast<const T *>(at + vs);
          });
    };
    // steps beyond K multiply zeros and leave the accumulator as it is
    Ops o0, o1;
    read(o0, 0);
    for (int kk = 0; kk < kt; kk += 2 * U) {
      read(o1, kk + U);  // (kk + U < KT: a tile holds an even number of groups)
      steps(o0, kk);
      if (kk + U >= kt) break;
      if (kk + 2 * U < kt) read(o0, kk + 2 * U);
      steps(o1, kk + U);
    }
    if (more) {
      store(buf ^ 1);
      __syncthreads();
    }
  }

  // MC x MC: the products of B's components are combined left to right.
  if (ROLE == SEQ_AMC && g.np > 1) {
    __syncthreads();
    T *parts = reinterpret_cast<T *>(lds);
    if (p > 0) {
#pragma unroll
      for (int c = 0; c < NC; ++c) parts[((p - 1) * NC + c) * SEQ_LANES + lane] = acc[c];
    }
    __syncthreads();
    if (p > 0) return;
    for (int q = 1; q < g.np; ++q) {
      T other[NC], h[NC + 1];
#pragma unroll
      for (int c = 0; c < NC; ++c) other[c] = parts[((q - 1) * NC + c) * SEQ_LANES + lane];
      add_terms<T, NC>(acc, other, h);
      compact_nz<T, NC + 1, NC>(h, acc);
    }
  }
  if (!valid) return;
  if (g.mode != 0) {
    T yv[NC], h[NC + 1];
#pragma unroll
    for (int c = 0; c < NC; ++c) yv[c] = g.y[c * g.y_plane + gm * g.y_ld + gn];
    if (g.mode == 2) {  // AddMM-MCN: both operands scaled first (ScalingN, expand off)
      scaling_n<T, NC, NC>(acc, g.alpha, acc);
      scaling_n<T, NC, NC>(yv, g.beta, yv);
    }
    add_terms<T, NC>(acc, yv, h);
    compact_nz<T, NC + 1, NC>(h, acc);
  }
  // zero components leave as +0, Simple-Renorm's padding
  if (g.last != nullptr && gn == g.N - 1) {
#pragma unroll
    for (int c = 0; c < NC; ++c) g.last[c * g.M + gm] = (acc[c] != T(0)) ? acc[c] : T(0);
  } else {
    T *out = g.C + bb * g.M * g.N + gm * n_stored + gn;
#pragma unroll
    for (int c = 0; c < NC; ++c) out[c * g.c_plane] = (acc[c] != T(0)) ? acc[c] : T(0);
  }
}

// ---------------------------------------------------------------------------------
// Launch
// ---------------------------------------------------------------------------------

// Block shape: the 8, 16 or 32 columns (by 32, 16 or 8 rows) that leave the fewest lanes
// outside the result; the widest of equals.
inline int seq_tx_log(int64_t M, int64_t N) {
  int best = 5;
  int64_t least = INT64_MAX;
  for (int l = 5; l >= 3; --l) {
    const int64_t bn = (int64_t)1 << l, bm = SEQ_LANES / bn;
    const int64_t blocks = (M + bm - 1) / bm * ((N + bn - 1) / bn);
    if (blocks < least) {
      best = l;
      least = blocks;
    }
  }
  return best;
}

template <typename T, int NC, int ROLE, bool AT, bool BT>
hipError_t seq_launch(SeqArgs<T> g, int64_t batches, hipStream_t s) {
  constexpr int VW = 16 / (int)sizeof(T);
  g.tx_log = seq_tx_log(g.M, g.N);
  const int bn = 1 << g.tx_log, bm = SEQ_LANES / bn;
  auto mult = [](int64_t v) { return v % VW == 0; };
  g.vec_a = mult(g.a_ld) && mult(g.a_plane) && mult(g.a_s1) && mult(g.a_s2) && (uintptr_t)g.A % 16 == 0;
  g.vec_b = mult(g.b_ld) && mult(g.b_plane) && mult(g.b_s1) && mult(g.b_s2) && (uintptr_t)g.B % 16 == 0;
  const int rows = (ROLE == SEQ_AMC ? NC : 1) * bm + (ROLE == SEQ_BMC ? NC : g.np) * bn;
  int lds = 2 * rows * SEQ_STRIDE;
  const int parts = (g.np - 1) * NC * SEQ_LANES * (int)sizeof(T);
  if (parts > lds) lds = parts;
  const int64_t tiles = ((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn);
  // batches go to grid y, tiles to grid x; a launch holds fewer than 2^32 lanes along x, so
  // results of one component with 2^31 outputs or more take several
  const int64_t most = ((int64_t)1 << 31) / (SEQ_LANES * g.np);
  for (int64_t b0 = 0; b0 < batches; b0 += 65535) {
    g.bb0 = b0;
    const unsigned nb = (unsigned)(batches - b0 < 65535 ? batches - b0 : 65535);
    for (int64_t t0 = 0; t0 < tiles; t0 += most) {
      g.tile0 = (uint32_t)t0;
      const unsigned nt = (unsigned)(tiles - t0 < most ? tiles - t0 : most);
      if (sizeof(T) == 2 && !(g.vec_a && g.vec_b))
        hipLaunchKernelGGL((seq_kernel<T, NC, ROLE, AT, BT, sizeof(T) == 2>), dim3(nt, nb), dim3(SEQ_LANES * g.np), lds, s,
                           g);
      else
        hipLaunchKernelGGL((seq_kernel<T, NC, ROLE, AT, BT, false>), dim3(nt, nb), dim3(SEQ_LANES * g.np), lds, s, g);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

template <typename T, int NC>
hipError_t seq_kinds(const SeqArgs<T> &g, int64_t batches, int a_mc, int b_mc, int a_trans, int b_trans,
                     hipStream_t s) {
  if (a_trans) {  // MC-Linear's weight gradient
    if (b_mc || b_trans) return hipErrorInvalidValue;
    return a_mc ? seq_launch<T, NC, SEQ_AMC, true, false>(g, batches, s)
                : seq_launch<T, NC, SEQ_PLAIN, true, false>(g, batches, s);
  }
  if (b_trans)  // MC-Linear: plain input, MC weight stored [out][in]
    return !a_mc && b_mc ? seq_launch<T, NC, SEQ_BMC, false, true>(g, batches, s) : hipErrorInvalidValue;
  if (a_mc) return seq_launch<T, NC, SEQ_AMC, false, false>(g, batches, s);
  return b_mc ? seq_launch<T, NC, SEQ_BMC, false, false>(g, batches, s) : hipErrorInvalidValue;
}

template <typename T>
hipError_t seq_typed(const MmLaunch &L, hipStream_t s) {
  SeqArgs<T> g = {};
  g.A = (const T *)L.A;
  g.B = (const T *)L.B;
  g.C = (T *)L.C;
  g.y = (const T *)L.y;
  g.M = L.M;
  g.N = L.N;
  g.K = L.K;
  g.a_plane = L.a_plane;
  g.b_plane = L.b_plane;
  g.last = (T *)L.last;
  const int64_t n_stored = L.last ? L.N - 1 : L.N;
  g.c_plane = L.B1 * L.B2 * L.M * n_stored;
  g.y_plane = L.y_plane;
  g.y_ld = L.y_ld;
  g.a_ld = L.a_trans ? L.M : L.K;
  g.b_ld = L.b_trans ? L.K : n_stored;
  g.B2 = L.B2;
  g.a_s1 = L.a_s1;
  g.a_s2 = L.a_s2;
  g.b_s1 = L.b_s1;
  g.b_s2 = L.b_s2;
  g.np = L.a_mc && L.b_mc ? L.nc : 1;
  g.mode = L.mode;
  g.alpha = (T)L.alpha;
  g.beta = (T)L.beta;
  const int64_t batches = L.B1 * L.B2;
  switch (L.nc) {
    case 1: return seq_kinds<T, 1>(g, batches, L.a_mc, L.b_mc, L.a_trans, L.b_trans, s);
    case 2: return seq_kinds<T, 2>(g, batches, L.a_mc, L.b_mc, L.a_trans, L.b_trans, s);
    case 3: return seq_kinds<T, 3>(g, batches, L.a_mc, L.b_mc, L.a_trans, L.b_trans, s);
    case 4: return seq_kinds<T, 4>(g, batches, L.a_mc, L.b_mc, L.a_trans, L.b_trans, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace mcf

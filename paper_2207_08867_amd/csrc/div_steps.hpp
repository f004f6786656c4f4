// div_steps.hpp -- Div-MCN and Mult-MCN (A.2.1) as the elementwise kernels run them.
//
// They return exactly what div_mcn / mult_mcn of mcf_arith.hpp return, bit for bit,
// with four shortcuts:
//   * each ScalingN(y, q) takes the kept-terms form of mm_steps.hpp (the nc terms
//     Simple-Renorm keeps, no final carry, and a per-lane test that Simple-Renorm
//     would not change them; failing lanes compute the full terms and compact them).
//     A zero term of either sign may then reach the next Add-MCN where the literal
//     step has +0; that only changes zero signs of that Add-MCN's Two-Sum errors,
//     which Simple-Renorm drops, and its outputs are the same;
//   * the quotient digits share the reciprocal of the divisor's leading component
//     (Divisor below; not so Div-MCN of binary32);
//   * the last quotient digit q_nc is computed only by lanes whose first digit is zero.
//     The remainder is a Simple-Renorm output after the first update, so a later digit is
//     zero only when the remainder is or when its quotient underflows, and then the update
//     with it leaves the remainder as it is: zero digits trail, Simple-Renorm of the nc+1
//     digits keeps the first nc as they are, and q_nc is not needed (it is zero whenever
//     one of those is).  A divisor with infinite or NaN low components leaves the remainder's
//     last component infinite or NaN: such lanes take the full algorithm too;
//   * the remainder updates x - y q compact their terms by a shift (add_mcn_shift).
// Measured on 2^26 elements at nc = 3 against the literal algorithm: binary16 Div-MCN
// 514 -> 207 us and Mult-MCN 986 -> 432 us; binary32 562 -> 418 and 1112 -> 500 us (at
// about 5.5 TB/s; before the shared reciprocal, the digit test below and the short
// Renormalize: 338, 734, 423 and 563 us).
// The remainder updates x - y q cancel the leading component, so their terms usually
// start with a zero and trail off in zeros; the shift compaction covers those
// patterns (a simulation of the binary16 nc = 3 workload found no other pattern in
// more than 99.99% of the updates).
#pragma once

#include <type_traits>

#include "mcf_arith.hpp"
#include "mm_steps.hpp"

namespace mcf {

// ScalingN(y, q) with expand off, kept-terms form.
template <typename T, int N>
__device__ __forceinline__ void scaling_n_kept(const T (&y)[N], T q, T (&out)[N]) {
  T last;
  scaling_kept<T, N, false, false>(y, q, out, last);
  if (kept_invalid<T, N, false, true>(out, last)) {
    T h[N + 1];
    scaling_terms<T, N>(y, q, h);
    compact_nz<T, N + 1, N>(h, out);
  }
}

// Add-MCN(x, y) for the remainder updates x - y q, whose leading term usually cancels
// to zero and whose last terms are often zero (binary16).  Simple-Renorm of the nc+1
// terms is a shift by one slot when h_0 is zero and the identity otherwise, provided
// no zero precedes a non-zero among h_1 .. h_nc; lanes where one does take the
// general compaction.  (A zero output component may differ from the literal step in
// sign only; Div-MCN's zero remainders only ever yield zero quotient digits, which
// Simple-Renorm drops.)
template <typename T, int N>
__device__ __forceinline__ void add_mcn_shift(const T (&x)[N], const T (&y)[N], T (&out)[N]) {
  T h[N + 1];
  add_terms<T, N>(x, y, h);
  bool z[N + 1];
#pragma unroll
  for (int i = 0; i <= N; ++i) z[i] = h[i] == T(0);
  bool bad = false;
#pragma unroll
  for (int i = 1; i < N; ++i) bad = bad | (z[i] & !z[i + 1]);
  if (__builtin_expect(bad, 0)) {
    compact_nz<T, N + 1, N>(h, out);
    return;
  }
#pragma unroll
  for (int i = 0; i < N; ++i) out[i] = z[0] ? h[i + 1] : h[i];
}

// Component divisions by one divisor, each by itself.
template <typename T>
struct IeeeDivisor {
  T y;
  __device__ __forceinline__ explicit IeeeDivisor(T y0) : y(y0) {}
  __device__ __forceinline__ T divide(T a) const { return div_(a, y); }
};

// Component divisions that share the divisor's reciprocal.  General case: none.
template <typename T>
struct Divisor : IeeeDivisor<T> {
  using IeeeDivisor<T>::IeeeDivisor;
};

// binary16 through binary32: q = a r with r within one unit in the last place of 1 / y,
// then q + (a - y q) r.  The residual a - y q is exact (24-bit q and 11-bit y against an
// a that nearly cancels), so the result is within 2^-24 (1 + 2^-20) |a / y| of a / y.  A
// point halfway between two binary16 values is M 2^k with M < 2^12, and |a / y - M 2^k|,
// if not zero, is at least 2^k / B for y = B 2^j, B < 2^11: more than 2^-23 |a / y|.  So no
// halfway point lies between, and rounding to binary16 gives RN(a / y); a quotient that
// is itself a halfway point (below the normal range) is a 12-bit binary32 value and
// comes out exact.  Zero, infinite or NaN operands that matter make the residual a NaN.
// 9 issue slots a quotient instead of 23 (binary32's division and the conversions).
template <>
struct Divisor<_Float16> {
  _Float16 y;
  float yf, r;
  __device__ __forceinline__ explicit Divisor(_Float16 y0) : y(y0), yf((float)y0), r(__builtin_amdgcn_rcpf(yf)) {}
  __device__ __forceinline__ _Float16 divide(_Float16 a) const {
    const float af = (float)a;
    float q = af * r;
    q = __builtin_fmaf(__builtin_fmaf(-yf, q, af), r, q);
    if (__builtin_expect(q != q, 0)) return div_(a, y);
    return (_Float16)q;
  }
};

// binary32: the steps of LLVM's published lowering of an IEEE division for AMDGPU
// (SITargetLowering::LowerFDIV32: reciprocal, one Newton step on it, quotient, two residual
// corrections), without its scaling, which leaves operands in this range as they are: 2^-20 < |y| < 2^20, 2^-80 < |q| < 2^40 (so
// |a| > 2^-100: every residual is exact).  Outside it, and for zero, infinite or NaN
// operands, div_.  For Mult-MCN and Mult-MCN-Slow, which their arithmetic bounds (2^24
// elements, nc = 3 / 4: 141 / 252 us with divisions by themselves, 123 / 232 with this).
// Div-MCN at those sizes is bound by memory, and a zero remainder sends its wavefront to
// div_: EwDivisor.
template <>
struct Divisor<float> {
  float y, r;
  __device__ __forceinline__ explicit Divisor(float y0) : y(y0) {
    const float r0 = __builtin_amdgcn_rcpf(y);
    r = __builtin_fmaf(__builtin_fmaf(-y, r0, 1.0f), r0, r0);
    const float m = __builtin_fabsf(y);
    if (!(m > 0x1p-20f && m < 0x1p20f)) r = __builtin_nanf("");
  }
  __device__ __forceinline__ float divide(float a) const {
    float q = a * r;
    q = __builtin_fmaf(__builtin_fmaf(-y, q, a), r, q);
    q = __builtin_fmaf(__builtin_fmaf(-y, q, a), r, q);
    const float m = __builtin_fabsf(q);
    if (__builtin_expect(!(m > 0x1p-80f && m < 0x1p40f), 0)) return div_(a, y);
    return q;
  }
};

// What Div-MCN of binary32 takes, us with Divisor -> IeeeDivisor: 2^24 elements nc = 2 67.0 -> 66.1,
// nc = 3 103.4 -> 101.4; 2^22 nc = 2 18.7 -> 18.0; 4096 to 2^16 nc = 4 9.4 .. 9.8 -> 8.6 .. 9.4.
template <typename T>
using EwDivisor = std::conditional_t<sizeof(T) == 4, IeeeDivisor<T>, Divisor<T>>;

template <typename T, int N, typename D = Divisor<T>>
__device__ __forceinline__ void div_mcn_fast(const T (&x_in)[N], const T (&y)[N], T (&out)[N]) {
  T x[N];
#pragma unroll
  for (int c = 0; c < N; ++c) x[c] = x_in[c];
  T h[N + 1];
  const D by(y[0]);
  T q = by.divide(x[0]);
  h[0] = q;
#pragma unroll
  for (int i = 1; i <= N; ++i) {
    if (i == N && h[0] != T(0) && (N == 1 || finite_(x[N - 1]))) {
#pragma unroll
      for (int c = 0; c < N; ++c) out[c] = h[c] + T(0);  // a zero digit leaves as +0, Simple-Renorm's padding
      return;
    }
    T s[N], neg[N];
    scaling_n_kept<T, N>(y, q, s);
#pragma unroll
    for (int c = 0; c < N; ++c) neg[c] = -s[c];
    add_mcn_shift<T, N>(x, neg, x);
    q = by.divide(x[0]);
    h[i] = q;
  }
  simple_renorm<T, N + 1, N>(h, out);
}

// Renormalize (Priest variant) of up to three components, what renormalize of mcf_arith.hpp
// returns.  Its second sweep starts with Two-Sum(s, 0), which emits nothing when s is
// finite, and at N = 2 goes on with Two-Sum(s, t_1) of a pair that a Two-Sum just
// returned: the pair again.  What is left emits at most twice before the final s, so
// the compaction is three selects.  (x + 0 makes the padding +0.)
template <typename T, int N>
__device__ __forceinline__ void renormalize_fast(const T (&x)[N], T (&b)[N]) {
  if constexpr (N == 2 || N == 3) {
    T s = x[0], t[N];
#pragma unroll
    for (int i = 1; i < N; ++i) two_sum(x[i], s, s, t[i]);
    if (__builtin_expect(!finite_(s), 0)) {
      renormalize<T, N, N>(x, b);
    } else if constexpr (N == 2) {
      b[0] = s;
      b[1] = t[1] + T(0);
    } else {
      T s1, e1, s2, e2;
      two_sum(s, t[1], s1, e1);
      const bool emit = e1 != T(0);
      two_sum(emit ? e1 : s1, t[2], s2, e2);
      e2 = e2 + T(0);
      b[0] = emit ? s1 : s2;
      b[1] = emit ? s2 : e2;
      b[2] = emit ? e2 : T(0);
    }
  } else {
    renormalize<T, N, N>(x, b);
  }
}

// Mult-MCN, fast version: Renormalize(Div-MCN(x, Renormalize(Div-MCN(1, y)))).
template <typename T, int N>
__device__ __forceinline__ void mult_mcn_fast(const T (&x)[N], const T (&y)[N], T (&out)[N]) {
  T one[N], q[N], yinv[N];
  one[0] = T(1);
#pragma unroll
  for (int c = 1; c < N; ++c) one[c] = T(0);
  div_mcn_fast<T, N>(one, y, q);
  renormalize_fast<T, N>(q, yinv);
  div_mcn_fast<T, N>(x, yinv, q);
  renormalize_fast<T, N>(q, out);
}

// Mult-MCN-Slow (mcf_arith.hpp: mult_mcn_slow) with its DivN steps taken by
// div_mcn_fast: the same bits.
template <typename T, int N>
__device__ __forceinline__ void mult_mcn_slow_fast(const T (&x_in)[N], const T (&y)[N], T (&out)[N]) {
  T x[N];
#pragma unroll
  for (int c = 0; c < N; ++c) x[c] = x_in[c];
  T h[N + 1];
  T p = x[0] * y[0];
  h[0] = p;
#pragma unroll
  for (int i = 1; i <= N; ++i) {
    T pv[N], d[N], neg[N];
    pv[0] = p;
#pragma unroll
    for (int c = 1; c < N; ++c) pv[c] = T(0);
    div_mcn_fast<T, N>(pv, y, d);
#pragma unroll
    for (int c = 0; c < N; ++c) neg[c] = -d[c];
    add_mcn_shift<T, N>(x, neg, x);
    p = x[0] * y[0];
    h[i] = p;
  }
  simple_renorm<T, N + 1, N>(h, out);
}

}  // namespace mcf

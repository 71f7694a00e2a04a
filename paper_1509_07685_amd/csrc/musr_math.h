// FP64 quotient and logarithm of the fit statistic's terms.
//
// Both are written from IEEE multiply-adds and a machine's reciprocal
// estimate, taken from a policy class Ops (estimate(d): 1/d to 2^-22 or better; fma_const(a, b, c): a b + c), so that a host-only test runs the
// same operations.  Arguments are normal and finite; the caller keeps them
// within 2^-960 .. 2^960.
#ifndef DKS_MUSR_MATH_H
#define DKS_MUSR_MATH_H

#include <string.h>

#ifdef __HIPCC__
#define DKS_MUSR_FN __device__ __forceinline__
#else
#define DKS_MUSR_FN inline
#endif

namespace dks {
namespace musr {

// 1 / d to about a unit in the last place: the estimate and two Newton steps.
template <class Ops> DKS_MUSR_FN double recip(double d) {
  double y = Ops::estimate(d);
  y = __builtin_fma(__builtin_fma(-d, y, 1.0), y, y);
  return __builtin_fma(__builtin_fma(-d, y, 1.0), y, y);
}

// n / d from y = recip(d): the product's remainder n - d q is exact in one
// fma, and q plus that remainder times y is n / d rounded once (but for a
// rare neighbour), so no error of y is left in it.  With d = 0 and y = 1/2
// the result is n.
DKS_MUSR_FN double quotient(double n, double d, double y) {
  const double q = n * y;
  return __builtin_fma(__builtin_fma(-d, q, n), y, q);
}

// log(q) of q > 0: q = 2^k m with m in [sqrt(1/2), sqrt(2)), s = f / (m + 1)
// with f = m - 1 (exact), log m = 2 atanh(s) = 2 s + 2 s z P(z), z = s^2 <=
// 0.02945.  P interpolates 1/3 + z/5 + z^2/7 + ... at the seven Chebyshev
// nodes of that interval (z P off by at most 4.7e-18).  The rounding of s and
// of m + 1 is taken from the exact remainder f - s (m + 1) and carried with
// the low part of k log 2 and of the leading sum beside the series, so that
// one rounding of the result is left: at most 0.55 units in the last place
// over 2^-960 .. 2^960, 0.289 in the mean square (1.7 and 0.6 without the
// remainder).
template <class Ops> DKS_MUSR_FN double log_normal(double q) {
  unsigned long long bits;
  memcpy(&bits, &q, sizeof(bits));
  const int hi = (int)(bits >> 32);
  const int k = (hi - 0x3fe6a09e) >> 20;                  // sqrt(1/2) = 0x3fe6a09e...
  bits = (bits & 0xffffffffull) | ((unsigned long long)(unsigned)(hi - k * 0x100000) << 32);
  double m;
  memcpy(&m, &bits, sizeof(m));
  const double f = m - 1.0, w = m + 1.0, low = m - (w - 1.0);    // w + low = m + 1
  double y = Ops::estimate(w);
  y = __builtin_fma(__builtin_fma(-w, y, 1.0), y, y);
  const double s = f * y;
  const double ds = y * __builtin_fma(-s, low, __builtin_fma(-s, w, f));
  const double t = s + ds, z = t * t;
  double p = 0.0730856419990365;
  p = Ops::fma_const(p, z, 0.07665833338298587);
  p = Ops::fma_const(p, z, 0.09091445389013066);
  p = Ops::fma_const(p, z, 0.11111105556052474);
  p = Ops::fma_const(p, z, 0.1428571431305726);
  p = Ops::fma_const(p, z, 0.199999999999496);
  p = Ops::fma_const(p, z, 0.3333333333333335);
  const double s2 = s + s, kd = (double)k;
  const double a = kd * 0x1.62e42fefa3p-1;                // log 2 to 41 bits: exact
  const double b = a + s2, r = s2 - (b - a);              // |a| >= |s2| or a = 0: r is exact
  const double tail = __builtin_fma((t + t) * z, p, __builtin_fma(2.0, ds, r));
  return b + __builtin_fma(kd, 0x1.3de6af278ece6p-42, tail);
}

}  // namespace musr
}  // namespace dks

#endif  // DKS_MUSR_MATH_H

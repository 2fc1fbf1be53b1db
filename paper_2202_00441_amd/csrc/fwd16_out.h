// fwd16_out.h -- output factors of the bf16 table forward, by input pattern.
//
// A bf16 pattern's top 9 bits are its sign and octave (power of two), the
// other 7 its place in the octave, so all patterns of the octaves in which an
// activation is neither linear nor constant to bf16 precision are a few
// thousand: [2^lo, 2^hi) of either sign, 128 patterns an octave.  For each
// the table holds one fp32 word T, from which the kernel forms the output in
// fp32 and rounds it once:
//
//   product    y = max(x, -X) T     GELU, SiLU, SELU; Tanh with |x| <= X
//   sum        y = max(x, -0) + T   Softplus
//   value      y = T                Sigmoid
//
// X the largest magnitude of the range.  Patterns below the range use its
// lowest entry, patterns above it the highest: the lowest holds the factor's
// limit at 0, the highest its limit at infinity, and the range ends where that
// still gives the correctly rounded output.  Inside the range T is taken from
// the output itself: y* is f(x) in double rounded once to bf16, and T is
// y* / x (y* - max(x, 0), y*), so the fp32 result differs from y* by a few
// units of 2^-20 and rounds to it.  The low 4 bits of T are left 0: the
// kernel puts the element's interval index there, which changes y by less
// than 2^-19 of itself.
//
// Everything here is evaluated at compile time, in double, from the
// functions' definitions and classical series.
#pragma once

#include <cstdint>

#include "../../include/fewbit.h"

namespace fwd16_out {

// ---------------------------------------------------------------- double
constexpr double two_to(int e) {          // -1022 <= e <= 1023
  return __builtin_bit_cast(double, static_cast<uint64_t>(1023 + e) << 52);
}

// e^x for -600 < x <= 0: Taylor series of the remainder of ln 2, which is
// subtracted in two parts (the split of fdlibm's e_exp.c: the first has trailing
// zeros, so its multiple is exact)
constexpr double exp_of(double x) {
  const int k = static_cast<int>(x * 1.4426950408889634074 - 0.5);
  const double r = (x - k * 0.693147180369123816490) - k * 1.90821492927058770002e-10;
  double s = 1.0;
  for (int i = 14; i >= 1; --i) s = 1.0 + s * r / i;
  return s * two_to(k);
}

// log(1 + u), 0 <= u <= 1: 2 artanh(u / (2 + u))
constexpr double log1p_of(double u) {
  const double z = u / (2.0 + u), z2 = z * z;
  double s = 0.0;
  for (int k = 18; k >= 0; --k) s = s * z2 + 1.0 / (2 * k + 1);
  return 2.0 * z * s;
}

// upper tail of the standard normal, t >= 0: below 3 from the power series
// Phi(t) - 1/2 = phi(t) (t + t^3/3 + t^5/(3 5) + ...), above from Laplace's
// continued fraction phi(t) / (t + 1/(t + 2/(t + 3/...)))
constexpr double normal_tail(double t) {
  const double phi = 0.39894228040143267794 * exp_of(-0.5 * t * t);
  if (t < 3.0) {
    double term = t, sum = t;
    for (int k = 1; k < 45 && term > sum * 1e-18; ++k) {
      term *= t * t / (2 * k + 1);
      sum += term;
    }
    return 0.5 - phi * sum;
  }
  double c = t;
  for (int k = 45; k >= 1; --k) c = t + k / c;
  return phi / c;
}

constexpr double kLambda = 1.0507009873554804934193349852946;
constexpr double kAlpha = 1.6732632423543772848170429916717;

constexpr double f_of(int act, double x) {
  const double t = x < 0.0 ? -x : x;
  if (act == FEWBIT_GELU) return x < 0.0 ? x * normal_tail(t) : x * (1.0 - normal_tail(t));
  const double e = exp_of(act == FEWBIT_TANH ? -2.0 * t : -t);
  if (act == FEWBIT_SILU) return x * ((x < 0.0 ? e : 1.0) / (1.0 + e));
  if (act == FEWBIT_SIGMOID) return (x < 0.0 ? e : 1.0) / (1.0 + e);
  if (act == FEWBIT_TANH) return (x < 0.0 ? e - 1.0 : 1.0 - e) / (1.0 + e);
  if (act == FEWBIT_SELU) return x < 0.0 ? kLambda * kAlpha * (e - 1.0) : kLambda * x;
  return (x < 0.0 ? 0.0 : x) + log1p_of(e);       // Softplus
}

// v rounded once to bf16, nearest even, subnormals kept
constexpr double round_bf16(double v) {
  const double a = v < 0.0 ? -v : v;
  int e = static_cast<int>(__builtin_bit_cast(uint64_t, a) >> 52) - 1023;
  if (e < -126) e = -126;
  const double q = a / two_to(e - 7);             // exact; below 2^8 + 1
  int64_t i = static_cast<int64_t>(q);
  const double rest = q - static_cast<double>(i);
  if (rest > 0.5 || (rest == 0.5 && (i & 1))) ++i;
  const double r = static_cast<double>(i) * two_to(e - 7);
  return v < 0.0 ? -r : r;
}

// ---------------------------------------------------------------- the table
// Octaves [lo, hi) of the table per activation.  lo: from 2^lo down the
// factor's limit at 0 gives the correctly rounded output (SELU's irrational
// factor asks for the most octaves).  hi: GELU's left tail is below half the
// smallest bf16 subnormal from x = -13.6, the tails that fall as e^x from -98;
// Tanh and SELU are constant to bf16 from |x| = 7.  No more octaves than that
// asks for: 1 KiB of table each, and at 16 or fewer every thread of a
// 512-thread workgroup places two chunks instead of three.
constexpr int lo_of(int act) {
  return act == FEWBIT_SELU ? -17 : act == FEWBIT_SOFTPLUS ? -12 : act == FEWBIT_GELU ? -10 : -9;
}
constexpr int hi_of(int act) {
  return act == FEWBIT_SILU || act == FEWBIT_SIGMOID || act == FEWBIT_SOFTPLUS ? 7 : 4;
}
// entries per sign; magnitude pattern of the first
constexpr uint32_t count_of(int act) { return static_cast<uint32_t>(hi_of(act) - lo_of(act)) * 128u; }
constexpr uint32_t base_of(int act) { return static_cast<uint32_t>(127 + lo_of(act)) << 7; }
// value of the magnitude pattern p (normal)
constexpr float value_of(uint32_t p) { return __builtin_bit_cast(float, p << 16); }
// X: the range's largest magnitude
constexpr float max_of(int act) { return value_of(base_of(act) + count_of(act) - 1u); }

// The factor of the entry m of one sign.  SELU's at the ends is its limit
// there: the outputs of a linear range are multiples of it, not of the
// rounded output at the range's end.
constexpr double factor(int act, bool neg, uint32_t m) {
  const double t = value_of(base_of(act) + m);
  const double x = neg ? -t : t;
  if (act == FEWBIT_SELU && !neg && m + 1 == count_of(act)) return kLambda;
  if (act == FEWBIT_SELU && m == 0) return neg ? kLambda * kAlpha : kLambda;
  const double y = round_bf16(f_of(act, x));
  if (act == FEWBIT_SOFTPLUS) return neg ? y : y - x;
  if (act == FEWBIT_SIGMOID) return y;
  return y / x;
}

// fp32 pattern of the factor, rounded to a multiple of 16 units
constexpr uint32_t entry(int act, bool neg, uint32_t m) {
  const uint32_t u = __builtin_bit_cast(uint32_t, static_cast<float>(factor(act, neg, m)));
  return (u + 8u) & ~15u;
}

// Whether the table can hold the interval indices of these boundaries: each
// entry has one index only if no boundary lies among the magnitudes below the
// range, other than at 0, or beyond it.  A symmetric table's indices are
// those of |x|, which its boundaries up to 0 do not divide.
inline bool holds(int act, bool symmetric, const float* s, int boundaries) {
  const float lo = value_of(base_of(act)), hi = max_of(act);
  for (int m = 0; m < boundaries; ++m) {
    const float a = s[m] < 0.0f ? -s[m] : s[m];
    if (a == 0.0f || (symmetric && s[m] < 0.0f)) continue;
    if (!(a > lo && a < hi)) return false;
  }
  return true;
}

// entries of x >= 0, then of x < 0
template <int ACT>
struct Table {
  alignas(16) uint32_t e[2 * count_of(ACT)];
};

template <int ACT>
constexpr Table<ACT> make() {
  Table<ACT> t{};
  for (uint32_t m = 0; m < count_of(ACT); ++m) {
    t.e[m] = entry(ACT, false, m);
    t.e[count_of(ACT) + m] = entry(ACT, true, m);
  }
  return t;
}

}  // namespace fwd16_out

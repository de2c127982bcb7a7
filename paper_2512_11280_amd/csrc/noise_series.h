// log2(1 - t) for small t, and what a logit can still reach under its noise, plain float arithmetic: the CPU tests compile
// this file as it is and hold its error, and the bound, against 64 bits.
#pragma once
#include "records.h"

namespace adasd {

// Below kSerBelow the logarithm of u = 1 - t is taken from t (which is exact to a rounding there, u is not).  The first
// coefficient is -1/ln 2 (what decides at the smallest t), the other three make the largest relative error on
// [0, 1/12] smallest: 1.0e-7.  Error of log2 |log2 u| over all words: 1.13e-7 rms, 7.4e-7 at most (1.08e-6 where the value
// is near -32 and its own rounding is that large).  Five Taylor terms below 1/16 have 1.29e-7 rms, 9.4e-7 at most;
// three below 1/64 2.2e-7 and 3.0e-6, and one multiplication and addition less.
constexpr float kSer0 = -1.44269502f, kSer1 = -0.721385062f, kSer2 = -0.478304029f, kSer3 = -0.412017643f;
constexpr float kSerBelow = 1.0f / 12;
ADASD_ANYWHERE float log2_series(float t) {
  return t * __builtin_fmaf(t, __builtin_fmaf(t, __builtin_fmaf(t, kSer3, kSer2), kSer1), kSer0);
}

// With E = -ln u >= 1 - u, a logit whose key without noise is k (log2 units) stays below k - log2((1 - u) log2 e).  So with
// ef = 2^(k - floor + kReach) it stays below `floor` by more than 2^-13, the guard of the comparisons of keys, if
// ef < (1 - u) 2^32: if noise_reach <= kNoiseTop, which is four ulps of the sum below 2^32.
constexpr float kSlack = 9.765625e-04f;                    // 2^-10: the guard, and the rounding of ef
constexpr float kReach = 32.0f - 0.528766373f + kSlack;    // log2(2^32 / log2 e), and the slack
constexpr float kNoiseTop = 4294966272.0f;                 // 2^32 - 1024
ADASD_ANYWHERE float noise_reach(float e, float f, uint32_t word) { return __builtin_fmaf(e, f, (float)word); }
// Floors are kept less kReach.  The one that a key is good for lies below it by what the roundings of large keys can add up to:
// 2^-24 of its size each for the key, for the other's, and for the two here, and a little more (logits around 1e7 have keys a
// whole unit apart).
ADASD_ANYWHERE float floor_of(float key) { return __builtin_fmaf(__builtin_fabsf(key), -0x1.4p-22f, key - kReach); }
// While nothing has been looked at: below every finite key, and finite itself, so that a masked logit (-inf, or 2^-inf = 0)
// comes to nothing and not to -inf + inf or 0 * inf, which would count as one that may win.
constexpr float kNoFloor = -3.402823466e38f;
// The exponent k - floor of the factor f, for the same reason no more than 127.  What falls out for that has e <= 2^-95 and a
// key below -62, and the row (drafting: the lane's own logits) has an element with e >= 2^-38, whose key is -43.1 at least and
// which is looked at, or lies below one that was: neither the best nor within its margin (2.2 at most where the best is certain).
ADASD_ANYWHERE float reach_exponent(float above) { return __builtin_fminf(above, 127.0f); }

}  // namespace adasd

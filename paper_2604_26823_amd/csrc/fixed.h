// Fixed-point image of the contributions that FP32 paints add into their LDS
// windows (FixAcc in blocks.h): value = integer x 2^-e, e one per work item.
#pragma once

#include <cmath>

#include "common.h"

namespace ic {
namespace fx {

struct Scale {
  double s, inv;
};

// 2^e with amax 2^e < 2^52 (amax < 2^k from frexp, e = 52 - k): every contribution
// is at most amax in magnitude (cloud-in-cell weights are at most 1), and
// the sum of 1024 of them stays below 2^62.  A contribution is rounded by half a
// unit, at most 2^-52 amax.
__host__ __device__ inline Scale scale_for(double amax) {
  if (!(amax > 0.0)) return Scale{1.0, 1.0};
  int k;
  frexp(amax, &k);
  return Scale{ldexp(1.0, 52 - k), ldexp(1.0, k - 52)};
}

// w x rounded to the nearest integer, for 0 <= w <= 1 and |x| <= 2^52, by one
// fused multiply-add onto a constant o: 2^52 for x >= 0 and 2^53 for x < 0 keep
// the result in [2^52, 2^53], where neighbouring doubles are 1 apart and their
// bit patterns count up with them, so the integer is the difference of the bit
// patterns.  o depends on x alone and the low words of its bits are zero: an
// addition costs the fma and one 32-bit subtraction.  (One constant for both
// signs, 1.5 2^52, leaves 51 bits; the cotangent paint takes 257 us instead of 254 at
// 256^3 for the bit, the density paint 168 either way.)
__host__ __device__ inline long long rounded(double w, double x) {
  const double o = x < 0.0 ? 0x1p53 : 0x1p52;
  return __builtin_bit_cast(long long, fma(w, x, o)) - __builtin_bit_cast(long long, o);
}

}  // namespace fx
}  // namespace ic

// Quotients by a reciprocal taken once, for the triangular block solves, whose
// steps each wait for one (a division is ten dependent instructions, this
// three).
#pragma once

#include <hip/hip_runtime.h>

namespace hss {

// num / d by r = 1 / d, correctly rounded: one Newton step (Markstein).  q is
// off by at most 1.5 units in the last place, and the step's own error is
// below 2^-50 of one before its single rounding.
__device__ __forceinline__ double quot_by(double num, double d, double r) {
  const double q = num * r;
  return fma(fma(-q, d, num), r, q);
}

// Whether quot_by(num, d, r) was x = num / d, for 2^-500 < |d| < 2^500.  The
// residual num - q d is a multiple of 2^-106 |num| or so: below 2^-960 it may
// underflow, and the step then corrects q by nothing or by too little; and x
// itself may be neither infinite nor so small that it is rounded at a fixed
// place.  (Dividends below 2^-1010: up to 7 % of the quotients one place off.)
__device__ __forceinline__ bool quot_same(double num, double x) {
  return num == 0.0 || (fabs(num) >= 0x1p-960 && fabs(x) >= 0x1p-1000 && fabs(x) <= 0x1p1000);
}

}  // namespace hss

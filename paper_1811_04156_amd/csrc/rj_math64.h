// rj_math64.h -- FP64 reciprocal, reciprocal square root and exponential of
// ordinary numbers (no zeros, infinities, NaN or subnormals), for the anchors'
// kernels.  The hardware's starting value is an argument, so that the host can
// run the same arithmetic.
#pragma once

#include <math.h>

#ifdef __HIPCC__
#define RJ_FN __host__ __device__ __forceinline__
#else
#define RJ_FN inline
#endif

namespace rj {

// One third-order correction of a value y good to 2^-23 or better: with
// e = 1 - x y, 1 / x = y / (1 - e) = y (1 + e + e^2 + O(e^3)).
RJ_FN double rcp_from(double x, double y) {
    const double e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
}

// With e = 1 - x y^2, x^(-1/2) = y (1 - e)^(-1/2) = y (1 + e / 2 + 3 e^2 / 8 + O(e^3)).
RJ_FN double rsq_from(double x, double y) {
    const double e = fma(-(x * y), y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// e^x = 2^k e^r with r = x - k ln 2 by Cody and Waite's reduction (Software
// Manual for the Elementary Functions, 1980): ln 2 in two pieces, the first with
// 21 trailing zero bits, so that k times it is exact; e^r, |r| <= ln 2 / 2, by its
// power series to r^13 / 13! (the rest is below 2^-57).
RJ_FN double exp_series(double x, double& k) {
    k = rint(x * 1.4426950408889634074);
    double r = fma(k, -0x1.62e42fee00000p-1, x);
    r = fma(k, -0x1.a39ef35793c76p-33, r);
    double p = 1.0 / 6227020800.0; // 1 / 13!
    p = fma(p, r, 1.0 / 479001600.0);
    p = fma(p, r, 1.0 / 39916800.0);
    p = fma(p, r, 1.0 / 3628800.0);
    p = fma(p, r, 1.0 / 362880.0);
    p = fma(p, r, 1.0 / 40320.0);
    p = fma(p, r, 1.0 / 5040.0);
    p = fma(p, r, 1.0 / 720.0);
    p = fma(p, r, 1.0 / 120.0);
    p = fma(p, r, 1.0 / 24.0);
    p = fma(p, r, 1.0 / 6.0);
    p = fma(p, r, 0.5);
    p = fma(p, r, 1.0);
    return fma(p, r, 1.0);
}

} // namespace rj

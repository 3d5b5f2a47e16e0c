// dk_sum.h -- FP64 sums of an observable that keep their rounding errors.  An observable is centred by a mean
// of its own size before the factor sqrt(N): at N = 2e9 one rounding of the sum is 1e-12 of the result.
#pragma once
#include <hip/hip_runtime.h>

namespace dk {

// a sum and its rounding errors
struct Sum {
    double hi = 0.0, lo = 0.0;
    // + v + e
    __device__ __forceinline__ void add(double v, double e)
    {
#pragma clang fp contract(off)
        const double s = hi + v, b = s - hi;
        lo += ((hi - (s - b)) + (v - b)) + e;
        hi = s;
    }
    // + a * b
    __device__ __forceinline__ void add_product(double a, double b)
    {
        const double v = a * b;
        add(v, fma(a, b, -v));
    }
    // h2 * sum - c.  Where a sum went to infinity its errors are not numbers, and hi is what a plain sum gives.
    __device__ __forceinline__ double centred(double h2, double c) const
    {
        const double e = h2 * lo;
        return fma(h2, hi, -c) + (e == e ? e : 0.0);
    }
};

}  // namespace dk

// Shape of the sinc kernels (host and device, so that its error can be measured on
// the host; the reciprocal's first estimate, good to 2^-20 or better, comes from the
// caller).
#pragma once

#include <hip/hip_runtime.h>

namespace sph {

// The sinc shape S = sin(x) / x, x = pi q / 2, and dS/dq for q in [0, 2) in FP64.
//   S: its Taylor series in q^2 up to x^22 on [0, 1], where the first omitted term is
//      below 1e-18; beyond, by the reflection S = (2 - q) / q times S at 2 - q, which
//      keeps the relative accuracy where S goes to zero.
//   dS/dq: q times the Taylor series of dS/dq / q in q^2 about q^2 = 5/2, where its
//      terms hardly cancel (about 0 they do by a factor of 8 at q = 2); the first
//      omitted one is below 2e-18 of it (it has no zero).
// Largest relative error, measured on the host: S 2.8e-16, dS/dq 3.0e-16 (series
// about 0 with a rounded reciprocal 3.7e-16 and 6.4e-16; sine, cosine and divisions up
// to 2e-11 for S near q = 2, 4e-8 for the slope near 0 and 5.4e-16 near 2).
// 22 instructions for S and 14 for dS/dq, where sin, sincos and their divisions took
// some 60 to 100: 262,000 particles, exponent 5: density 160 -> 126 us, IAD matrices
// 361 -> 162, momentum with IAD 414 -> 352.
struct SincSeries {
    double s[12];
    // the series about 5/2, from the one about 0 in 113 bits
    double d[13] = {-0.41498307213969732,    0.12749130128742714,     -0.01254916620411933,
                    0.00061340794405985238,  -1.8001687330729437e-05, 3.5312524507558498e-07,
                    -4.9629957774186507e-09, 5.2470527861712425e-11,  -4.3265069506750305e-13,
                    2.8610737814739403e-15,  -1.551454261555551e-17,  7.0248187987627409e-20,
                    -2.6962414647826329e-22};
    constexpr SincSeries() : s()
    {
        double f = 1.0, p = 1.0;  // (2k + 1)! and (pi / 2)^(2k)
        for (int k = 0; k < 12; ++k) {
            if (k > 0) {
                f *= (double)(2 * k) * (double)(2 * k + 1);
                p *= 1.5707963267948966 * 1.5707963267948966;
            }
            s[k] = (k % 2 ? -1.0 : 1.0) * (p / f);
        }
    }
};

// a / b from an estimate y of 1 / b: one Newton step, then the quotient corrected by
// its remainder (about half an ulp; as many operations as the reciprocal to one ulp
// and a product).
__host__ __device__ inline double sinc_quotient(double a, double b, double y)
{
    y = __builtin_fma(y, __builtin_fma(-b, y, 1.0), y);
    const double t = a * y;
    return __builtin_fma(__builtin_fma(-b, t, a), y, t);
}

// est(q): the estimate of 1 / q.
template <typename Est>
__host__ __device__ inline double sinc_s(double q, Est est)
{
    constexpr SincSeries c{};
    const double y = __builtin_fmin(q, 2.0 - q), y2 = y * y;
    double v = c.s[11];
#pragma unroll
    for (int k = 10; k >= 0; --k) v = __builtin_fma(v, y2, c.s[k]);
    return q > 1.0 ? v * sinc_quotient(y, q, est(q)) : v;
}

__host__ __device__ inline double sinc_ds(double q)
{
    constexpr SincSeries c{};
    const double z = __builtin_fma(q, q, -2.5);
    double v = c.d[12];
#pragma unroll
    for (int k = 11; k >= 0; --k) v = __builtin_fma(v, z, c.d[k]);
    return q * v;
}

}  // namespace sph

// 10^x for the lambdas of the prior smoothing's search in the run kernel.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

namespace m2m {

// 10^x = 2^k e^r with r = x ln 10 - k ln 2, |r| <= ln(2) / 2, in two parts hi + lo
// (ln 10 and ln 2 in two parts each; k times the first part of ln 2, 34 bits, is
// exact for |k| < 2^19), and e^r = 1 + hi + (lo (1 + hi) + hi^2 q(hi)) with the
// Taylor polynomial q of (e^r - 1 - r) / r^2 of degree 12 (remainder 1e-19 of
// e^r) over 14!, its coefficients 14! / n! made on the way. Worst of 65536 points in
// |x| < 30, in units of the last place: 0.61; the device library's pow 1.24 and
// exp10 0.97. With r in one part, from x log2(10), it was off by 3e-15 at |x| = 25.
// The kernel has no registers to spare for constants: the library's exp10 kept
// its coefficients in registers through the whole step loop, 16 of 128 spilled, and
// 24 steps of 600 000 FP32 particles with one refresh took 332 us, so 285. The
// constants here are loaded where they are used.
__host__ __device__ inline double pow10_of(double x) {
#pragma clang fp contract(off)
    // log2(10); ln 10 and ln 2, each in two parts; 14!
    static constexpr double table[6] = {3.32192809488736234787, 0x1.26bb1bbb55516p+1,
                                        -2.1707562233822494e-16, 0x1.62e42fef80000p-1,
                                        1.619851018665656e-11, 87178291200.0};
#ifdef __HIP_DEVICE_COMPILE__
    auto c = (const __attribute__((address_space(4))) double*)table;
    asm volatile("" : "+s"(c));
#else
    const double* c = table;
#endif
    const double k = rint(x * c[0]);
    const double p = x * c[1], kh = k * c[3];
    const double d = p - kh;
    const double tail = fma(-k, c[4], (p - (d + kh)) + fma(x, c[2], fma(x, c[1], -p)));
    const double hi = d + tail, lo = tail - (hi - d);
    double e = 1.0, f = 1.0;
#pragma unroll 1
    for (int n = 14; n >= 3; --n) {
        f *= n;
        e = fma(e, hi, f);
    }
    const double q = e / c[5];
    const double s = 1.0 + hi;
    return ldexp(s + ((hi - (s - 1.0)) + fma(hi * hi, q, lo * s)), (int)k);
}

}  // namespace m2m

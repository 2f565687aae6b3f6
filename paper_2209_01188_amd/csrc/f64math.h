// fp64 functions of the row kernels, attention and GeLU: straight-line forms for kernels that wait for them, with errors
// no larger than those of the library forms they stand in for.  Nothing here needs a GPU but the two estimates
// (reciprocal, reciprocal square root), so the errors are checked on the CPU as well.
#pragma once

// 1 / sqrt(v) for normal v > 0: the instruction's estimate and two cubic Newton steps, within 1.0 units in the last place
// (the quotient of the rounded root is within 1.5, in a chain of some 60 dependent instructions, which a one-row kernel
// waits for)
__device__ __forceinline__ double rsqrt_f64(double v) {
    double y = __builtin_amdgcn_rsq(v);
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const double e = fma(-v * y, y, 1.0);
        y = fma(y * e, fma(0.375, e, 0.5), y);
    }
    return y;
}
// e^x in fp64, within 0.75 units in the last place (the library's: 0.88) in some 24 instructions without a branch:
// x = n ln 2 + r, |r| <= 0.347, with r also as rh - n ln2_lo, e^x = 2^n (1 + r + r^2 q(r)), 1 + rh as a sum of two and q the
// degree-9 interpolation of (e^r - 1 - r) / r^2 in Chebyshev points.  (r + r^2 q rounded, then 1 added: 1.08.)
// For x <= 709; 0 below -745 and for -infinity; NaN stays NaN (the clamp is a comparison: fmax would turn a NaN into the
// bound, and a key whose score is NaN would drop out of a softmax).
__device__ __forceinline__ double exp_f64(double x) {
    constexpr double MAGIC = 6755399441055744.0;                    // 1.5 * 2^52: rounds to an integer, which sits in the low word
    x = x < -800.0 ? -800.0 : x;
    const double t = fma(x, 0x1.71547652b82fep+0, MAGIC), n = t - MAGIC;
    const double rh = fma(n, -0x1.62e42fef00000p-1, x);             // n ln2_hi and the difference are exact
    const double r = fma(n, -0x1.473de6af278edp-34, rh);
    double q = 0x1.af38ed3540c23p-26;
    q = fma(q, r, 0x1.289186dc77ac4p-22);
    q = fma(q, r, 0x1.71de0d8a3250fp-19);
    q = fma(q, r, 0x1.a019b90ba6b3fp-16);
    q = fma(q, r, 0x1.a01a01a7d1625p-13);
    q = fma(q, r, 0x1.6c16c1788c5e4p-10);
    q = fma(q, r, 0x1.1111111110994p-7);
    q = fma(q, r, 0x1.5555555553d61p-5);
    q = fma(q, r, 0x1.5555555555556p-3);
    q = fma(q, r, 0x1.0000000000001p-1);
    const double h = 1.0 + rh, l = fma(n, -0x1.473de6af278edp-34, (1.0 - h) + rh);
    return __builtin_amdgcn_ldexp(h + fma(r * r, q, l), (int)(unsigned)__builtin_bit_cast(unsigned long long, t));
}
// tanh-form GeLU in fp64: 0.5 v (1 + tanh u) == v / (1 + exp(-2u)); the quotient from the reciprocal instruction, two
// Newton steps and one correction by the remainder
__device__ __forceinline__ double gelu_tanh(double v) {
    const double u = 0.7978845608028654 * (v + 0.044715 * v * v * v);
    const double d = 1.0 + exp_f64(fmin(-2.0 * u, 709.0));           // a NaN comes back in through v
    double y = __builtin_amdgcn_rcp(d);
    y = fma(fma(-d, y, 1.0), y, y);
    y = fma(fma(-d, y, 1.0), y, y);
    const double q = v * y;
    return q == (double)INFINITY ? q : fma(fma(-d, q, v), y, q);     // GeLU(+infinity): there the remainder would be NaN
}

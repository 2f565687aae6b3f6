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
// tanh-form GeLU in fp64: 0.5 v (1 + tanh u) == v / (1 + exp(-2u)), in some 32 instructions of its own (on exp_f64 41; a
// prefill call's up linear spends a fifth of its time on them): y = -2 u / ln 2 straight from v (-1.5957... / ln 2 as a sum of
// two numbers, and that times 0.044715), its last product with the part that rounding would drop, 2^y as 2^n 2^f with the
// degree-10 interpolation of (2^f - 1) / f in Chebyshev points, the quotient from the reciprocal instruction, one cubic step and
// one correction by the remainder.  Where 1 + tanh u nearly vanishes the rounding of the argument is what the error consists
// of: on [-6, -5] up to 36 units in the last place of the function with these constants as doubles (44 with the square root of
// 2 / pi itself); the form on exp_f64 45 and 51 as the compiler contracts it here, 57 and 61 uncontracted; without the dropped
// part 56 and 63 either way.  Beyond +-20 the result is v, or less than 1e-250.  NaN gets lost in the clamps and comes back in
// through v in the remainder; +infinity is kept out of the quotient, where its remainder would be NaN, and comes back in there
// too.
__device__ __forceinline__ double gelu_tanh(double v) {
    constexpr double MAGIC = 6755399441055744.0;
    const double c = fmin(fmax(v, -20.0), 20.0);
    const double s = fma(c * c, -0x1.a5a7cf7572a98p-4, -0x1.26aec21bce75ap+1), y = c * s;
    const double k = y + MAGIC, f = (y - (k - MAGIC)) + fma(c, 0x1.85892a664356cp-53, fma(c, s, -y));
    double q = 0x1.e9d3fe3952179p-32;
    q = fma(q, f, 0x1.e6063f7217bc6p-28);
    q = fma(q, f, 0x1.b524fae627834p-24);
    q = fma(q, f, 0x1.62bfd47773353p-20);
    q = fma(q, f, 0x1.ffcbfc670dcd4p-17);
    q = fma(q, f, 0x1.430913096fd9fp-13);
    q = fma(q, f, 0x1.5d87fe78a5276p-10);
    q = fma(q, f, 0x1.3b2ab6fba1ddap-7);
    q = fma(q, f, 0x1.c6b08d704a0c2p-5);
    q = fma(q, f, 0x1.ebfbdff82c598p-3);
    q = fma(q, f, 0x1.62e42fefa39efp-1);
    const double d = 1.0 + __builtin_amdgcn_ldexp(fma(q, f, 1.0), (int)(unsigned)__builtin_bit_cast(unsigned long long, k));
    double r = __builtin_amdgcn_rcp(d);
    const double h = fma(-d, r, 1.0);
    r = fma(r, fma(h, h, h), r);
    const double g = fmin(v, 1e300) * r;
    return fma(fma(-d, g, v), r, g);
}

// fp16 values as balanced 8-bit digits for exact products on the int8 matrix instruction.
// Every fp16 value is an integer multiple of 2^-24: x = 2^-24 sum_j 256^j d_j with d_j in [-128, 127]; four digits
// cover |x| < 127.5.  A sum of products of two such values is the sum over the digit pairs (i, j) of 256^(i + j - 6)
// sum d_i d_j (in units of 1), i.e. sixteen int8 x int8 -> int32 products, exact.
#pragma once
#include "common.h"

constexpr uint32_t DIGITS_BIG = 0x57f8;    // fp16 bits of 127.5: from here on four digits do not do

// The digit planes of four values below 127.5 in magnitude, one word per plane (byte k = value k).
// x * 256 rounded to an integer (up to a lower half in [-32896, 32639], which is what two balanced digits hold: the
// addend moves the rounding boundary by a little over 2^-9) carries the upper two digits, the exact rest times 2^24
// the lower two; both sit, plus 0x8080, in the low bytes of an fp32 sum.  (Fewer instructions than by conversion to integers and
// shifts; each runs at the same rate, conversions included.)
__device__ __forceinline__ void digit_planes4(const __half (&x)[4], int (&p)[4]) {
    constexpr float M = 8388608.0f + 0x8080;
    uint32_t t[4], u[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const float f = __half2float(x[i]);
        const float hi = fmaf(f, 256.0f, 0.001953125f + 0.00000762939453125f) + M;
        const float rest = fmaf(hi - M, -0.00390625f, f);
        t[i] = __float_as_uint(hi);
        u[i] = __float_as_uint(fmaf(rest, 16777216.0f, M));
    }
    const uint32_t a = __builtin_amdgcn_perm(u[1], u[0], 0x05010400), b = __builtin_amdgcn_perm(u[3], u[2], 0x05010400);
    const uint32_t c = __builtin_amdgcn_perm(t[1], t[0], 0x05010400), d = __builtin_amdgcn_perm(t[3], t[2], 0x05010400);
    p[0] = (int)(__builtin_amdgcn_perm(b, a, 0x05040100) ^ 0x80808080u);
    p[1] = (int)(__builtin_amdgcn_perm(b, a, 0x07060302) ^ 0x80808080u);
    p[2] = (int)(__builtin_amdgcn_perm(d, c, 0x05040100) ^ 0x80808080u);
    p[3] = (int)(__builtin_amdgcn_perm(d, c, 0x07060302) ^ 0x80808080u);
}

// Scale of the digit form of output row n's dequantized weights: a = sw / 127 (fp32, as everywhere),
// E = its binary exponent (not below fp16's smallest normal one), so that every fp16(code * a) is a
// multiple of u = 2^(E - 10); m = a / u rounded to an integer (0 is possible for a row whose scale is
// below fp16's subnormal spacing; its products can still round up to a few u).  False for a zero row.
__device__ __forceinline__ bool digit_scale(float sw, float &a, int &E, int &m) {
    a = sw / 127.0f;
    E = -14;
    m = 0;
    if (!(a > 0.0f) || !(a < 1.0e30f)) return false;
    E = max(ilogbf(a), -14);
    m = (int)rintf(ldexpf(a, 10 - E));
    return true;
}

typedef _Float16 v2h __attribute__((ext_vector_type(2)));
// The remainders of 16 codes of one output row: r = Wd / u - m code with Wd = fp16(fp32(code a)), exact in fp16: |r| <= 127
// in units of u, and adding 1536 u leaves r in the low byte.  For a <= 515 (no Wd overflows); mu = m u = fp16(a).
// Bytes become floats as code + 128, which the multiply-add takes off again with the one rounding of the product itself.
__device__ __forceinline__ v4i digit_remainders(const v4i &codes, float a, _Float16 mu, _Float16 magic) {
    const float a128 = -128.0f * a;
    v4i out;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const uint32_t b = (uint32_t)codes[q] ^ 0x80808080u;
        uint32_t t[2];
#pragma unroll
        for (int p = 0; p < 2; p++) {
            const float f0 = (float)((b >> (16 * p)) & 255u), f1 = (float)((b >> (16 * p + 8)) & 255u);
            float w0 = fmaf(f0, a, a128), w1 = fmaf(f1, a, a128);
            asm("" : "+v"(w0), "+v"(w1));      // two roundings, fp32 and fp16, as everywhere
            const uint32_t biased = __builtin_amdgcn_perm(0x64646464u, b, p ? 0x04030402u : 0x04010400u);    // 1024 + code + 128
            const v2h c = *(const v2h *)&biased - (v2h){(_Float16)1152.0f, (_Float16)1152.0f}, wd = {(_Float16)w0, (_Float16)w1};
            v2h r = __builtin_elementwise_fma(c, (v2h){(_Float16)-mu, (_Float16)-mu}, wd);
            r += (v2h){magic, magic};
            t[p] = *(const uint32_t *)&r;
        }
        out[q] = (int)__builtin_amdgcn_perm(t[1], t[0], 0x06040200);
    }
    return out;
}

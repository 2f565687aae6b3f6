// Decode-time linear for ONE row (batch-1 generation).  Every workgroup first turns the
// fp16 input row into int8 codes in LDS (optionally after a LayerNorm), then streams the
// int8 weight tiles of its 16-row panel from HBM once, 16 bytes per lane per load, and
// accumulates with v_dot4_i32_i8.  HBM-bound: every weight byte is read exactly once per
// token; the input row (a few tens of KB) comes from L2.
#include <stdlib.h>

#include <mutex>

#include "common.h"
#include "epilogue.h"

namespace {

__device__ __forceinline__ int byte_of(const v4i &w, int j) {
    int word = (j < 8) ? ((j < 4) ? w[0] : w[1]) : ((j < 12) ? w[2] : w[3]);
    return (int)(int8_t)((word >> ((j & 3) * 8)) & 0xff);
}

struct RowIn {
    const __half *x;            // the input row [K]
    const __half *ln_g, *ln_b;  // LayerNorm gain/bias (used by the LN variant)
    float eps;
    uint32_t theta_bits;
    // LN variant only: the row arrives as blockwise 8-bit codes (q8 non-null; x is then unused) and is decoded
    // while it is loaded; workgroup 0 stores the decoded fp16 row to q8_x_out for the residual that follows
    const uint8_t *q8;
    const float *q8_absmax;
    int q8_block;
    __half *q8_x_out;
    // optional copies for tests, written by workgroup 0 (each may be null)
    __half *a_out;              // LayerNorm output
    int8_t *xq_out;
    uint32_t *mask_out;
    float *sx_out;
};

static __device__ const CodeTable d_code_table = ps_make_code_table();

// The fp16 value of column k the linear sees: the input itself, or its LayerNorm.
template <bool LN>
__device__ __forceinline__ __half row_value(const RowIn &in, int k, double mean, double inv) {
    if (!LN) return in.x[k];
    const __half xk = in.q8 ? decode_q8(d_code_table.code, in.q8[k], in.q8_absmax[k / in.q8_block]) : in.x[k];
    return d2h_rn(((double)__half2float(xk) - mean) * inv * (double)__half2float(in.ln_g[k]) +
                  (double)__half2float(in.ln_b[k]));
}

// fp16 part of a 16-column group that contains outlier columns (rare path), in fp64
template <bool LN>
__device__ __forceinline__ double outlier_group(const v4i &w, uint32_t bits, const RowIn &in, int k0, double mean,
                                                double inv, float swd) {
    double o = 0.0;
    while (bits) {
        const int j = __ffs(bits) - 1;
        bits &= bits - 1;
        o += (double)__half2float(row_value<LN>(in, k0 + j, mean, inv)) * (double)dequant_w16(byte_of(w, j), swd);
    }
    return o;
}

constexpr int GEMV_GROUP = 512;      // 8 waves share one 16-row panel at a time

// Persistent-style one-row linear.  The grid is sized so that every workgroup is resident at
// once (up to two per compute unit) and owns a contiguous range of 16-row panels.  Each workgroup
//  1. (LN variant) normalises the row in fp64,
//  2. marks outlier columns (|v| >= threshold, compared as fp16 bit patterns, which order like
//     the magnitudes), takes the absolute maximum of the rest, writes int8 codes to LDS;
//     all of it from registers, once per workgroup,
//  3. streams its panels one after the other: the 8 waves split a panel's K/64 tiles in chunks of U
//     consecutive tiles; lane l holds row l%16 and the 16 columns of group l/16, so one wave
//     load is 1 KB contiguous; v_dot4_i32_i8 accumulates exactly.
// NG = 2: one workgroup of 16 waves per compute unit, two groups of 8 waves working on two panels at a
// time - the row is then prepared once per compute unit instead of twice, by twice the threads.
// While the row is prepared (4 to 9 us: its loads, three workgroup-wide reductions, the quantization) nothing else
// would keep HBM busy, so the waves request weights of their first panel ahead: one chunk into registers as soon
// as the row has arrived, then one more chunk at each of up to three later points of the preparation - NPF of them
// into a private LDS staging area (asynchronous copies), and, if NPF > 0, a last one into registers again.  One
// chunk per wave at a time: HBM delivers 16 waves x 4 KB per compute unit in about 2 us, and a wave that asks for
// more than the memory pipeline takes on stalls at the request until earlier data has arrived - the preparation
// then waits with it (all chunks requested at once: the preparation takes 2.5 to 5 us longer, nothing gained).
// CW: consecutive columns a thread takes at a time (MAXCH times).  8 for wide rows; 4 and 2 where the row has fewer than
// 8 columns per thread, so that all 8 waves share the preparation instead of two or four (24 blocks of K = 1024: a step of 658 -> 621 us).
template <int CW>
__device__ __forceinline__ void load_words(const __half *p, int (&w)[CW / 2]) {
    if constexpr (CW == 8) *(v4i *)w = *(const v4i *)p;
    else if constexpr (CW == 4) *(v2i *)w = *(const v2i *)p;
    else w[0] = *(const int *)p;
}
template <int CW>
__device__ __forceinline__ float word_half(const int (&w)[CW / 2], int e) {
    const unsigned short hb = (unsigned short)((uint32_t)w[e >> 1] >> ((e & 1) * 16));
    return __half2float(*(const __half *)&hb);
}

template <int U, int MAXCH, bool LN, int NG, int NPF, int CW>
__global__ void __launch_bounds__(GEMV_GROUP * NG) k_gemv_row(LinearW w, RowIn in, OutDesc o,
                                                             const SessTable *__restrict__ sess, int panels_per_wg,
                                                             int panels_extra) {
    constexpr int GEMV_THREADS = GEMV_GROUP * NG, NWV = GEMV_THREADS / 64;
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ double smd[NWV], smq[NWV];
    __shared__ int smi[NWV];
    const int K = w.K, KT = K >> 6, nch8 = K / CW;
    int8_t *xs = (int8_t *)lds;                               // K codes
    uint8_t *m8 = (uint8_t *)(lds + K);                       // K/8 mask bytes = K/16 group masks
    int *red_i = (int *)(lds + K + K / 8);                    // [2 parities][NG groups][8 waves][16]
    double *red_f = (double *)(red_i + 256 * NG);             // same shape
    const uint16_t *ms = (const uint16_t *)m8;
    const bool first = blockIdx.x == 0;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, kg = lane >> 4;
    const int grp = wave >> 3, tw = wave & 7;                 // group of 8 waves, wave inside the group
    // this workgroup's panels: [p0, p0 + np)
    const int g = blockIdx.x;
    const int np = panels_per_wg + (g < panels_extra ? 1 : 0);
    const int p0 = g * panels_per_wg + min(g, panels_extra);
    const int nchunks = KT / U;

    // 1. the row (with LayerNorm also the gain and the bias): requested first, kept in registers
    int xr[LN ? MAXCH : 1][CW / 2], gr[LN ? MAXCH : 1][CW / 2], br[LN ? MAXCH : 1][CW / 2];
    int vals[MAXCH][CW / 2];
    if (LN) {
#pragma unroll
        for (int i = 0; i < MAXCH; i++) {
            const int c = threadIdx.x + GEMV_THREADS * i;
            if (c < nch8) {
                if (in.q8) {                        // uniform over the grid; the CW columns share a codec block
                    uint32_t qq[2] = {0u, 0u};
                    if constexpr (CW == 8) *(uint2 *)qq = *(const uint2 *)(in.q8 + c * CW);
                    else if constexpr (CW == 4) qq[0] = *(const uint32_t *)(in.q8 + c * CW);
                    else qq[0] = *(const uint16_t *)(in.q8 + c * CW);
                    const float am = in.q8_absmax[(c * CW) / in.q8_block];
#pragma unroll
                    for (int e = 0; e < CW; e += 2) {
                        const __half d0 = decode_q8(d_code_table.code, (qq[e >> 2] >> ((e & 3) * 8)) & 255u, am);
                        const __half d1 = decode_q8(d_code_table.code, (qq[e >> 2] >> ((e & 3) * 8 + 8)) & 255u, am);
                        xr[i][e >> 1] = (int)((uint32_t)__half_as_ushort(d0) | (uint32_t)__half_as_ushort(d1) << 16);
                        if (first) *(int *)(in.q8_x_out + c * CW + e) = xr[i][e >> 1];
                    }
                } else {
                    load_words<CW>(in.x + c * CW, xr[i]);
                }
                load_words<CW>(in.ln_g + c * CW, gr[i]);
                load_words<CW>(in.ln_b + c * CW, br[i]);
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < MAXCH; i++) {
            const int c = threadIdx.x + GEMV_THREADS * i;
            if (c < nch8) load_words<CW>(in.x + c * CW, vals[i]);
        }
    }
    // A compute unit serves its waves' requests in order and takes on only so many ahead of the data (a wave that
    // asks for more stalls at the request).  So: wait until the row has ARRIVED, request one chunk of weights per
    // wave into registers, and request the next chunks one at a time at later points of the row preparation, when
    // the chunk before has landed.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    v4i wv[U];
    // (an LDS object of its own: the compiler then knows that the prologue's other LDS traffic cannot touch it and
    // does not wait for the copies in front of every LDS access)
    __shared__ __align__(16) unsigned char stage_buf[NPF > 0 ? 8 * NG * NPF * U * 1024 : 16];
    unsigned char *stage = stage_buf + (size_t)wave * NPF * (U * 1024);
    const int8_t *panel0 = w.wt + (size_t)(p0 + min(grp, np - 1)) * KT * 1024;
    {
        const v4i *wp = (const v4i *)panel0 + lane;
#pragma unroll
        for (int u = 0; u < U; u++) wv[u] = __builtin_nontemporal_load(wp + (size_t)(min(tw, nchunks - 1) * U + u) * 64);
    }
    // buffer form of the copy (descriptor = this wave's first panel, bounds-checked by the hardware): the flat form
    // makes the compiler wait for ALL loads at the next wait of any kind
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)panel0, 0, KT * 1024, 0x00020000);
    // Request point k = 1, 2, 3 (in program order) asks for chunk tw + 8 k of the first panel: into staging slot
    // k - 1 while k <= NPF, into the second register set at k = NPF + 1; the host chooses NPF so that the chunks exist.
    v4i wv2[NPF > 0 ? U : 1];
    auto request_point = [&](auto kc) {
        constexpr int k = decltype(kc)::value;
        if constexpr (NPF > 0 && k <= NPF) {
#pragma unroll
            for (int u = 0; u < U; u++)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void *)(stage + (size_t)((k - 1) * U + u) * 1024),
                                                         16, lane * 16, ((tw + 8 * k) * U + u) * 1024, 0, 2 /* non-temporal */);
        } else if constexpr (NPF > 0 && k == NPF + 1) {
            const v4i *wp = (const v4i *)panel0 + lane;
#pragma unroll
            for (int u = 0; u < U; u++) wv2[u] = __builtin_nontemporal_load(wp + (size_t)((tw + 8 * k) * U + u) * 64);
        }
    };
    __builtin_amdgcn_sched_barrier(0);

    for (int i = threadIdx.x; i < K / 32; i += GEMV_THREADS) ((uint32_t *)m8)[i] = 0u;
    double mean = 0.0, inv = 0.0;
    if (LN) {
        // Both moments in one pass and one reduction.  The squares of fp16 values are exact in fp64 and the sums
        // carry 1e-16 of relative error, so the variance as "mean of squares minus squared mean" is as good as
        // the two-pass form unless the mean dwarfs the spread by a factor of 1e6, which a hidden state never does.
        double s = 0.0, q = 0.0;
#pragma unroll
        for (int i = 0; i < MAXCH; i++) {
            if (threadIdx.x + GEMV_THREADS * i < nch8) {
#pragma unroll
                for (int e = 0; e < CW; e++) { const double a = (double)word_half<CW>(xr[i], e); s += a; q = fma(a, a, q); }
            }
        }
        s = wave_sum(s);
        q = wave_sum(q);
        if (lane == 0) { smd[wave] = s; smq[wave] = q; }
        lds_barrier();
        request_point(std::integral_constant<int, 1>());   // (the first chunk has landed by now)
        s = q = 0.0;
#pragma unroll
        for (int i = 0; i < NWV; i++) { s += smd[i]; q += smq[i]; }
        mean = s / (double)K;
        inv = rsqrt_f64(fmax(q / (double)K - mean * mean, 0.0) + (double)in.eps);
    } else {
        lds_barrier();        // mask bytes cleared before anybody sets one
    }

    // detect + absolute maximum over regular columns, 8 columns per register quad
    uint32_t mreg = 0, obits[MAXCH];
#pragma unroll
    for (int i = 0; i < MAXCH; i++) {
        const int c = threadIdx.x + GEMV_THREADS * i;
        if (c < nch8) {
            if (LN) {
                __half out[CW];
#pragma unroll
                for (int e = 0; e < CW; e++)
                    out[e] = d2h_rn(((double)word_half<CW>(xr[i], e) - mean) * inv * (double)word_half<CW>(gr[i], e) + (double)word_half<CW>(br[i], e));
#pragma unroll
                for (int e = 0; e < CW; e += 2) {
                    vals[i][e >> 1] = (int)((uint32_t)__half_as_ushort(out[e]) | (uint32_t)__half_as_ushort(out[e + 1]) << 16);
                    if (first && in.a_out) *(int *)(in.a_out + c * CW + e) = vals[i][e >> 1];
                }
            }
            uint32_t cm = 0;
#pragma unroll
            for (int e = 0; e < CW / 2; e++) cm = pk_max_u16(cm, (uint32_t)vals[i][e] & 0x7fff7fffu);
            const uint32_t cmax = max(cm & 0xffffu, cm >> 16);
            obits[i] = 0;
            if (cmax >= in.theta_bits) {
                uint32_t byte = 0;
#pragma unroll
                for (int e = 0; e < CW; e++) {
                    const uint32_t a = ((uint32_t)vals[i][e >> 1] >> ((e & 1) * 16)) & 0x7fffu;
                    if (a >= in.theta_bits) byte |= 1u << e; else mreg = max(mreg, a);
                }
                obits[i] = byte;
                if constexpr (CW == 8) m8[c] = (uint8_t)byte;
                else atomicOr((uint32_t *)m8 + (c * CW >> 5), byte << (c * CW & 31));
            } else {
                mreg = max(mreg, cmax);
            }
        }
        if (LN && i == (MAXCH - 1) / 2) request_point(std::integral_constant<int, 2>());   // halfway through the arithmetic
    }
    mreg = wave_max(mreg);
    if (lane == 0) smi[wave] = (int)mreg;
    lds_barrier();
    request_point(std::integral_constant<int, LN ? 3 : 1>());
#pragma unroll
    for (int i = 0; i < NWV; i++) mreg = max(mreg, (uint32_t)smi[i]);
    const unsigned short sb = (unsigned short)mreg;
    const float s_x = __half2float(*(const __half *)&sb);
    const float r = s_x > 0.0f ? 127.0f / s_x : 0.0f;
    float neg0 = -0.0f;
    asm("" : "+v"(neg0));
#pragma unroll
    for (int i = 0; i < MAXCH; i++) {
        const int c = threadIdx.x + GEMV_THREADS * i;
        if (c < nch8) {
            // all codes first, straight-line; the codes of outlier columns are then cleared byte by byte in the
            // packed words (a test per element compiles to a branch per element, and a chunk with outlier
            // columns is rare)
            // (fp32 product straight from fp16 by a multiply-add with -0, rounded by an addition that leaves the integer
            // in the low byte; |x r| <= 127.00002 for regular columns)
            uint32_t t[CW], o2[2] = {0u, 0u};
#pragma unroll
            for (int e = 0; e < CW; e++) t[e] = __float_as_uint(fmaf(word_half<CW>(vals[i], e), r, neg0) + 12582912.0f);
#pragma unroll
            for (int e = 0; e < CW; e += 4) {
                const uint32_t lo = __builtin_amdgcn_perm(t[e + 1], t[e], 0x0c0c0400);
                if constexpr (CW == 2) o2[0] = lo;
                else o2[e >> 2] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(t[(e + 3) % CW], t[(e + 2) % CW], 0x0c0c0400), lo, 0x05040100);
            }
            if (obits[i]) {
#pragma unroll
                for (int e = 0; e < CW; e++) o2[e >> 2] &= ~(((obits[i] >> e) & 1u) * (0xffu << (8 * (e & 3))));
            }
            if constexpr (CW == 8) *(uint2 *)(xs + c * 8) = *(const uint2 *)o2;
            else if constexpr (CW == 4) *(uint32_t *)(xs + c * 4) = o2[0];
            else *(uint16_t *)(xs + c * 2) = (uint16_t)o2[0];
        }
        if (!LN && i == (MAXCH - 1) / 2) request_point(std::integral_constant<int, 2>());  // halfway through the quantization
    }
    lds_barrier();
    if (first) {
        if (in.sx_out && threadIdx.x == 0) *in.sx_out = s_x;
        if (in.xq_out) for (int i = threadIdx.x; i < K / 16; i += GEMV_THREADS) ((v4i *)in.xq_out)[i] = ((const v4i *)xs)[i];
        if (in.mask_out) for (int i = threadIdx.x; i < K / 32; i += GEMV_THREADS) in.mask_out[i] = ((const uint32_t *)m8)[i];
    }

    for (int it = 0; it * NG < np; it++) {
        const bool active = it * NG + grp < np;        // the last round of an odd count leaves one group idle
        const int p = p0 + min(it * NG + grp, np - 1);
        const v4i *wp = (const v4i *)(w.wt + (size_t)p * KT * 1024) + lane;
        const int n = p * 16 + (lane & 15);
        const float swd = w.sw[n] / 127.0f;
        int acc = 0;
        double outl = 0.0;
        if (active) {
            for (int c = tw, j = 0; c < nchunks; c += 8, j++) {
                // the first panel's first chunks were requested during the row preparation: registers, staging area, registers
                // chunks requested ahead besides the first: the staged ones, then the second register set
                constexpr int NPOINTS = LN ? 3 : 2, NSTAGED = NPF < NPOINTS ? NPF : NPOINTS;
                constexpr bool REG2 = NPF > 0 && NPF + 1 <= NPOINTS;
                constexpr int NAHEAD = NSTAGED + (REG2 ? 1 : 0);
                if (it > 0 || j > NAHEAD) {
#pragma unroll
                    for (int u = 0; u < U; u++) wv[u] = __builtin_nontemporal_load(wp + (size_t)(c * U + u) * 64);
                } else if (REG2 && j == NAHEAD) {
#pragma unroll
                    for (int u = 0; u < U; u++) wv[u] = wv2[u];
                } else if (j > 0) {
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's own copies have landed
#pragma unroll
                    for (int u = 0; u < U; u++) wv[u] = *(const v4i *)(stage + (size_t)((j - 1) * U + u) * 1024 + lane * 16);
                }
#pragma unroll
                for (int u = 0; u < U; u++) {
                    const int kt = c * U + u;
                    const v4i xv = *(const v4i *)(xs + kt * 64 + kg * 16);
                    acc = __builtin_amdgcn_sdot4(wv[u][0], xv[0], acc, false);
                    acc = __builtin_amdgcn_sdot4(wv[u][1], xv[1], acc, false);
                    acc = __builtin_amdgcn_sdot4(wv[u][2], xv[2], acc, false);
                    acc = __builtin_amdgcn_sdot4(wv[u][3], xv[3], acc, false);
                    const uint32_t bits = ms[kt * 4 + kg];
                    if (bits) outl += outlier_group<LN>(wv[u], bits, in, kt * 64 + kg * 16, mean, inv, swd);
                }
            }
            for (int kt = nchunks * U + tw; kt < KT; kt += 8) {
                const v4i w1 = __builtin_nontemporal_load(wp + (size_t)kt * 64);
                const v4i xv = *(const v4i *)(xs + kt * 64 + kg * 16);
                acc = __builtin_amdgcn_sdot4(w1[0], xv[0], acc, false);
                acc = __builtin_amdgcn_sdot4(w1[1], xv[1], acc, false);
                acc = __builtin_amdgcn_sdot4(w1[2], xv[2], acc, false);
                acc = __builtin_amdgcn_sdot4(w1[3], xv[3], acc, false);
                const uint32_t bits = ms[kt * 4 + kg];
                if (bits) outl += outlier_group<LN>(w1, bits, in, kt * 64 + kg * 16, mean, inv, swd);
            }
        }
        acc = swap_sum<32>(swap_sum<16>(acc));
        outl = swap_reduce<32>(swap_reduce<16>(outl, add_f64), add_f64);
        int *ri = red_i + ((it & 1) * NG + grp) * 128;
        double *rf = red_f + ((it & 1) * NG + grp) * 128;
        if (lane < 16) { ri[tw * 16 + lane] = acc; rf[tw * 16 + lane] = outl; }
        __syncthreads();
        if (active && tw == 0 && lane < 16) {          // lanes 0..15 of a group's first wave finish the 16 rows
            int a = 0;
            double f = 0.0;
#pragma unroll
            for (int i = 0; i < 8; i++) { a += ri[i * 16 + lane]; f += rf[i * 16 + lane]; }
            emit_output(o, sess, w.N, 0, n, a, f, s_x / 127.0f, swd, __half2float(w.bias[n]));
        }
    }
}

template <int U, int MAXCH, int NG, int NPF, int CW>
hipError_t launch4(bool ln, const LinearW &w, const RowIn &in, const OutDesc &o, const SessTable *sess, int G, int per,
                   int extra, size_t base, size_t lds, size_t budget, hipStream_t st) {
    auto kern = ln ? k_gemv_row<U, MAXCH, true, NG, NPF, CW> : k_gemv_row<U, MAXCH, false, NG, NPF, CW>;
    if (base > 64 * 1024) {
        static std::mutex attr_lock;
        static bool attr_set[2] = {false, false};
        std::lock_guard<std::mutex> hold(attr_lock);
        if (!attr_set[ln]) {
            hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(budget - (lds - base)));
            if (e != hipSuccess) return e;
            attr_set[ln] = true;
        }
    }
    kern<<<G, GEMV_GROUP * NG, base, st>>>(w, in, o, sess, per, extra);
    return hipGetLastError();
}

template <int U, int MAXCH, int NG, int CW = 8>
hipError_t launch3(bool ln, const LinearW &w, const RowIn &in, const OutDesc &o, const SessTable *sess, hipStream_t st) {
    const size_t base = ((size_t)w.K + w.K / 8 + 256 * 12 * NG + 15) & ~(size_t)15;
    // staging for the weight chunks requested before the row is prepared: up to two chunks per wave, as far as every
    // wave has such chunks in its first panel and the compute unit's 160 KB of LDS allow (one 16-wave workgroup
    // per unit, or two of 8 waves)
    const size_t budget = (NG == 2 ? 160 : 80) * 1024 - 1024, per_chunk = (size_t)8 * NG * U * 1024;
    const int nchunks = w.K / 64 / U;
    int npf = base + per_chunk <= budget ? (int)min((size_t)2, (budget - base) / per_chunk) : 0;
    if (!ln) npf = min(npf, 1);                         // without LayerNorm there are two request points, with it three
    npf = CW < 8 ? 0 : max(0, min(npf, nchunks / 8 - 2));   // every wave's chunks tw + 8 k, k <= npf + 1, must exist
    const size_t lds = base + npf * per_chunk;
    // one resident round: at most 1024 threads' worth of workgroups per compute unit twice over (512 groups of
    // 8 waves); prefer a split of the panels without remainder
    const int panels = w.N / 16, units = panels / NG, max_wg = 512 / NG;
    int G = min(max_wg, units);
    for (int cand = G; cand >= max(1, (G * 3) / 4); cand--)
        if (units % cand == 0) { G = cand; break; }
    const int per = panels / G, extra = panels % G;
    if (lds > budget) return hipErrorInvalidValue;      // K <= 65536 (base at most 86 KB) always fits
    if constexpr (CW == 8) {
        if (npf == 2) return launch4<U, MAXCH, NG, 2, CW>(ln, w, in, o, sess, G, per, extra, base, lds, budget, st);
        if (npf == 1) return launch4<U, MAXCH, NG, 1, CW>(ln, w, in, o, sess, G, per, extra, base, lds, budget, st);
    }
    return launch4<U, MAXCH, NG, 0, CW>(ln, w, in, o, sess, G, per, extra, base, lds, budget, st);
}

template <int U, int MAXCH>
hipError_t launch2(bool ln, const LinearW &w, const RowIn &in, const OutDesc &o, const SessTable *sess, hipStream_t st) {
    // large linears: one 16-wave workgroup per compute unit (the row is prepared once per unit)
    const int panels = w.N / 16;
    if (panels % 2 == 0 && panels >= 448 && MAXCH >= 4) return launch3<U, (MAXCH + 1) / 2, 2>(ln, w, in, o, sess, st);
    return launch3<U, MAXCH, 1>(ln, w, in, o, sess, st);
}

template <int U>
hipError_t launch1(bool ln, const LinearW &w, const RowIn &in, const OutDesc &o, const SessTable *sess, hipStream_t st) {
    const int per_thread = (w.K / 8 + GEMV_GROUP - 1) / GEMV_GROUP;   // 8-column chunks a thread of an 8-wave workgroup holds in registers
    if (w.K <= 2 * GEMV_GROUP) return launch3<U, 1, 1, 2>(ln, w, in, o, sess, st);
    if (w.K <= 4 * GEMV_GROUP) return launch3<U, 1, 1, 4>(ln, w, in, o, sess, st);
    if (per_thread <= 1) return launch2<U, 1>(ln, w, in, o, sess, st);
    if (per_thread <= 4) return launch2<U, 4>(ln, w, in, o, sess, st);
    return launch2<U, 16>(ln, w, in, o, sess, st);
}

}  // namespace

hipError_t ps_gemv_row(const LinearW &w, const __half *x, const __half *ln_g, const __half *ln_b, float eps,
                       float theta, const RowDebug &dbg, const OutDesc &o, const SessTable *sess, const QuantIn *qin,
                       hipStream_t st) {
    RowIn in;
    in.x = x; in.ln_g = ln_g; in.ln_b = ln_b; in.eps = eps; in.theta_bits = ps_theta_to_bits(theta);
    in.q8 = nullptr; in.q8_absmax = nullptr; in.q8_block = 1; in.q8_x_out = nullptr;
    if (qin) {
        if (!ln_g) return hipErrorInvalidValue;   // codes are only decoded in front of a LayerNorm
        in.q8 = qin->q; in.q8_absmax = qin->absmax; in.q8_block = qin->block; in.q8_x_out = qin->x_out;
    }
    in.a_out = dbg.a_out; in.xq_out = dbg.xq_out; in.mask_out = dbg.mask_out; in.sx_out = dbg.sx_out;
    const bool ln = ln_g != nullptr;
    const int KT = w.K / 64;
    // tiles per chunk: 4 where the tile count allows (8 measured no faster and costs registers)
    if (KT % 32 == 0) return launch1<4>(ln, w, in, o, sess, st);
    if (KT % 16 == 0) return launch1<2>(ln, w, in, o, sess, st);
    return launch1<1>(ln, w, in, o, sess, st);
}

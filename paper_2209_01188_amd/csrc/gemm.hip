// Batched-decode linear (2 <= M <= 64 rows) on the matrix cores.  HBM bound: every weight tile is
// streamed once.  Regular columns: int8 x int8 -> int32 with v_mfma_i32_16x16x64_i8.  Outlier
// columns are added exactly, inside the loop, from the weight bytes already in registers: on a
// 64-column tile that holds outliers, each of the four 16-column lane groups hands its next outlier
// column to one k-slot of v_mfma_f64_16x16x4_f64 (products of fp16 values are exact in fp64).
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <mutex>

#include "common.h"
#include "epilogue.h"
#include "gemm_digits.h"

namespace {

__device__ __forceinline__ int byte_of16(const v4i &w, int j) {
    const int word = (j < 8) ? ((j < 4) ? w[0] : w[1]) : ((j < 12) ? w[2] : w[3]);
    return (int)(int8_t)((word >> ((j & 3) * 8)) & 0xff);
}
__device__ __forceinline__ float half_of8(const v4i &x, int r) {   // r-th of the 8 halves in x
    const int word = (r < 4) ? ((r < 2) ? x[0] : x[1]) : ((r < 6) ? x[2] : x[3]);
    return __half2float(__ushort_as_half((unsigned short)((word >> ((r & 1) * 16)) & 0xffff)));
}

struct NoDigits {};
template <bool DIG>
auto digit_arg(const DigitCall &dc) {
    if constexpr (DIG) return dc;
    else return NoDigits{};
}

// One workgroup = WVK waves on WN consecutive 16-row weight panels; wave wk takes chunks of UK
// consecutive k-tiles (chunk c = wk, wk + WVK, ...) for MT token tiles of 16 rows, so a token tile
// fetched once meets WN weight tiles.  Weights are the A operand (lane l: row l%16, 16 codes of
// column group l/16), tokens the B operand in the same tile order: D[lane][r] is output row
// 4*(l/16)+r of token l%16.  The next chunk's operands are requested before the current chunk is
// multiplied.  xo: per token tile and k-tile, lane (token, column group) holds the values of the
// group's first 8 outlier columns (written by ps_rowquant_tiled); a group with more takes the rest
// from X.  The waves' partial sums meet in LDS once; up to four waves finish the (panel, token tile)
// pairs.
template <int WN, int MT, int UK, int WVK, bool DIG>
__global__ void __launch_bounds__(64 * WVK)
k_gemm(LinearW w, const int8_t *__restrict__ xq_tiled, const int8_t *__restrict__ xo_tiled,
       const uint32_t *__restrict__ mask, const __half *__restrict__ X, const float *__restrict__ sx, int M,
       OutDesc o, const SessTable *__restrict__ sess, typename std::conditional<DIG, DigitCall, NoDigits>::type dc) {
    extern __shared__ __align__(16) unsigned char lds[];
    if constexpr (DIG) {                             // (at most 64 rows)
        const int l = threadIdx.x & 63;
        if (!__ballot(l < M && dc.rowstate[l] != PS_ROWS_IN_DIGITS)) {
            digit_linear(w, xq_tiled, mask, X, sx, M, o, sess, dc, lds);
            return;
        }
        if ((int)blockIdx.x * 16 * WN >= w.N) return;
    }
    const int K = w.K, KT = K >> 6, N = w.N;
    if (gridDim.y > 1) {
        // a call of more rows than MT token tiles: blockIdx.y takes MT of them
        const int r0 = blockIdx.y * 16 * MT;
        const size_t at = (size_t)r0 * N;
        xq_tiled += (size_t)(r0 >> 4) * KT * 1024;
        xo_tiled += (size_t)(r0 >> 4) * KT * 1024;
        X += (size_t)r0 * K;
        sx += r0;
        M = min(16 * MT, M - r0);
        if (o.scatter) {
            o.t0 = r0;
        } else {
            o.y += at;
            if (o.resid) o.resid += at;
            if (o.pre_out) o.pre_out += at;
        }
        if (o.acc_out) o.acc_out += at;
    }
    const int MTT = (M + 15) >> 4;
    const int wk = threadIdx.x >> 6, lane = threadIdx.x & 63, row = lane & 15, kg = lane >> 4;
    const int nt0 = blockIdx.x * WN;

    v4i acc[WN][MT];
    v4d od[WN][MT];
#pragma unroll
    for (int p = 0; p < WN; p++)
#pragma unroll
        for (int j = 0; j < MT; j++) {
            acc[p][j] = (v4i){0, 0, 0, 0};
            od[p][j] = (v4d){0.0, 0.0, 0.0, 0.0};
        }
    const int8_t *wbase = w.wt + (size_t)nt0 * KT * 1024 + lane * 16;
    float swd[WN];
#pragma unroll
    for (int p = 0; p < WN; p++) swd[p] = w.sw[(nt0 + p) * 16 + row] / 127.0f;
    size_t xoff[MT];
    const __half *xrow[MT];
#pragma unroll
    for (int j = 0; j < MT; j++) {
        const int mt = min(j, MTT - 1);
        xoff[j] = (size_t)mt * KT * 1024 + lane * 16;
        xrow[j] = X + (size_t)min(mt * 16 + row, M - 1) * K + kg * 16;
    }
    const uint64_t *mask64 = (const uint64_t *)mask;
    const int nch = (KT + UK - 1) / UK;

    struct Buf {
        v4i w[UK][WN], x[UK][MT], xo[UK][MT];
        uint64_t m[UK];
    };
    auto load = [&](Buf &b, int c) {
#pragma unroll
        for (int u = 0; u < UK; u++) {
            const int kt = min(c * UK + u, KT - 1);
#pragma unroll
            for (int p = 0; p < WN; p++)
                b.w[u][p] = __builtin_nontemporal_load((const v4i *)(wbase + ((size_t)p * KT + kt) * 1024));
#pragma unroll
            for (int j = 0; j < MT; j++) b.x[u][j] = *(const v4i *)(xq_tiled + xoff[j] + (size_t)kt * 1024);
        }
#pragma unroll
        for (int u = 0; u < UK; u++) {
            const int kt = min(c * UK + u, KT - 1);
            b.m[u] = mask64[kt];                              // same for the whole wave
#pragma unroll
            for (int j = 0; j < MT; j++) b.xo[u][j] = (v4i){0, 0, 0, 0};
            if (b.m[u]) {
#pragma unroll
                for (int j = 0; j < MT; j++) b.xo[u][j] = *(const v4i *)(xo_tiled + xoff[j] + (size_t)kt * 1024);
            }
        }
    };
    auto compute = [&](const Buf &b, int c) {
#pragma unroll
        for (int u = 0; u < UK; u++) {
            const int kt = c * UK + u;
            if (kt >= KT) break;                              // ragged last chunk
#pragma unroll
            for (int p = 0; p < WN; p++)
#pragma unroll
                for (int j = 0; j < MT; j++)
                    acc[p][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(b.w[u][p], b.x[u][j], acc[p][j], 0, 0, 0);
            const uint64_t mbits = b.m[u];
            if (mbits) {
                // outlier columns of this tile, exactly: round r takes the r-th outlier column of each of
                // the four 16-column groups into one k-slot of the fp64 instruction
                uint32_t gb = (uint32_t)(mbits >> (kg * 16)) & 0xffffu;
                const int rounds =
                    max(max(__popc((uint32_t)mbits & 0xffffu), __popc((uint32_t)(mbits >> 16) & 0xffffu)),
                        max(__popc((uint32_t)(mbits >> 32) & 0xffffu), __popc((uint32_t)(mbits >> 48))));
                for (int r = 0; r < rounds; r++) {
                    const bool have = gb != 0;
                    const int jcol = have ? __ffs(gb) - 1 : 0;
                    gb &= gb - 1;
                    double a[WN];
#pragma unroll
                    for (int p = 0; p < WN; p++)
                        a[p] = have ? (double)dequant_w16(byte_of16(b.w[u][p], jcol), swd[p]) : 0.0;
#pragma unroll
                    for (int j = 0; j < MT; j++) {
                        float xv = r < 8 ? half_of8(b.xo[u][j], r) : __half2float(xrow[j][kt * 64 + jcol]);
                        const double bx = have ? (double)xv : 0.0;
#pragma unroll
                        for (int p = 0; p < WN; p++)
                            od[p][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[p], bx, od[p][j], 0, 0, 0);
                    }
                }
            }
        }
    };

    Buf A, B;
    int c = wk;
    if (c < nch) load(A, c);
    while (c < nch) {
        const int c1 = c + WVK, c2 = c1 + WVK;
        if (c1 < nch) load(B, c1);
        compute(A, c);
        if (c2 < nch) load(A, c2);
        if (c1 < nch) compute(B, c1);
        c = c2;
    }

    // The waves' partial sums meet in LDS, up to four (panel, token tile) pairs at a time; one wave per
    // pair adds them in wave order (the fp64 terms are exact products of fp16 values) and finishes it.
    constexpr int G = WN * MT, NPP = G < 4 ? G : 4;
    v4i *ri = (v4i *)lds;                                             // [WVK][NPP][64]
    v4d *rf = (v4d *)(lds + (size_t)WVK * NPP * 64 * 16);             // [WVK][NPP][64]
#pragma unroll
    for (int g0 = 0; g0 < G; g0 += NPP) {
        if (g0) __syncthreads();
#pragma unroll
        for (int i = 0; i < NPP; i++) {
            ri[(wk * NPP + i) * 64 + lane] = acc[(g0 + i) / MT][(g0 + i) % MT];
            rf[(wk * NPP + i) * 64 + lane] = od[(g0 + i) / MT][(g0 + i) % MT];
        }
        __syncthreads();
        if (wk >= NPP) continue;
        const int p = (g0 + wk) / MT, j = (g0 + wk) % MT;
        if (j >= MTT) continue;                                         // wave-uniform
        v4i a = ri[wk * 64 + lane];
        v4d f = rf[wk * 64 + lane];
        for (int s = 1; s < WVK; s++) {
            a += ri[(s * NPP + wk) * 64 + lane];
            f += rf[(s * NPP + wk) * 64 + lane];
        }
        // the fp64 instruction returns row 4r + g in register r of lane group g, the int8 one row 4g + r:
        // transpose the 4 x 4 (group, register) block among the four lanes that share a token
        v4d ft;
#pragma unroll
        for (int r = 0; r < 4; r++) {
            double v = 0.0;
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const double t = __shfl(f[q], row + 16 * r);
                if (q == kg) v = t;
            }
            ft[r] = v;
        }
        const int t = j * 16 + row;
        if (t < M) emit_output4(o, sess, N, t, (nt0 + p) * 16 + 4 * kg, a, ft, sx[t] / 127.0f, w.sw, w.bias);
    }
}

template <int WN, int MT, int UK, int WVK = 8, bool DIG = false>
hipError_t launch(const LinearW &w, const int8_t *xq_tiled, const int8_t *xo_tiled, const uint32_t *mask,
                  const __half *X, const float *sx, int M, const OutDesc &o, const SessTable *sess, const DigitCall &dc, hipStream_t st) {
    constexpr int G = WN * MT, NPP = G < 4 ? G : 4;
    constexpr size_t sums = (size_t)WVK * NPP * 64 * (16 + 32), ring = DIG ? DIGIT_SLOTS * 10 * 1024 : 0;
    constexpr size_t lds = sums > ring ? sums : ring;        // up to 96 KB
    const int wgs = w.N / (16 * WN), digit_wgs = DIG ? digit_grid_x(w.N, M) * PS_DIGIT_SPLITS : 0;
    auto kern = k_gemm<WN, MT, UK, WVK, DIG>;
    static std::mutex attr_lock;
    static bool attr_set = false;
    std::lock_guard<std::mutex> hold(attr_lock);
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    kern<<<dim3(wgs > digit_wgs ? wgs : digit_wgs, (M + 16 * MT - 1) / (16 * MT)), 64 * WVK, lds, st>>>(w, xq_tiled, xo_tiled, mask, X, sx, M, o, sess, digit_arg<DIG>(dc));
    return hipGetLastError();
}

}  // namespace

// Narrower outputs belong to narrower blocks, whose inputs hold few outlier columns in a trained model, and there the calls that
// don't go to digits would pay for this form's registers and its eight waves (steps through two 10240-wide blocks with few outlier
// columns, 17, 32, 48 and 64 rows: 784 -> 791, 795 -> 807, 926 -> 937, 1032 -> 1056 us; where one in six or more is one they would
// gain: 929 -> 954, 1051 -> 972, 1680 -> 1435, 1924 -> 1524).  From 12288 on the former is 0 to 0.3 %, the latter up to a half.
// 16384 is the widest there is.  Up to 16 rows a column is rarely an outlier and the fp64 form's cost is half (one token tile).
bool ps_gemm_digits_applies(int N, int K, int M) { return M > 16 && M <= 64 && N >= 12288 && N <= 16384 && K >= 4096; }

// panels of 16 output rows per workgroup of ps_gemm: as many as still leave about one workgroup per compute unit
static int gemm_panels_per_wg(int N) {
    const int panels = N / 16;
    return (panels % 4 == 0 && panels / 4 >= 224) ? 4 : (panels % 2 == 0 && panels / 2 >= 224) ? 2 : 1;
}

// Microseconds of the 64-rows-per-workgroup form without its row kernels, and whether four waves per workgroup do better than
// eight.  Eight: one workgroup to a compute unit (registers, and local memory for the sums to meet in), in rounds of 256 that
// each walk the K/64 tiles in 3.4 us + 0.095 per tile with one panel, 5 us + 0.123 with two; four: two to a unit, rounds of
// 512 in 4 us + 0.18 per tile and 8 us + 0.22.  So four wherever eight would leave a second round nearly empty (128 rows:
// 3072 x 1024 with its row kernels 23.1 -> 20.5 us, 9216 x 3072 at 192 rows 55.3 -> 45.5, 16384 x 4096 at 64 rows 39.4 -> 34.9),
// eight in single rounds (1024 x 4096 at 128 rows: 21.8 against 24.8) and where their rounds come out even (24576 x 8192 at
// 64 rows: 75 against 81).
static double gemm_rows64_us(const LinearW &w, int M, int wn, bool &four) {
    const int groups = w.N / 16 / wn * ((M + 63) / 64);
    const double tiles = w.K / 64;
    const double t8 = (groups + 255) / 256 * (wn == 2 ? 5.0 + 0.123 * tiles : 3.4 + 0.095 * tiles);
    const double t4 = (groups + 511) / 512 * (wn == 2 ? 8.0 + 0.22 * tiles : 4.0 + 0.18 * tiles);
    four = t4 < t8;
    return fmin(t4, t8);
}

// The forms of 33 to 512 rows: 64 rows per workgroup as above, or 32.  32 rows: two panels and four waves, three workgroups to a
// compute unit, so rounds of 768 (2.75 us + 0.24 per tile), where 64 rows fill their rounds badly or their waves wait for each
// other: 6144 x 2048 at 128 rows 31.3 -> 24.4 us, 2048 x 2048 at 300 31.8 -> 24.0, 4096 x 16384 at 300 156 -> 136 (16384 x 4096 at
// 128 rows the other way round: 55.5 against 68.5); or one panel and sixteen waves in rounds of 256 (3.5 us + 0.06), where there
// are few panels and many tiles: 2048 x 8192 at 64 rows 27.9 -> 23.5, 1024 x 4096 at 128 22.1 -> 19.9.  On 72 linears of 1024- to 4096-wide
// blocks at 40 to 300 rows 5 % less, none more.
enum { ROWS64_8, ROWS64_4, ROWS32_4, ROWS32_16 };
static double gemm_rows_us(const LinearW &w, int M, int &form) {
    bool four;
    const int panels = w.N / 16, y = (M + 31) / 32;
    const double tiles = w.K / 64, us64 = gemm_rows64_us(w, M, gemm_panels_per_wg(w.N) > 1 ? 2 : 1, four);
    const double us4 = panels % 2 ? 1e30 : (panels / 2 * y + 767) / 768 * (2.75 + 0.24 * tiles), us16 = (panels * y + 255) / 256 * (3.5 + 0.06 * tiles);
    form = us64 <= us4 && us64 <= us16 ? (four ? ROWS64_4 : ROWS64_8) : us4 <= us16 ? ROWS32_4 : ROWS32_16;
    return fmin(us64, fmin(us4, us16));
}

// Rough times in microseconds of a linear with its row kernels, fitted to both forms measured on the four linears of
// blocks 1024 to 14336 wide at 65 to 512 rows with few outlier columns (the choice is 0.6 % behind the faster one on average).
// They know nothing of many: there blocks win, whose digit products cost the same for all, while the 64-row form grows with each
// (3072 x 3072 at 352 rows: 10 columns 37 us, in blocks 41; 460 columns 86 and 68).
// 64 rows per workgroup: see above, 13 us for the row kernels in front.  All rows go in one launch: charged by 64 rows, as
// when each 64 were a launch, narrow outputs went to the blocks too early (1024 x 1024 at 320 rows: 24 us in this form, 36 in
// blocks).
// From 2.1 to 2.6 million codes in the call it grows by 11 us (an XCD's L2 holds 4 MB, and the weights pass through it as well): 2048 x
// 8192 at 280, 300, 320 and 376 rows 53, 56, 59, 59 us where 46 were expected, in blocks 53, 54, 54, 54 (with half of the
// columns outliers 264 and 111).
// Output blocks: ps_gemm_lds_us.
// PETALS_SPAN_MIDSIZE=blocks / =chunks in the environment overrides the choice (tests run both ways).
bool ps_gemm_prefers_chunks(const LinearW &w, int M) {
    if (M <= 64 || M > PS_CHUNKED_ROWS_MAX) return false;
    if (const char *force = getenv("PETALS_SPAN_MIDSIZE")) {
        if (!strcmp(force, "blocks")) return false;
        if (!strcmp(force, "chunks")) return true;
    }
    int form;
    const double beyond_l2 = 11.0 * fmin(1.0, fmax(0.0, ((double)M * w.K - 2.1e6) / 0.5e6));
    return 13.0 + beyond_l2 + gemm_rows_us(w, M, form) < ps_gemm_lds_us(w.N, w.K, M);
}

hipError_t ps_gemm(const LinearW &w, const int8_t *xq_tiled, const int8_t *xo_tiled, const uint32_t *mask,
                   const __half *X, const float *sx, int M, const OutDesc &o, const SessTable *sess, const DigitCall &dc, hipStream_t st) {
    const int panels = w.N / 16, wn = gemm_panels_per_wg(w.N);
#define PS_GEMM_CASE(WN_, MT_, UK_) return launch<WN_, MT_, UK_>(w, xq_tiled, xo_tiled, mask, X, sx, M, o, sess, dc, st)
    // Up to 32 rows: four waves per workgroup, two workgroups to a compute unit, where eight (one to a unit by their
    // registers) would leave at least half of the units idle in the last of an odd number of rounds of 256 (2, 3 or 4 panels per
    // workgroup, QKV of blocks 2048 to 8192 wide at 24 rows 19.0 -> 17.5, 28.4 -> 26.4, 56.2 -> 52.1 us; 57344 x 12288 8 % less).
    // Not where that round is fuller (43008 x 14336: 123 against 139), nor with an even number of rounds: rounds of 512 end with
    // a nearly empty one themselves (40960 x 10240 at 8 rows 82 against 95, QKV of a 12288-wide block at 24 rows 105 against 118;
    // only inputs of less than some 3000 columns gain there, 4 to 18 %, and no block's up or QKV linear has them).
    const int wgs = panels / wn, rest = (wgs - 1) % 512 + 1;
    const bool four32 = rest > 256 && rest <= 384;
#define PS_GEMM_CASE4(WN_, MT_, UK_) \
    do { \
        if (four32) return launch<WN_, MT_, UK_, 4>(w, xq_tiled, xo_tiled, mask, X, sx, M, o, sess, dc, st); \
        PS_GEMM_CASE(WN_, MT_, UK_); \
    } while (0)
    if (M <= 16) {
        // one panel per workgroup (narrow outputs): 16 waves split the k-tiles, twice the weight bytes in flight per
        // compute unit (C3, 8 rows: down 2.85 -> 3.2 TB/s, dense 1.5 -> 1.65 TB/s; with 2 panels 16 waves are slower)
        // - eight where a second round of 16 waves would be mostly empty (8 rows: 5120 x 5120 21.6 -> 18.8 us, 6144 x 24576 51.1 -> 49.0)
        if (wn == 1 && w.K >= 4096 && four32) return launch<1, 1, 2, 8>(w, xq_tiled, xo_tiled, mask, X, sx, M, o, sess, dc, st);
        if (wn == 1 && w.K >= 4096) return launch<1, 1, 2, 16>(w, xq_tiled, xo_tiled, mask, X, sx, M, o, sess, dc, st);
        // small matrices (C3: 50-67 MB, 13-16 us per launch) do better with two workgroups per compute unit and
        // short chunks (up 3.5 -> 3.8, QKV 3.2 -> 3.25 TB/s); large ones with four panels per workgroup
        if (wn == 4 && panels / 4 < 448 && (size_t)w.N * w.K <= ((size_t)1 << 27)) PS_GEMM_CASE(2, 1, 2);
        if (wn == 4) PS_GEMM_CASE4(4, 1, 2);
        if (wn == 2) PS_GEMM_CASE(2, 1, 1);
        PS_GEMM_CASE4(1, 1, 4);
    }
    if (dc.xd) {
        if (!ps_gemm_digits_applies(w.N, w.K, M)) return hipErrorInvalidValue;
        if (M > 32) return launch<2, 4, 1, 8, true>(w, xq_tiled, xo_tiled, mask, X, sx, M, o, sess, dc, st);
        if (wn == 4) return launch<4, 2, 1, 8, true>(w, xq_tiled, xo_tiled, mask, X, sx, M, o, sess, dc, st);
        return launch<2, 2, 2, 8, true>(w, xq_tiled, xo_tiled, mask, X, sx, M, o, sess, dc, st);
    }
    if (M <= 32) {
        if (wn == 4) PS_GEMM_CASE4(4, 2, 1);
        if (wn == 2) PS_GEMM_CASE4(2, 2, 2);
        PS_GEMM_CASE4(1, 2, 2);
    }
    if (M <= PS_CHUNKED_ROWS_MAX) {   // 64 or 32 rows per workgroup, see the kernel
        int form;
        gemm_rows_us(w, M, form);
        if (form == ROWS32_4) return launch<2, 2, 1, 4>(w, xq_tiled, xo_tiled, mask, X, sx, M, o, sess, dc, st);
        if (form == ROWS32_16) return launch<1, 2, 1, 16>(w, xq_tiled, xo_tiled, mask, X, sx, M, o, sess, dc, st);
        if (wn >= 2 && form == ROWS64_4) return launch<2, 4, 1, 4>(w, xq_tiled, xo_tiled, mask, X, sx, M, o, sess, dc, st);
        if (wn >= 2) PS_GEMM_CASE(2, 4, 1);
        if (form == ROWS64_4) return launch<1, 4, 1, 4>(w, xq_tiled, xo_tiled, mask, X, sx, M, o, sess, dc, st);
        PS_GEMM_CASE(1, 4, 1);
    }
#undef PS_GEMM_CASE4
#undef PS_GEMM_CASE
    return hipErrorInvalidValue;   // larger calls belong to ps_gemm_lds
}

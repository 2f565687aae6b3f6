// Elementwise / per-row kernels of the span library: weight quantization into the
// streaming tile order, LayerNorm, outlier-column detection, row-wise int8
// quantization of activations, the blockwise 8-bit hidden-state codec, cache copies.
#include <atomic>

#include "common.h"
#include "digits.h"
#include "outlier_prep.h"
#include "rowops.h"

namespace {

// ---------------------------------------------------------------- weights

// One workgroup per 16 output rows.  Vector-wise int8 quantization of the fp32 rows
// (one scale per row = its absolute maximum) written straight into tile order.
__global__ void __launch_bounds__(256) k_quantize_weight(const float *__restrict__ W, int K,
                                                         int8_t *__restrict__ wt, float *__restrict__ sw) {
    __shared__ float s_abs[16];
    const int p = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int rr = 0; rr < 4; rr++) {
        const int row = wave * 4 + rr;
        const float *w = W + (size_t)(p * 16 + row) * K;
        float m = 0.0f;
        for (int k = lane * 4; k < K; k += 256) {
            float4 v = *(const float4 *)(w + k);
            m = fmaxf(m, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
        }
        m = wave_max(m);
        if (lane == 0) { s_abs[row] = m; sw[p * 16 + row] = m; }
    }
    __syncthreads();
    const int row = lane & 15, kg = lane >> 4, KT = K >> 6;
    const float s = s_abs[row];
    const float r = s > 0.0f ? 127.0f / s : 0.0f;
    for (int kt = wave; kt < KT; kt += 4) {
        const float4 *w = (const float4 *)(W + (size_t)(p * 16 + row) * K + kt * 64 + kg * 16);
        v4i out;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            float4 a = w[i];
            out[i] = pack4(q8(a.x, r), q8(a.y, r), q8(a.z, r), q8(a.w, r));
        }
        *(v4i *)(wt + ((size_t)(p * KT + kt) * 64 + lane) * 16) = out;
    }
}

__global__ void __launch_bounds__(256) k_untile_weight(const int8_t *__restrict__ wt, int K,
                                                       int8_t *__restrict__ wq) {
    const int p = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int row = lane & 15, kg = lane >> 4, KT = K >> 6;
    for (int kt = wave; kt < KT; kt += 4) {
        v4i v = *(const v4i *)(wt + ((size_t)(p * KT + kt) * 64 + lane) * 16);
        *(v4i *)(wq + (size_t)(p * 16 + row) * K + kt * 64 + kg * 16) = v;
    }
}

__global__ void k_fill_u32(uint32_t *p, size_t n, uint32_t v) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void k_copy_bytes(const uint8_t *__restrict__ s, uint8_t *__restrict__ d, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) d[i] = s[i];
}

// -------------------------------------------------------------- LayerNorm

// One workgroup per row that arrives as blockwise 8-bit codes: every thread decodes the elements it will normalise, stores
// them as the fp16 row the residual reads later, and normalises that row (1024 threads: the sums of k_layernorm_wide, in
// the same order).  These kernels flag outlier columns as bytes, for calls of more than 64 rows that k_layernorm_codes doesn't take.
static __device__ const CodeTable d_code_table = ps_make_code_table();

template <int NT>
__global__ void __launch_bounds__(NT) k_layernorm_q8(QuantIn qin, const __half *__restrict__ g,
                                                     const __half *__restrict__ b, float eps, int H,
                                                     __half *__restrict__ y, uint8_t *__restrict__ flags, float theta) {
    __shared__ double sm[NT / 64];
    __shared__ float table[256];
    for (int i = threadIdx.x; i < 256; i += NT) table[i] = d_code_table.code[i];
    __syncthreads();
    const size_t row0 = (size_t)blockIdx.x * H;
    __half *xr = qin.x_out + row0;
    __half *yr = y + row0;
    for (int k = threadIdx.x * 2; k < H; k += NT * 2) {
        const size_t i = row0 + k;                           // H and the codec block are even: both share a block
        const float am = qin.absmax[i / (size_t)qin.block];
        const uint32_t two = *(const uint16_t *)(qin.q + i);
        *(__half2 *)(xr + k) = __halves2half2(decode_q8(table, two & 255u, am), decode_q8(table, two >> 8, am));
    }
    double mean, inv;
    row_moments<NT>(xr, H, sm, mean, inv, (double)eps);     // every thread reads back what it wrote itself
    for (int k = threadIdx.x * 2; k < H; k += NT * 2) {
        const __half2 o = ln_affine(*(const __half2 *)(xr + k), *(const __half2 *)(g + k),
                                    *(const __half2 *)(b + k), mean, inv);
        *(__half2 *)(yr + k) = o;
        const uint32_t bits = (fabsf(__half2float(o.x)) >= theta ? 1u : 0u) | (fabsf(__half2float(o.y)) >= theta ? 2u : 0u);
        flag_outlier_bytes(flags, k, bits);
    }
}

// One workgroup per fp16 row, held in registers (H <= 16384: at most 8 pairs per thread of 1024) and so read from memory
// once instead of three times.
template <bool FLAGS>
__global__ void __launch_bounds__(1024) k_layernorm_wide(const __half *__restrict__ x, const __half *__restrict__ g,
                                                         const __half *__restrict__ b, float eps, int H,
                                                         __half *__restrict__ y, uint8_t *__restrict__ flags, float theta) {
    constexpr int NT = 1024, PER = 8;
    __shared__ double sm[NT / 64];
    const __half *xr = x + (size_t)blockIdx.x * H;
    __half *yr = y + (size_t)blockIdx.x * H;
    __half2 v[PER];
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < PER; i++) {
        const int k = (threadIdx.x + i * NT) * 2;
        if (k < H) {
            v[i] = *(const __half2 *)(xr + k);
            const float2 f = __half22float2(v[i]);
            s += (double)f.x + (double)f.y;
        }
    }
    const double mean = block_sum<NT / 64>(s, sm) / (double)H;
    double q = 0.0;
#pragma unroll
    for (int i = 0; i < PER; i++) {
        if ((int)(threadIdx.x + i * NT) * 2 < H) {
            const float2 f = __half22float2(v[i]);
            const double a = (double)f.x - mean, c = (double)f.y - mean;
            q += a * a + c * c;
        }
    }
    const double inv = 1.0 / sqrt(block_sum<NT / 64>(q, sm) / (double)H + (double)eps);
#pragma unroll
    for (int i = 0; i < PER; i++) {
        const int k = (threadIdx.x + i * NT) * 2;
        if (k < H) {
            const __half2 o = ln_affine(v[i], *(const __half2 *)(g + k), *(const __half2 *)(b + k), mean, inv);
            *(__half2 *)(yr + k) = o;
            if constexpr (FLAGS)
                flag_outlier_bytes(flags, k, (fabsf(__half2float(o.x)) >= theta ? 1u : 0u) | (fabsf(__half2float(o.y)) >= theta ? 2u : 0u));
        }
    }
}

// Many rows (a prefill-size call): 256 threads per row and 16-byte loads.  A workgroup takes every gridDim.x-th row;
// the next row is requested before the current one is reduced, so a compute unit's few workgroups keep memory busy,
// and the outlier columns of all its rows are flagged ONCE, at the end.  (One workgroup per row sent every row's
// flags to the same few words of the mask: an outlier feature is one in every row, another XCD's bits are not seen
// in this one's L2, and the memory takes 7 ns per access to one address - 4096 rows of 4096 with four outlier
// columns: 58 us, without any 28 us.)  The elements a thread sums differ from the kernel above, i.e. the fp64 sums
// are rounded in another order.  PER chunks of 8 columns per thread (H <= 2048 PER).  Q8: the rows arrive as 8-bit
// codes, see k_layernorm_q8.
template <int PER, bool Q8>
__global__ void __launch_bounds__(256, 3) k_layernorm_rows(const __half *__restrict__ x, QuantIn qin,
                                                        const __half *__restrict__ g, const __half *__restrict__ b,
                                                        float eps, int M, int H, __half *__restrict__ y,
                                                        uint8_t *__restrict__ cols, uint32_t theta_bits) {
    constexpr int NT = 256;
    // narrow rows: gain and bias stay in registers as fp64 over the rows of the workgroup, and so do a row's values over
    // its three passes (two conversions each, where a pass has one to three operations on a value)
    constexpr bool WIDE_REGS = PER <= 2;
    constexpr int NE = WIDE_REGS ? PER * 8 : 1;
    double gd[NE], bd[NE];
    if constexpr (WIDE_REGS) {
#pragma unroll
        for (int i = 0; i < PER; i++) {
            const int k = (threadIdx.x + i * NT) * 8;
            if (k < H) {
                const v8h gv = *(const v8h_any *)(g + k), bv = *(const v8h_any *)(b + k);
#pragma unroll
                for (int e = 0; e < 8; e++) { gd[i * 8 + e] = (double)(float)gv[e]; bd[i * 8 + e] = (double)(float)bv[e]; }
            }
        }
    }
    __shared__ double sm[NT / 64];
    __shared__ float table[Q8 ? 256 : 1];
    if constexpr (Q8) {
        table[threadIdx.x] = d_code_table.code[threadIdx.x];
        __syncthreads();
    }
    // raw bits of the row in flight: fp16 values, or 8 codes and their block's maximum
    struct Raw {
        v8h h;
        uint2 q;
        float am;
    };
    Raw nx[PER];
    auto request = [&](int row) {
        const size_t row0 = (size_t)row * H;
#pragma unroll
        for (int i = 0; i < PER; i++) {
            const int k = (threadIdx.x + i * NT) * 8;
            if (k < H) {
                if constexpr (Q8) {                          // H and the codec block are multiples of 8: one block per chunk
                    nx[i].q = *(const uint2 *)(qin.q + row0 + k);
                    nx[i].am = qin.absmax[(row0 + k) / (size_t)qin.block];
                } else {
                    nx[i].h = *(const v8h_any *)(x + row0 + k);
                }
            }
        }
    };
    uint32_t flags[PER] = {};
    if ((int)blockIdx.x < M) request(blockIdx.x);
    for (int row = blockIdx.x; row < M; row += gridDim.x) {
        const size_t row0 = (size_t)row * H;
        v8h v[PER];
#pragma unroll
        for (int i = 0; i < PER; i++) {
            const int k = (threadIdx.x + i * NT) * 8;
            if (k < H) {
                if constexpr (Q8) {
                    __half dec[8];
#pragma unroll
                    for (int e = 0; e < 8; e++)
                        dec[e] = decode_q8(table, ((e < 4 ? nx[i].q.x : nx[i].q.y) >> ((e & 3) * 8)) & 255u, nx[i].am);
                    v[i] = *(const v8h *)dec;
                    *(v8h *)(qin.x_out + row0 + k) = v[i];
                } else {
                    v[i] = nx[i].h;
                }
            }
        }
        if (row + (int)gridDim.x < M) request(row + gridDim.x);
        double s = 0.0, xd[NE];
#pragma unroll
        for (int i = 0; i < PER; i++) {
            if ((int)(threadIdx.x + i * NT) * 8 < H) {
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    const double x1 = (double)(float)v[i][e];
                    if constexpr (WIDE_REGS) xd[i * 8 + e] = x1;
                    s += x1;
                }
            }
        }
        const double mean = block_sum<NT / 64>(s, sm) / (double)H;
        // wide rows: converted again in every pass (kept as fp64 they would not fit the registers)
        auto forget = [&]() {
            if constexpr (!WIDE_REGS)
#pragma unroll
                for (int i = 0; i < PER; i++) {
                    v4i &w = *(v4i *)&v[i];
                    asm volatile("" : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]));
                }
        };
        forget();
        double q = 0.0;
#pragma unroll
        for (int i = 0; i < PER; i++) {
            if ((int)(threadIdx.x + i * NT) * 8 < H) {
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    double a;
                    if constexpr (WIDE_REGS) a = xd[i * 8 + e] -= mean;
                    else a = (double)(float)v[i][e] - mean;
                    q += a * a;
                }
            }
        }
        const double inv = 1.0 / sqrt(block_sum<NT / 64>(q, sm) / (double)H + (double)eps);
        forget();
#pragma unroll
        for (int i = 0; i < PER; i++) {
            const int k = (threadIdx.x + i * NT) * 8;
            if (k < H) {
                __half out[8];
                if constexpr (WIDE_REGS) {
#pragma unroll
                    for (int e = 0; e < 8; e++) out[e] = d2h_rn(xd[i * 8 + e] * inv * gd[i * 8 + e] + bd[i * 8 + e]);
                } else {
                    const v8h gv = *(const v8h_any *)(g + k), bv = *(const v8h_any *)(b + k);
#pragma unroll
                    for (int e = 0; e < 8; e++)
                        out[e] = d2h_rn(((double)(float)v[i][e] - mean) * inv * (double)(float)gv[e] + (double)(float)bv[e]);
                }
                const v4i ov = *(const v4i *)out;
                *(v4i *)(y + row0 + k) = ov;
                uint32_t m = 0;
#pragma unroll
                for (int e = 0; e < 4; e++) m = pk_max_u16(m, (uint32_t)ov[e] & 0x7fff7fffu);
                if (max(m & 0xffffu, m >> 16) >= theta_bits) {
#pragma unroll
                    for (int e = 0; e < 8; e++) {      // NaN (bits above infinity's) is no outlier: a row that overflowed
                        const uint32_t b = ((uint32_t)ov[e >> 1] >> ((e & 1) * 16)) & 0x7fffu;   // would flag every column
                        flags[i] |= (b >= theta_bits && b <= 0x7c00u ? 1u : 0u) << e;              // of the other rows
                    }
                }
            }
        }
    }
    if (!cols) return;
#pragma unroll
    for (int i = 0; i < PER; i++) {
        const int k = (threadIdx.x + i * NT) * 8;
        if (k < H) flag_outlier_bytes(cols, k, flags[i]);
    }
}

template <bool Q8>
hipError_t launch_layernorm_rows(const __half *x, const QuantIn &qin, const __half *g, const __half *b, float eps, int M, int H,
                                 __half *y, uint8_t *flags, float theta, hipStream_t st) {
    const int v = H <= 2048 ? 0 : H <= 4096 ? 1 : H <= 8192 ? 2 : 3;
    const uint32_t tb = ps_theta_to_bits(theta);
    auto kern = v == 0 ? k_layernorm_rows<1, Q8> : v == 1 ? k_layernorm_rows<2, Q8> : v == 2 ? k_layernorm_rows<4, Q8> : k_layernorm_rows<8, Q8>;
    // Workgroups that are resident at once on the 256 units, by the kernel's registers (5, 3, 4 and 3 to a unit as compiled now): a
    // grid of 1024 with room for 768 ran the last 256 alone (4096 rows of 4096 22.6 us, 21.5 this way).
    static std::atomic<int> resident[4];
    int per_unit = resident[v].load(std::memory_order_relaxed);
    if (!per_unit) {
        const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_unit, kern, 256, 0);
        if (e != hipSuccess) return e;
        if (per_unit < 1) return hipErrorInvalidConfiguration;
        resident[v].store(per_unit, std::memory_order_relaxed);
    }
    kern<<<M < 256 * per_unit ? M : 256 * per_unit, 256, 0, st>>>(x, qin, g, b, eps, M, H, y, flags, tb);
    return hipGetLastError();
}

// -------------------------------------------------- many rows: mask, then quantize

// Column c is an outlier if any row reaches theta.  grid.x covers columns (64 per
// wave), grid.y covers 64-row slabs; slabs combine with atomicOr (order-free).
__global__ void __launch_bounds__(256) k_colmask(const __half *__restrict__ X, int M, int K, float theta,
                                                 uint32_t *__restrict__ mask) {
    const int k0 = blockIdx.x * 256 + (threadIdx.x >> 6) * 64;
    if (k0 >= K) return;                                   // wave-uniform
    const int lane = threadIdx.x & 63;
    const int t0 = blockIdx.y * 64, t1 = min(M, t0 + 64);
    float m = 0.0f;
    for (int t = t0; t < t1; t++) m = fmaxf(m, fabsf(__half2float(X[(size_t)t * K + k0 + lane])));
    unsigned long long bal = __ballot(m >= theta);
    if (lane == 0) {
        if ((uint32_t)bal) atomicOr(&mask[k0 >> 5], (uint32_t)bal);
        if ((uint32_t)(bal >> 32)) atomicOr(&mask[(k0 >> 5) + 1], (uint32_t)(bal >> 32));
    }
}

// Row of a workgroup of the row quantizers.  Consecutive workgroup ids land on different XCDs (8, each with its
// own L2), and the 16 rows of a token tile interleave their 16-byte pieces in every 128-byte line of the tile: each
// XCD gets a contiguous run of whole tiles, so that a line is completed in ONE L2 instead of being written back
// in pieces by eight.  8 * per workgroups (`grid`), per a multiple of 16; ids beyond `rows` have nothing to do.  The
// workgroups behind them prepare the linear's outlier columns.
__device__ __forceinline__ int rowquant_row(int grid) {
    const int per = grid >> 3;
    return ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
}
template <int NT>
__device__ __forceinline__ void rowquant_prep(const OutlierPrep &pr, const uint32_t *mask, const uint8_t *flags, const __half *X,
                                              int M, int grid, int *list) {
    const int wave = threadIdx.x >> 6, item = ((int)blockIdx.x - grid) * (NT / 64) + wave;
    if (item < outlier_prep_items(pr, M)) outlier_prep_wave(pr, mask, flags, X, M, item, list + wave * PS_EXACT_OUTLIERS);
}
__host__ inline int rowquant_grid(int rows) { return 8 * (((rows / 16 + 7) / 8) * 16); }

// Arithmetic of the row quantizers on a chunk of 16 columns (8 words of two halves), written for few instructions: with
// a conversion, a clamp and a mask test per element the quantizer of 4096 rows of 16384 spent 28 of its 54 us in the
// vector ALU.  bits: the chunk's outlier columns (usually none).
typedef uint32_t chunk_t[8];
__device__ __forceinline__ uint32_t chunk_absmax(const chunk_t &w, uint32_t bits) {     // packed: one maximum per half
    uint32_t m = 0;
    if (bits == 0) {
#pragma unroll
        for (int i = 0; i < 8; i++) m = pk_max_u16(m, w[i] & 0x7fff7fffu);
    } else {
#pragma unroll
        for (int i = 0; i < 8; i++) {
            const uint32_t two = bits >> (2 * i);
            m = pk_max_u16(m, w[i] & (((two & 1u) ? 0u : 0x7fffu) | ((two & 2u) ? 0u : 0x7fff0000u)));
        }
    }
    return m;
}
// codes rint(fp32(x r)): the fp32 product straight from fp16 (a multiply-add with -0, which the compiler must not see
// through), the rounding by an addition that leaves the integer in the low byte.  No clamp: |x| <= the row's maximum
// s and r = fp32(127 / s) give |x r| <= 127.00002; codes of outlier columns are cleared.
__device__ __forceinline__ v4i chunk_codes(const chunk_t &w, uint32_t bits, float r) {
    float neg0 = -0.0f;
    asm("" : "+v"(neg0));
    v4i out;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        uint32_t t[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const unsigned short hb = (unsigned short)(w[2 * k + (e >> 1)] >> ((e & 1) * 16));
            t[e] = __float_as_uint(fmaf(__half2float(*(const __half *)&hb), r, neg0) + 12582912.0f);
        }
        out[k] = (int)__builtin_amdgcn_perm(__builtin_amdgcn_perm(t[3], t[2], 0x0c0c0400), __builtin_amdgcn_perm(t[1], t[0], 0x0c0c0400), 0x05040100);
    }
    if (bits) {
#pragma unroll
        for (int k = 0; k < 4; k++)
#pragma unroll
            for (int e = 0; e < 4; e++)
                if ((bits >> (4 * k + e)) & 1u) out[k] &= ~(0xff << (8 * e));
    }
    return out;
}
template <int NW>
__device__ __forceinline__ float row_scale(uint32_t m, uint32_t *sm) {
    m = wave_max(max(m & 0xffffu, m >> 16));
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = m;
    __syncthreads();
    m = sm[0];
#pragma unroll
    for (int i = 1; i < NW; i++) m = max(m, sm[i]);
    const unsigned short b = (unsigned short)m;
    return __half2float(*(const __half *)&b);
}

// Where the outlier columns come from: the mask, or (LayerNorm outputs of calls of more than 64 rows) FLAGS.  A template
// argument: a test per chunk puts a branch between its loads, and the compiler waits for all of them where its ends meet.
enum { ROWS_MASK = 0, ROWS_DIGITS = 1, ROWS_FLAGS = 2 };
template <int MODE>
__device__ __forceinline__ uint32_t row_chunk_outliers(uint32_t *mask, const uint8_t *flags, int c, int t) {
    if constexpr (MODE != ROWS_FLAGS) return ((const uint16_t *)mask)[c];
    const uint32_t bits = flag_bits16(*(const v4i *)(flags + (size_t)c * 16));
    if (t == 0) ((uint16_t *)mask)[c] = (uint16_t)bits;                  // for the kernels that read bits
    return bits;
}

// One workgroup per row of the 16-padded row range.  Row scale = absolute maximum over
// non-outlier columns; codes go to the MFMA operand tile order (same tiling as the
// weights, rows = tokens); padding rows are written as zeros.
template <int MODE>
__global__ void __launch_bounds__(256) k_rowquant_tiled(const __half *__restrict__ X, int M, int K,
                                                        uint32_t *__restrict__ mask, const uint8_t *__restrict__ flags,
                                                        int8_t *__restrict__ xq_tiled,
                                                        int8_t *__restrict__ xo_tiled, float *__restrict__ sx,
                                                        int8_t *__restrict__ xq_dbg, int rows, int grid, OutlierPrep pr) {
    __shared__ uint32_t sm[4];
    __shared__ int list[4 * PS_EXACT_OUTLIERS];
    if ((int)blockIdx.x >= grid) {
        rowquant_prep<256>(pr, mask, flags, X, M, grid, list);
        return;
    }
    const int t = rowquant_row(grid), KT = K >> 6, nchunk = K >> 4;
    if (t >= rows) return;
    const size_t tile_row = (size_t)(t >> 4) * KT;
    if (t >= M) {
        for (int c = threadIdx.x; c < nchunk; c += 256) {
            v4i z = {0, 0, 0, 0};
            *(v4i *)(xq_tiled + ((tile_row + (c >> 2)) * 64 + (c & 3) * 16 + (t & 15)) * 16) = z;
        }
        return;
    }
    const __half *xr = X + (size_t)t * K;
    uint32_t m = 0;
    for (int c = threadIdx.x; c < nchunk; c += 256) {
        chunk_t w;
        *(v4i *)w = *(const v4i *)(xr + c * 16);
        *(v4i *)(w + 4) = *(const v4i *)(xr + c * 16 + 8);
        const uint32_t bits = row_chunk_outliers<MODE>(mask, flags, c, t);
        m = pk_max_u16(m, chunk_absmax(w, bits));
    }
    const float s = row_scale<4>(m, sm);
    if (threadIdx.x == 0) sx[t] = s;
    const float r = s > 0.0f ? 127.0f / s : 0.0f;
    for (int c = threadIdx.x; c < nchunk; c += 256) {
        const uint32_t bits = row_chunk_outliers<MODE>(mask, flags, c, t);
        const v8h a = *(const v8h *)(xr + c * 16), b = *(const v8h *)(xr + c * 16 + 8);
        chunk_t w;
        *(v8h *)w = a;
        *(v8h *)(w + 4) = b;
        const v4i o = chunk_codes(w, bits, r);
        const size_t slot = ((tile_row + (c >> 2)) * 64 + (c & 3) * 16 + (t & 15)) * 16;
        *(v4i *)(xq_tiled + slot) = o;
        if (xq_dbg) *(v4i *)(xq_dbg + (size_t)t * K + c * 16) = o;
        if (xo_tiled && bits) {   // the group's first 8 outlier values, ascending column order
            v8h ov;
            uint32_t rest = bits;
#pragma unroll
            for (int r = 0; r < 8; r++) {
                const int j = rest ? __ffs(rest) - 1 : 0;
                _Float16 v = (_Float16)0.0f;
#pragma unroll
                for (int i = 0; i < 8; i++) {
                    if (j == i) v = a[i];
                    if (j == i + 8) v = b[i];
                }
                ov[r] = rest ? v : (_Float16)0.0f;
                rest &= rest - 1;
            }
            *(v8h *)(xo_tiled + slot) = ov;
        }
    }
}

// The same for wide rows (4096 <= K <= NT * CPT * 16): NT threads, each keeps its (at most CPT) chunks of 16
// columns in registers between the absolute-maximum pass and the quantization, so X is read once;
// for calls of few rows, where the latency of the loads is the whole cost, this halves it (1024 threads);
// for calls of many rows, 256 threads per row put four times as many rows on a compute unit.
// ROWS_DIGITS: also counts the outlier columns, and if they are more than one in 16 writes the row's outlier values as
// digits, zero in regular columns.  (14336 x 57344, 32 rows, digits against fp64 form: one column in 12 304 and 357 us, one
// in 4 300 and 623; the fp64 form at one in 16 305, one in 32 250; at 64 rows 539 and 605, 550 and 1105, 528, 430.)
template <int NT, int CPT, int MODE>
__global__ void __launch_bounds__(NT) k_rowquant_tiled_wide(const __half *__restrict__ X, int M, int K,
                                                             uint32_t *__restrict__ mask, const uint8_t *__restrict__ flags,
                                                             int8_t *__restrict__ xq_tiled,
                                                             int8_t *__restrict__ xo_tiled, float *__restrict__ sx,
                                                             int8_t *__restrict__ xq_dbg, int rows, int grid, OutlierPrep pr,
                                                             RowDigits rd) {
    constexpr bool DIGITS = MODE == ROWS_DIGITS;
    __shared__ uint32_t sm[NT / 64], smc[DIGITS ? NT / 64 : 1];
    __shared__ int big;
    __shared__ int list[NT / 64 * PS_EXACT_OUTLIERS];
    if ((int)blockIdx.x >= grid) {
        rowquant_prep<NT>(pr, mask, flags, X, M, grid, list);
        return;
    }
    const int t = rowquant_row(grid), KT = K >> 6, nchunk = K >> 4;
    if (t >= rows) return;
    const size_t tile_row = (size_t)(t >> 4) * KT;
    if (t >= M) {
        for (int c = threadIdx.x; c < nchunk; c += NT) {
            v4i z = {0, 0, 0, 0};
            *(v4i *)(xq_tiled + ((tile_row + (c >> 2)) * 64 + (c & 3) * 16 + (t & 15)) * 16) = z;
        }
        return;
    }
    const __half *xr = X + (size_t)t * K;
    v8h a[CPT], b[CPT];
    uint32_t bits[CPT];
#pragma unroll
    for (int i = 0; i < CPT; i++) {
        const int c = threadIdx.x + i * NT;
        if (c < nchunk) {
            a[i] = *(const v8h *)(xr + c * 16);
            b[i] = *(const v8h *)(xr + c * 16 + 8);
            bits[i] = row_chunk_outliers<MODE>(mask, flags, c, t);
        }
    }
    uint32_t m = 0, n_out = 0;
#pragma unroll
    for (int i = 0; i < CPT; i++) {
        if ((int)(threadIdx.x + i * NT) < nchunk) {
            chunk_t w;
            *(v8h *)w = a[i];
            *(v8h *)(w + 4) = b[i];
            m = pk_max_u16(m, chunk_absmax(w, bits[i]));
            if constexpr (DIGITS) n_out += __popc(bits[i]);
        }
    }
    if constexpr (DIGITS) {
        n_out = wave_reduce(n_out, 0u, [](uint32_t a, uint32_t b) { return a + b; });
        if ((threadIdx.x & 63) == 0) smc[threadIdx.x >> 6] = n_out;
        if (threadIdx.x == 0) big = 0;
        static_assert(NT >= PS_DIGIT_DONE, "one thread clears each counter");
        if (t == 0 && threadIdx.x < PS_DIGIT_DONE) rd.done[threadIdx.x] = 0;
    }
    const float s = row_scale<NT / 64>(m, sm);
    bool digits = false;
    if constexpr (DIGITS) {
        n_out = 0;
#pragma unroll
        for (int i = 0; i < NT / 64; i++) n_out += smc[i];
        digits = n_out * 16 > (uint32_t)K;
    }
    if (threadIdx.x == 0) sx[t] = s;
    const float r = s > 0.0f ? 127.0f / s : 0.0f;
#pragma unroll
    for (int i = 0; i < CPT; i++) {
        const int c = threadIdx.x + i * NT;
        if (c < nchunk) {
            chunk_t w;
            *(v8h *)w = a[i];
            *(v8h *)(w + 4) = b[i];
            const v4i o = chunk_codes(w, bits[i], r);
            const size_t slot = ((tile_row + (c >> 2)) * 64 + (c & 3) * 16 + (t & 15)) * 16;
            *(v4i *)(xq_tiled + slot) = o;
            if (xq_dbg) *(v4i *)(xq_dbg + (size_t)t * K + c * 16) = o;
            if (DIGITS && digits) {
                __half v[16];
                uint32_t am = 0;
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    const uint32_t two = bits[i] >> (2 * e), h = w[e] & (((two & 1u) ? 0xffffu : 0u) | ((two & 2u) ? 0xffff0000u : 0u));
                    am = pk_max_u16(am, h & 0x7fff7fffu);
                    *(uint32_t *)(v + 2 * e) = h;
                }
                if (max(am & 0xffffu, am >> 16) >= DIGITS_BIG) big = 1;
                v4i pl[4];
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    int p4[4];
                    digit_planes4(*(const __half(*)[4])(v + 4 * q), p4);
#pragma unroll
                    for (int d = 0; d < 4; d++) pl[d][q] = p4[d];
                }
                int8_t *to = rd.xd + (tile_row + (c >> 2)) * 4096 + ((c & 3) * 16 + (t & 15)) * 16;
#pragma unroll
                for (int d = 0; d < 4; d++) *(v4i *)(to + d * 1024) = pl[d];
            }
            if (xo_tiled && bits[i]) {   // the group's first 8 outlier values, ascending column order
                v8h ov;
                uint32_t rest = bits[i];
#pragma unroll
                for (int rr = 0; rr < 8; rr++) {
                    const int j = rest ? __ffs(rest) - 1 : 0;
                    _Float16 v = (_Float16)0.0f;
#pragma unroll
                    for (int k = 0; k < 8; k++) {
                        if (j == k) v = a[i][k];
                        if (j == k + 8) v = b[i][k];
                    }
                    ov[rr] = rest ? v : (_Float16)0.0f;
                    rest &= rest - 1;
                }
                *(v8h *)(xo_tiled + slot) = ov;
            }
        }
    }
    if constexpr (DIGITS) {              // a value that takes more than four digits (or is none): the fp64 form for the call
        __syncthreads();
        if (threadIdx.x == 0) rd.rowstate[t] = digits && !big ? PS_ROWS_IN_DIGITS : 0;
    }
}

// LayerNorm and row quantizer in one launch, for calls of up to PS_NORM_ROWS_MAX rows: the codes of a row need the outlier
// columns of ALL rows, which the workgroups - one per row - tell each other while they run.  A row's columns go into a record
// of eight 64-bit words in device memory: three columns and the tag of this LayerNorm in each, written and read by relaxed
// atomics of agent scope, so that a word that carries the tag is complete; more than 24 columns go as a bit mask that is in
// memory before the record says so.  What this saves is a launch (2.5 us) and the rows' way through memory; the exchange takes
// about 1 us.  8 rows of 4096: LayerNorm 5.7 and quantizer 4.7 us, together 6.5 (decode step of 8 sessions through four such
// blocks 400 -> 370); 128 rows of 1024 3.8 and 4.5, together 6.4, where a workgroup reads 8 KB of records: the line of
// PS_NORM_ROWS_MAX.
// A workgroup that has waited for `patience` ticks of the 100 MHz clock (not all of them may be resident at once when other
// work shares the device) finds the outlier columns by itself, from all rows; with a patience of 0 every one does.
constexpr int NORM_WORDS = 8, NORM_COLS = 3 * NORM_WORDS, NORM_NONE = 0xffff, NORM_MASK = 0xfffe;

template <int NT, int PER, bool Q8>
__global__ void __launch_bounds__(NT) k_layernorm_codes(const __half *__restrict__ x, QuantIn qin, const __half *__restrict__ g,
                                                        const __half *__restrict__ b, float eps, int M, int H, __half *__restrict__ y,
                                                        uint32_t *__restrict__ mask, int8_t *__restrict__ xq_tiled,
                                                        int8_t *__restrict__ xo_tiled, float *__restrict__ sx, int8_t *__restrict__ xq_dbg,
                                                        uint32_t theta_bits, double inv_h, NormExchange ex, int rows, int grid) {
    extern __shared__ __align__(16) unsigned char dyn[];             // the normalised row, [H] halves
    __half *row = (__half *)dyn;
    __shared__ double sm[2][NT / 64];
    __shared__ uint32_t smm[NT / 64], cols[512];                     // cols: outlier columns, a bit each
    __shared__ uint16_t mine[NORM_COLS];
    __shared__ int n_mine, late;
    __shared__ uint32_t masked[PS_NORM_ROWS_MAX / 32];               // other rows whose columns are a mask, a bit each
    __shared__ float table[Q8 ? 256 : 1];
    const int t = rowquant_row(grid), KT = H >> 6, nchunk = H >> 4, words = H >> 5;
    if (t >= M) {                                                    // rows that pad the last tile
        if (t < rows)
            for (int c = threadIdx.x; c < nchunk; c += NT)
                *(v4i *)(xq_tiled + (((size_t)(t >> 4) * KT + (c >> 2)) * 64 + (c & 3) * 16 + (t & 15)) * 16) = (v4i){0, 0, 0, 0};
        return;
    }
    for (int i = threadIdx.x; i < words; i += NT) cols[i] = 0u;
    if (threadIdx.x == 0) n_mine = late = 0;
    if (threadIdx.x < PS_NORM_ROWS_MAX / 32) masked[threadIdx.x] = 0u;
    if constexpr (Q8)
        for (int i = threadIdx.x; i < 256; i += NT) table[i] = d_code_table.code[i];
    __syncthreads();

    uint32_t v[PER][2], own[PER];                                    // this thread's four columns, PER times; outliers among them
    auto normalise = [&](int r, bool store) {
        const size_t row0 = (size_t)r * H;
        double s = 0.0, q = 0.0;
#pragma unroll
        for (int i = 0; i < PER; i++) {
            const int k = (threadIdx.x + i * NT) * 4;
            v[i][0] = v[i][1] = 0u;
            if (k >= H) continue;
            if constexpr (Q8) {                                      // H and the codec block are multiples of 4: one block
                const float am = qin.absmax[(row0 + k) / (size_t)qin.block];
                const uint32_t a = *(const uint16_t *)(qin.q + row0 + k), c = *(const uint16_t *)(qin.q + row0 + k + 2);
                v[i][0] = (uint32_t)__half_as_ushort(decode_q8(table, a & 255u, am)) | (uint32_t)__half_as_ushort(decode_q8(table, a >> 8, am)) << 16;
                v[i][1] = (uint32_t)__half_as_ushort(decode_q8(table, c & 255u, am)) | (uint32_t)__half_as_ushort(decode_q8(table, c >> 8, am)) << 16;
                if (store) *(uint2 *)(qin.x_out + row0 + k) = make_uint2(v[i][0], v[i][1]);
            } else {
                const uint32_t *from = (const uint32_t *)(x + row0 + k);
                v[i][0] = from[0];
                v[i][1] = from[1];
            }
        }
        auto value = [&](int i, int e) { return (double)__half2float(__ushort_as_half((unsigned short)(v[i][e >> 1] >> ((e & 1) * 16)))); };
#pragma unroll
        for (int i = 0; i < PER; i++)
#pragma unroll
            for (int e = 0; e < 4; e++) s += value(i, e);            // (zeros beyond the row)
        // (a workgroup's sum with one barrier: the next one goes to another array; quotients by the row's length from its
        // reciprocal and the exact remainder)
        auto row_mean = [&](double p, int which) {
            p = wave_sum(p);
            if ((threadIdx.x & 63) == 0) sm[which][threadIdx.x >> 6] = p;
            lds_barrier();
            p = sm[which][0];
#pragma unroll
            for (int i = 1; i < NT / 64; i++) p += sm[which][i];
            const double m = p * inv_h;
            return fma(fma(-m, (double)H, p), inv_h, m);
        };
        const double mean = row_mean(s, 0);
#pragma unroll
        for (int i = 0; i < PER; i++)
            if ((int)(threadIdx.x + i * NT) * 4 < H)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const double d = value(i, e) - mean;
                    q += d * d;
                }
        const double inv = rsqrt_f64(row_mean(q, 1) + (double)eps);
#pragma unroll
        for (int i = 0; i < PER; i++) {
            const int k = (threadIdx.x + i * NT) * 4;
            own[i] = 0;
            if (k >= H) continue;
            const uint2 gw = *(const uint2 *)(g + k), bw = *(const uint2 *)(b + k);
            uint32_t out[2];
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const uint32_t gs = e < 2 ? gw.x : gw.y, bs = e < 2 ? bw.x : bw.y;
                const __half gh = __ushort_as_half((unsigned short)(gs >> ((e & 1) * 16))), bh = __ushort_as_half((unsigned short)(bs >> ((e & 1) * 16)));
                const uint32_t o = __half_as_ushort(d2h_rn((value(i, e) - mean) * inv * (double)__half2float(gh) + (double)__half2float(bh)));
                const uint32_t a = o & 0x7fffu;                      // NaN is no outlier, see k_layernorm_rows
                own[i] |= (a >= theta_bits && a <= 0x7c00u ? 1u : 0u) << e;
                out[e >> 1] = e & 1 ? out[e >> 1] | o << 16 : o;
            }
            v[i][0] = out[0];
            v[i][1] = out[1];
            if (store) {
                *(uint2 *)(y + row0 + k) = make_uint2(out[0], out[1]);
                *(uint2 *)(row + k) = make_uint2(out[0], out[1]);
            }
            if (own[i]) atomicOr(&cols[k >> 5], own[i] << (k & 31));
        }
    };
    normalise(t, true);
#pragma unroll
    for (int i = 0; i < PER; i++)
        for (uint32_t left = own[i]; left; left &= left - 1) {
            const int at = atomicAdd(&n_mine, 1);
            if (at < NORM_COLS) mine[at] = (uint16_t)((threadIdx.x + i * NT) * 4 + __ffs(left) - 1);
        }
    __syncthreads();
    const uint64_t tagged = (uint64_t)ex.tag << 48;
    const bool as_mask = n_mine > NORM_COLS;
    if (as_mask) {
        for (int i = threadIdx.x; i < words; i += NT)
            __hip_atomic_store(ex.masks + (size_t)t * words + i, cols[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // this wave's words are where every XCD sees them
        __syncthreads();
    }
    if (threadIdx.x < NORM_WORDS) {
        uint64_t w = tagged;
#pragma unroll
        for (int e = 0; e < 3; e++) {
            const int i = 3 * threadIdx.x + e;
            w |= (uint64_t)(as_mask ? NORM_MASK : i < n_mine ? mine[i] : NORM_NONE) << (16 * e);
        }
        __hip_atomic_store(ex.records + (size_t)t * NORM_WORDS + threadIdx.x, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // the other rows' records, AT words per thread at once (one, but for short rows and many of them)
    constexpr int AT = NT == 256 ? 4 : 2;
    static_assert(AT * NT >= PS_NORM_ROWS_MAX * NORM_WORDS, "every word has a thread");
    if (ex.patience == 0) {                                          // not even looked at
        late = 1;
    } else {
        uint64_t w[AT], start = 0;
        for (int spins = 0;; spins++) {
            bool there = true;
#pragma unroll
            for (int a = 0; a < AT; a++) {
                const int i = threadIdx.x + a * NT;
                w[a] = i < M * NORM_WORDS && i / NORM_WORDS != t ? __hip_atomic_load(ex.records + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                                                 : tagged | 0xffffffffffffull;
            }
#pragma unroll
            for (int a = 0; a < AT; a++) there = there && w[a] >> 48 == ex.tag;
            if (there) break;
            if ((spins & 7) == 7) {
                const uint64_t now = __builtin_amdgcn_s_memrealtime();
                if (!start) start = now;
                if (now - start >= ex.patience) { late = 1; break; }
            }
        }
#pragma unroll
        for (int a = 0; a < AT; a++) {
            if (w[a] >> 48 != ex.tag) continue;
            const int i = threadIdx.x + a * NT, r = i / NORM_WORDS;
            if ((int)(w[a] & 0xffff) == NORM_MASK) {
                if (i % NORM_WORDS == 0) atomicOr(&masked[r >> 5], 1u << (r & 31));
                continue;
            }
#pragma unroll
            for (int e = 0; e < 3; e++) {
                const int c = (int)(w[a] >> (16 * e)) & 0xffff;
                if (c < H) atomicOr(&cols[c >> 5], 1u << (c & 31));
            }
        }
    }
    __syncthreads();
    if (late) {                                                      // rare; the same in all threads
        uint32_t keep[PER][2];
#pragma unroll
        for (int i = 0; i < PER; i++) { keep[i][0] = v[i][0]; keep[i][1] = v[i][1]; }
        for (int r = 0; r < M; r++)
            if (r != t) normalise(r, false);
#pragma unroll
        for (int i = 0; i < PER; i++) { v[i][0] = keep[i][0]; v[i][1] = keep[i][1]; }
        __syncthreads();
    } else {
        uint32_t any = 0;
#pragma unroll
        for (int i = 0; i < PS_NORM_ROWS_MAX / 32; i++) any |= masked[i];
        if (any) {
            // rare: rows with many outlier columns.  A thread takes one word of every G-th row, eight of them requested at once (the
            // rows one after the other, two round trips to memory each, cost 128 rows of 1024 some 40 us).
            const int G = NT / words, g = (int)threadIdx.x / words, i = (int)threadIdx.x - g * words;    // H <= 32 NT: at least one row
            if (g < G) {
                uint32_t sum = 0;
                for (int r0 = g; r0 < M; r0 += 8 * G) {
                    uint32_t a[8];
#pragma unroll
                    for (int u = 0; u < 8; u++) {
                        const int r = r0 + u * G;
                        a[u] = r < M && (masked[r >> 5] >> (r & 31) & 1u) ? __hip_atomic_load(ex.masks + (size_t)r * words + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
                    }
#pragma unroll
                    for (int u = 0; u < 8; u++) sum |= a[u];
                }
                if (sum) atomicOr(&cols[i], sum);
            }
            __syncthreads();
        }
    }
    if (t == 0)
        for (int i = threadIdx.x; i < words; i += NT) mask[i] = cols[i];

    uint32_t m = 0, bits[PER];
#pragma unroll
    for (int i = 0; i < PER; i++) {
        const int k = (threadIdx.x + i * NT) * 4;
        bits[i] = k < H ? cols[k >> 5] >> (k & 31) & 15u : 0u;
#pragma unroll
        for (int e = 0; e < 2; e++) {
            const uint32_t two = bits[i] >> (2 * e);
            m = pk_max_u16(m, v[i][e] & (((two & 1u) ? 0u : 0x7fffu) | ((two & 2u) ? 0u : 0x7fff0000u)));
        }
    }
    const float s = row_scale<NT / 64>(m, smm);
    if (threadIdx.x == 0) sx[t] = s;
    const float r = s > 0.0f ? 127.0f / s : 0.0f;
    const size_t tile_row = (size_t)(t >> 4) * KT;
    float neg0 = -0.0f;
    asm("" : "+v"(neg0));
#pragma unroll
    for (int i = 0; i < PER; i++) {
        const int k = (threadIdx.x + i * NT) * 4, c = k >> 4;
        if (k >= H) continue;
        uint32_t u[4];                                               // see chunk_codes
#pragma unroll
        for (int e = 0; e < 4; e++)
            u[e] = __float_as_uint(fmaf(__half2float(__ushort_as_half((unsigned short)(v[i][e >> 1] >> ((e & 1) * 16)))), r, neg0) + 12582912.0f);
        uint32_t o = __builtin_amdgcn_perm(__builtin_amdgcn_perm(u[3], u[2], 0x0c0c0400), __builtin_amdgcn_perm(u[1], u[0], 0x0c0c0400), 0x05040100);
        if (bits[i]) {
#pragma unroll
            for (int e = 0; e < 4; e++)
                if (bits[i] >> e & 1u) o &= ~(0xffu << (8 * e));
        }
        const size_t slot = ((tile_row + (c >> 2)) * 64 + (c & 3) * 16 + (t & 15)) * 16;
        *(uint32_t *)(xq_tiled + slot + (k & 15)) = o;
        if (xq_dbg) *(uint32_t *)(xq_dbg + (size_t)t * H + k) = o;
        const uint32_t all = cols[c >> 1] >> ((c & 1) * 16) & 0xffffu;
        if ((k & 15) == 0 && all) {                                  // the group's first 8 outlier values, ascending column order
            __half first[8];
            uint32_t rest = all;
#pragma unroll
            for (int e = 0; e < 8; e++) {
                first[e] = rest ? row[k + __ffs(rest) - 1] : __ushort_as_half(0);
                rest &= rest - 1;
            }
            *(v4i *)(xo_tiled + slot) = *(const v4i *)first;
        }
    }
}

// out[i] = number of set bits of the i-th mask of `words` words (one workgroup per mask)
__global__ void __launch_bounds__(256) k_mask_count(const uint32_t *__restrict__ masks, int words, int32_t *__restrict__ out) {
    __shared__ float sm[4];
    int c = 0;
    for (int i = threadIdx.x; i < words; i += 256) c += __popc(masks[(size_t)blockIdx.x * words + i]);
    const float total = block_sum<4>((float)c, sm);          // at most 65536 bits: exact in fp32
    if (threadIdx.x == 0) out[blockIdx.x] = (int32_t)total;
}

__global__ void k_mask_to_bytes(const uint32_t *__restrict__ mask, int K, uint8_t *__restrict__ out) {
    int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < K) out[k] = (mask[k >> 5] >> (k & 31)) & 1u;
}

// ------------------------------------------------------------------- codec

// One workgroup per block of `block` elements (last block may be short).  A decode step has few blocks, so the
// kernel is latency bound: 1024 threads keep the chain of dependent table look-ups per thread short.
__global__ void __launch_bounds__(1024) k_hidden_quantize(const __half *__restrict__ x, size_t n, int block,
                                                         CodeTable tab, uint8_t *__restrict__ q,
                                                         float *__restrict__ absmax) {
    __shared__ float mids[256];
    __shared__ float sm[16];
    if (threadIdx.x < 255) mids[threadIdx.x] = (tab.code[threadIdx.x] + tab.code[threadIdx.x + 1]) * 0.5f;
    const size_t b0 = (size_t)blockIdx.x * block;
    const int len = (int)min((size_t)block, n - b0);
    float m = 0.0f;
    for (int i = threadIdx.x; i < len; i += 1024) m = fmaxf(m, fabsf(__half2float(x[b0 + i])));
    const float a = block_max<16>(m, sm);   // its barrier also publishes mids
    if (threadIdx.x == 0) absmax[blockIdx.x] = a;
    for (int i = threadIdx.x; i < len; i += 1024) {
        const float v = a > 0.0f ? __half2float(x[b0 + i]) / a : 0.0f;
        int lo = 0, hi = 255;               // count of midpoints strictly below v
        while (lo < hi) {
            int mid = (lo + hi) >> 1;
            if (mids[mid] < v) lo = mid + 1; else hi = mid;
        }
        q[b0 + i] = (uint8_t)lo;
    }
}

// The same for buffers aligned to 16 (values) and 8 (codes) bytes.  Memory bound in the large, latency bound at
// decode sizes: a thread holds 8 consecutive values per chunk in registers, so x is read once, with 16-byte loads;
// the quotients by the block's maximum are the IEEE ones from one reciprocal (q = x r corrected by the exact
// remainder: three instructions); and the midpoints below a quotient are counted with ONE comparison: quotients
// are binned by sign, exponent and 6 mantissa bits, no bin holds more than one midpoint, and a table says how many
// lie below each bin.  29.4 M values (2048 rows of 14336) into codes and back: 163 -> 42 us with the wide
// dequantizer below (92 us of it were the binary search over the 255 midpoints with two 2-byte reads of every value,
// 66 us one 2-byte store and one 64-bit division per value).  128 threads cover blocks
// of up to 1024 values, 512 with 1, 2 or 4 chunks blocks of up to 4096, 8192 and 16384.
constexpr int CODE_SHIFT = 17, CODE_KEY0 = 105 << (23 - CODE_SHIFT);         // bin 0: everything below 2^-22, no midpoint there
constexpr int CODE_BINS = (127 << (23 - CODE_SHIFT)) - CODE_KEY0 + 1;        // the last bin starts at 1.0
struct CodeBins {
    float mids[256];                 // mids[255] = +infinity
    uint8_t below[2 * CODE_BINS];    // midpoints below the values of a bin: positive values, then negative ones
};
constexpr CodeBins make_code_bins() {
    CodeBins t{};
    const CodeTable tab = ps_make_code_table();
    for (int i = 0; i < 255; i++) t.mids[i] = (tab.code[i] + tab.code[i + 1]) * 0.5f;
    t.mids[255] = __builtin_huge_valf();
    int c = 0;                                                               // positive bins, ascending
    for (int b = 0; b < CODE_BINS; b++) {
        const float lo = b == 0 ? 0.0f : __builtin_bit_cast(float, (uint32_t)(CODE_KEY0 + b) << CODE_SHIFT);
        while (t.mids[c] < lo) c++;
        t.below[b] = (uint8_t)c;
    }
    c = 0;                                                                   // negative bins, ascending from -1.0
    for (int b = CODE_BINS - 1; b >= 0; b--) {
        const float lo = -__builtin_bit_cast(float, ((uint32_t)(CODE_KEY0 + b + 1) << CODE_SHIFT) - 1u);
        while (t.mids[c] < lo) c++;
        t.below[CODE_BINS + b] = (uint8_t)c;
    }
    return t;
}
constexpr bool one_midpoint_per_bin(const CodeBins &t) {
    for (int b = 0; b < CODE_BINS; b++) {
        const float hi = __builtin_bit_cast(float, ((uint32_t)(CODE_KEY0 + b + 1) << CODE_SHIFT) - 1u);
        if (t.below[b] < 254 && t.mids[t.below[b] + 1] < hi) return false;
        const float nhi = b == 0 ? 0.0f : -__builtin_bit_cast(float, (uint32_t)(CODE_KEY0 + b) << CODE_SHIFT);
        if (t.mids[t.below[CODE_BINS + b] + 1] < nhi) return false;
    }
    return true;
}
static_assert(one_midpoint_per_bin(make_code_bins()), "one comparison per value needs at most one midpoint per bin");
static_assert(sizeof(CodeBins) % 4 == 0, "copied to LDS word by word");
static __device__ const CodeBins d_code_bins = make_code_bins();

template <int NT, int PER>
__global__ void __launch_bounds__(NT) k_hidden_quantize_wide(const __half *__restrict__ x, size_t n, int block,
                                                              uint8_t *__restrict__ q, float *__restrict__ absmax) {
    __shared__ CodeBins cb;
    __shared__ uint32_t s_max[NT / 64];
    const size_t b0 = (size_t)blockIdx.x * block;
    const int len = (int)min((size_t)block, n - b0);
    const __half *xb = x + b0;
    v4i xv[PER];
    uint32_t mb = 0;
#pragma unroll
    for (int i = 0; i < PER; i++) {
        const int k = (threadIdx.x + i * NT) * 8;
        xv[i] = (v4i){0, 0, 0, 0};
        if (k + 8 <= len) {
            xv[i] = *(const v4i *)(xb + k);
        } else {
#pragma unroll
            for (int e = 0; e < 8; e++)                        // the ragged end of the last block
                if (k + e < len) xv[i][e >> 1] |= (int)((uint32_t)__half_as_ushort(xb[k + e]) << ((e & 1) * 16));
        }
    }
    for (int i = threadIdx.x; i < (int)(sizeof(CodeBins) / 4); i += NT) ((uint32_t *)&cb)[i] = ((const uint32_t *)&d_code_bins)[i];
#pragma unroll
    for (int i = 0; i < PER; i++)
#pragma unroll
        for (int e = 0; e < 8; e++) mb = max(mb, ((uint32_t)xv[i][e >> 1] >> ((e & 1) * 16)) & 0x7fffu);   // fp16 magnitudes order like their bits
    mb = wave_max(mb);
    if ((threadIdx.x & 63) == 0) s_max[threadIdx.x >> 6] = mb;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NT / 64; w++) mb = max(mb, s_max[w]);
    const unsigned short ab = (unsigned short)mb;
    float a = __half2float(*(const __half *)&ab);
    const bool finite = mb < 0x7c00u;
    if (!finite) {                                             // (the whole workgroup) NaN does not count, as in fmaxf
        mb = 0;
#pragma unroll
        for (int i = 0; i < PER; i++)
#pragma unroll
            for (int e = 0; e < 8; e++) {
                const uint32_t b = ((uint32_t)xv[i][e >> 1] >> ((e & 1) * 16)) & 0x7fffu;
                mb = max(mb, b <= 0x7c00u ? b : 0u);
            }
        mb = wave_max(mb);
        __syncthreads();                                       // the first maxima have been read
        if ((threadIdx.x & 63) == 0) s_max[threadIdx.x >> 6] = mb;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < NT / 64; w++) mb = max(mb, s_max[w]);
        const unsigned short nb = (unsigned short)mb;
        a = __half2float(*(const __half *)&nb);
    }
    if (threadIdx.x == 0) absmax[blockIdx.x] = a;
    const float r = a > 0.0f ? 1.0f / a : 0.0f;
#pragma unroll
    for (int i = 0; i < PER; i++) {
        const int k = (threadIdx.x + i * NT) * 8;
        uint32_t w[2] = {0u, 0u};
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const unsigned short hb = (unsigned short)((uint32_t)xv[i][e >> 1] >> ((e & 1) * 16));
            const float f = __half2float(*(const __half *)&hb), q0 = f * r;
            float v = fmaf(fmaf(-q0, a, f), r, q0);            // == f / a in fp32: r is the rounded 1 / a, the remainder exact
            if (!finite) v = a > 0.0f ? f / a : 0.0f;
            const int key = min(max((int)(__float_as_uint(fabsf(v)) >> CODE_SHIFT) - CODE_KEY0, 0), CODE_BINS - 1);
            uint32_t c = cb.below[key + (v < 0.0f ? CODE_BINS : 0)];
            c += cb.mids[c] < v ? 1u : 0u;
            if (!finite && !(v == v)) c = 0;
            w[e >> 2] |= c << (8 * (e & 3));
        }
        if (k + 8 <= len) {
            *(uint2 *)(q + b0 + k) = make_uint2(w[0], w[1]);
        } else {
#pragma unroll
            for (int e = 0; e < 8; e++)
                if (k + e < len) q[b0 + k + e] = (uint8_t)(w[e >> 2] >> (8 * (e & 3)));
        }
    }
}

__global__ void __launch_bounds__(256) k_hidden_dequantize(const uint8_t *__restrict__ q,
                                                           const float *__restrict__ absmax, size_t n, int block,
                                                           CodeTable tab, __half *__restrict__ y) {
    __shared__ float code[256];
    code[threadIdx.x] = tab.code[threadIdx.x];
    __syncthreads();
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) y[i] = __float2half_rn(keep_f32(code[q[i]] * absmax[i / (size_t)block]));
}

// The same for buffers aligned to 16 bytes and n below 2^35: 16 codes per thread, one 16-byte load and two 16-byte
// stores, and one division for the block's number (blocks are multiples of 64 values: the 16 share one).  Memory bound.
__global__ void __launch_bounds__(256) k_hidden_dequantize_wide(const uint8_t *__restrict__ q,
                                                                const float *__restrict__ absmax, size_t n,
                                                                uint32_t block16, __half *__restrict__ y) {
    __shared__ float code[256];
    const uint32_t c = blockIdx.x * 256u + threadIdx.x;
    const size_t i = (size_t)c * 16;
    v4i cv = {0, 0, 0, 0};
    float am = 0.0f;
    const bool full = i + 16 <= n;
    if (full) cv = *(const v4i *)(q + i);
    if (i < n) am = absmax[c / block16];
    code[threadIdx.x] = d_code_table.code[threadIdx.x];
    __syncthreads();
    if (full) {
        __half out[16];
#pragma unroll
        for (int e = 0; e < 16; e++) out[e] = decode_q8(code, ((uint32_t)cv[e >> 2] >> (8 * (e & 3))) & 255u, am);
        *(v4i *)(y + i) = *(const v4i *)out;
        *(v4i *)(y + i + 8) = *(const v4i *)(out + 8);
    } else {
        for (size_t e = i; e < n; e++) y[e] = decode_q8(code, q[e], am);
    }
}

// ------------------------------------------------------------- cache copies

// cache [nh][cap][d] (keys) + [nh][cap][d] (values)  <->  packed [2][nh][len][d]
__global__ void k_kv_copy(__half *cache, int nh, int cap, int d, int len, __half *packed, int to_cache) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t total = (size_t)2 * nh * len * d;
    if (i >= total) return;
    int c = (int)(i % d);
    size_t r = i / d;
    int pos = (int)(r % len);
    size_t ph = r / len;     // p * nh + h
    size_t ci = (ph * cap + pos) * d + c;
    if (to_cache) cache[ci] = packed[i]; else packed[i] = cache[ci];
}

}  // namespace

// ------------------------------------------------------------------ launchers

hipError_t ps_quantize_weight(const float *W, int N, int K, int8_t *wt, float *sw, hipStream_t st) {
    k_quantize_weight<<<N / 16, 256, 0, st>>>(W, K, wt, sw);
    return hipGetLastError();
}
hipError_t ps_untile_weight(const int8_t *wt, int N, int K, int8_t *wq, hipStream_t st) {
    k_untile_weight<<<N / 16, 256, 0, st>>>(wt, K, wq);
    return hipGetLastError();
}
hipError_t ps_fill_u32(uint32_t *p, size_t n, uint32_t v, hipStream_t st) {
    if (n == 0) return hipSuccess;
    k_fill_u32<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(p, n, v);
    return hipGetLastError();
}
hipError_t ps_copy_bytes(const void *src, void *dst, size_t n, hipStream_t st) {
    if (n == 0) return hipSuccess;
    k_copy_bytes<<<(unsigned)((n + 255) / 256), 256, 0, st>>>((const uint8_t *)src, (uint8_t *)dst, n);
    return hipGetLastError();
}
hipError_t ps_layernorm(const __half *x, const __half *g, const __half *b, float eps, int M, int H, __half *y,
                        uint8_t *flags, float theta, hipStream_t st) {
    // few rows: more threads per row (latency), many rows: more rows in flight (prefill calls of a 4096-wide block, two
    // LayerNorms each: 140 rows 188 us with 1024 threads per row, 199 with several rows per 256 threads; 351 rows 244
    // and 242: the line lies between).  Rows below 4096 columns, of which 1024 threads would hold two pairs each or fewer,
    // always take 256 threads.
    if (H % 8 || H > 16384) return hipErrorInvalidValue;       // span and client take multiples of 64 up to 16384
    if (M >= 256 || H < 4096) return launch_layernorm_rows<false>(x, QuantIn{}, g, b, eps, M, H, y, flags, theta, st);
    (flags ? k_layernorm_wide<true> : k_layernorm_wide<false>)<<<M, 1024, 0, st>>>(x, g, b, eps, H, y, flags, theta);
    return hipGetLastError();
}
hipError_t ps_layernorm_q8(const QuantIn &qin, const __half *g, const __half *b, float eps, int M,
                           int H, __half *y, uint8_t *flags, float theta, hipStream_t st) {
    // the line of ps_layernorm (measured there, on fp16 rows)
    if ((M >= 256 || H < 4096) && H % 8 == 0 && H <= 16384 && ((uintptr_t)qin.q & 7) == 0)
        return launch_layernorm_rows<true>(nullptr, qin, g, b, eps, M, H, y, flags, theta, st);
    if (M <= 256 && H >= 4096) k_layernorm_q8<1024><<<M, 1024, 0, st>>>(qin, g, b, eps, H, y, flags, theta);
    else k_layernorm_q8<256><<<M, 256, 0, st>>>(qin, g, b, eps, H, y, flags, theta);
    return hipGetLastError();
}
hipError_t ps_layernorm_codes(const __half *x, const QuantIn *qin, const __half *g, const __half *b, float eps, int M, int H, __half *y,
                              uint32_t *mask, int8_t *xq_tiled, int8_t *xo_tiled, float *sx, int8_t *xq_dbg, float theta,
                              const NormExchange &ex, hipStream_t st) {
    if (M < 2 || M > PS_NORM_ROWS_MAX || H % 64 || H > 16384 || !ex.records || !ex.tag) return hipErrorInvalidValue;
    const int rows = (M + 15) / 16 * 16, grid = rowquant_grid(rows);
    const uint32_t tb = ps_theta_to_bits(theta);
    const QuantIn q = qin ? *qin : QuantIn{};
#define PS_NORM(NT_, PER_) (qin ? k_layernorm_codes<NT_, PER_, true> : k_layernorm_codes<NT_, PER_, false>)<<<grid, NT_, H * 2, st>>>(x, q, g, b, eps, M, H, y, mask, xq_tiled, xo_tiled, sx, xq_dbg, tb, 1.0 / H, ex, rows, grid)
    if (H <= 1024) PS_NORM(256, 1);
    else if (H <= 2048) PS_NORM(512, 1);
    else if (H <= 4096) PS_NORM(1024, 1);
    else if (H <= 8192) PS_NORM(1024, 2);
    else PS_NORM(1024, 4);
#undef PS_NORM
    return hipGetLastError();
}
hipError_t ps_colmask(const __half *X, int M, int K, float theta, uint32_t *mask, hipStream_t st) {
    dim3 grid((K + 255) / 256, (M + 63) / 64);
    k_colmask<<<grid, 256, 0, st>>>(X, M, K, theta, mask);
    return hipGetLastError();
}
hipError_t ps_rowquant_tiled(const __half *X, int M, int K, uint32_t *mask, const uint8_t *flags, int8_t *xq_tiled,
                             int8_t *xo_tiled, float *sx, int8_t *xq_dbg, const OutlierPrep &pr, const RowDigits &rd,
                             hipStream_t st) {
    const int rows = (M + 15) / 16 * 16, grid = rowquant_grid(rows), items = outlier_prep_items(pr, M);
    const int extra4 = (items + 3) / 4, extra16 = (items + 15) / 16;
#define PS_ROWS(NT_, MODE_) k_rowquant_tiled_wide<NT_, 4, MODE_><<<grid + (NT_ == 256 ? extra4 : extra16), NT_, 0, st>>>(X, M, K, mask, flags, xq_tiled, xo_tiled, sx, xq_dbg, rows, grid, pr, rd)
    if (rd.xd) {
        if (K < 4096 || K > 65536 || flags) return hipErrorInvalidValue;
        PS_ROWS(1024, ROWS_DIGITS);
    } else if (K >= 4096 && K <= 16384 && M >= 512) {   // many rows: four times as many rows in flight per compute unit
        if (flags) PS_ROWS(256, ROWS_FLAGS);
        else PS_ROWS(256, ROWS_MASK);
    } else if (K >= 4096 && K <= 65536) {               // wide rows: 1024 threads keep the row in registers, one pass over X
        if (flags) PS_ROWS(1024, ROWS_FLAGS);
        else PS_ROWS(1024, ROWS_MASK);
    } else {
        auto kern = flags ? k_rowquant_tiled<ROWS_FLAGS> : k_rowquant_tiled<ROWS_MASK>;
        kern<<<grid + extra4, 256, 0, st>>>(X, M, K, mask, flags, xq_tiled, xo_tiled, sx, xq_dbg, rows, grid, pr);
    }
#undef PS_ROWS
    return hipGetLastError();
}
hipError_t ps_mask_count(const uint32_t *masks, int n_masks, int words, int32_t *out, hipStream_t st) {
    k_mask_count<<<n_masks, 256, 0, st>>>(masks, words, out);
    return hipGetLastError();
}
hipError_t ps_mask_to_bytes(const uint32_t *mask, int K, uint8_t *out, hipStream_t st) {
    k_mask_to_bytes<<<(K + 255) / 256, 256, 0, st>>>(mask, K, out);
    return hipGetLastError();
}
hipError_t ps_hidden_quantize(const __half *x, size_t n, int block, const CodeTable &tab, uint8_t *q, float *absmax,
                              hipStream_t st) {
    if (n == 0) return hipSuccess;
    const unsigned blocks = (unsigned)((n + block - 1) / block);
    // (a block starts at a multiple of 64 values: aligned buffers make every chunk aligned)
    if ((((uintptr_t)x & 15) | ((uintptr_t)q & 7)) == 0) {
        if (block <= 1024) k_hidden_quantize_wide<128, 1><<<blocks, 128, 0, st>>>(x, n, block, q, absmax);
        else if (block <= 4096) k_hidden_quantize_wide<512, 1><<<blocks, 512, 0, st>>>(x, n, block, q, absmax);
        else if (block <= 8192) k_hidden_quantize_wide<512, 2><<<blocks, 512, 0, st>>>(x, n, block, q, absmax);
        else k_hidden_quantize_wide<512, 4><<<blocks, 512, 0, st>>>(x, n, block, q, absmax);
    } else {
        k_hidden_quantize<<<blocks, 1024, 0, st>>>(x, n, block, tab, q, absmax);
    }
    return hipGetLastError();
}
hipError_t ps_hidden_dequantize(const uint8_t *q, const float *absmax, size_t n, int block, const CodeTable &tab,
                                __half *y, hipStream_t st) {
    if (n == 0) return hipSuccess;
    if ((((uintptr_t)q | (uintptr_t)y) & 15) == 0 && n < ((size_t)1 << 35)) {
        k_hidden_dequantize_wide<<<(unsigned)((n + 4095) / 4096), 256, 0, st>>>(q, absmax, n, (uint32_t)block / 16, y);
        return hipGetLastError();
    }
    k_hidden_dequantize<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(q, absmax, n, block, tab, y);
    return hipGetLastError();
}
hipError_t ps_kv_export(const __half *kv, int nh, int cap, int d, int len, __half *out, hipStream_t st) {
    size_t total = (size_t)2 * nh * len * d;
    if (total == 0) return hipSuccess;
    k_kv_copy<<<(unsigned)((total + 255) / 256), 256, 0, st>>>((__half *)kv, nh, cap, d, len, out, 0);
    return hipGetLastError();
}
hipError_t ps_kv_import(__half *kv, int nh, int cap, int d, int len, const __half *in, hipStream_t st) {
    size_t total = (size_t)2 * nh * len * d;
    if (total == 0) return hipSuccess;
    k_kv_copy<<<(unsigned)((total + 255) / 256), 256, 0, st>>>(kv, nh, cap, d, len, (__half *)in, 1);
    return hipGetLastError();
}

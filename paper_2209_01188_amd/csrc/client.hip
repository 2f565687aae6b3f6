// Client-side ends of a generation step: embedding lookup with its LayerNorm, final
// LayerNorm + LM head over the tied embedding matrix + greedy choice.  The LM head is a
// matrix-vector product over V x H fp16 weights read once: HBM bound.
#include <stdarg.h>
#include <string.h>

#include <mutex>
#include <new>

#include "../../include/petals_client.h"
#include "../../include/petals_span.h"
#include "common.h"
#include "host_util.h"
#include "rowops.h"

namespace {

constexpr int LM_THREADS = 1024;           // 16 waves: enough 16-byte loads in flight for one workgroup per compute unit
constexpr int LM_WAVES = LM_THREADS / 64;
constexpr int LM_GROUPS = 256;             // workgroups of the LM head = partial results per row
constexpr int LM_MAX_HIDDEN = 16384;
constexpr int LM_MAX_ROWS = 32;            // rows of hidden states multiplied per pass over the matrix (matrix-core form)

// One workgroup per token: gather the embedding row, LayerNorm in fp64, store fp16.
template <int NT>
__global__ void __launch_bounds__(NT) k_embed_ln(const int32_t *__restrict__ ids, const __half *__restrict__ E, int V,
                                                 int H, const __half *__restrict__ g, const __half *__restrict__ b,
                                                 float eps, __half *__restrict__ y) {
    __shared__ double sm[NT / 64];
    const int id = min(max(ids[blockIdx.x], 0), V - 1);
    const __half *xr = E + (size_t)id * H;
    __half *yr = y + (size_t)blockIdx.x * H;
    double mean, inv;
    row_moments<NT>(xr, H, sm, mean, inv, (double)eps);
    for (int k = threadIdx.x * 2; k < H; k += NT * 2)
        *(__half2 *)(yr + k) = ln_affine(*(const __half2 *)(xr + k), *(const __half2 *)(g + k),
                                         *(const __half2 *)(b + k), mean, inv);
}

struct Best {
    double v;
    int i;
};
__device__ __forceinline__ void take_better(Best &a, double v, int i) {   // larger value, then smaller index
    if (v > a.v || (v == a.v && i < a.i)) {
        a.v = v;
        a.i = i;
    }
}

// logits of ONE row of fp16 hidden states a[H] against all V rows of E.  The hidden row sits in
// LDS as fp64 (converted once); wave w of workgroup g takes the matrix rows (g * 16 + w) + i * 16 * gridDim.x, one row
// at a time: 64 lanes x 16 bytes per load instruction, four instructions in flight, a wave-wide fp64
// sum at the end of the row.  Each workgroup leaves its best (value, index).
__global__ void __launch_bounds__(LM_THREADS) k_lm_head(const __half *__restrict__ a, const __half *__restrict__ E,
                                                        int V, int H, float *__restrict__ logits,
                                                        Best *__restrict__ partial) {
    // element k = 8 c + j at [j][c]: the lanes of a wave hold consecutive chunks c, so their
    // 8-byte reads of one j are consecutive in LDS (no bank conflicts)
    extern __shared__ __align__(16) double ad[];       // [8][H / 8]
    __shared__ Best wbest[LM_WAVES];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nchunk = H >> 3;
    for (int k = threadIdx.x; k < H; k += LM_THREADS) ad[(k & 7) * nchunk + (k >> 3)] = (double)__half2float(a[k]);
    __syncthreads();
    Best best = Best{-INFINITY, 0x7fffffff};
    for (int v = blockIdx.x * LM_WAVES + wave; v < V; v += gridDim.x * LM_WAVES) {
        const __half *er = E + (size_t)v * H;
        double acc = 0.0;
        for (int c0 = lane; c0 < nchunk; c0 += 256) {
            v8h e[4];
#pragma unroll
            for (int u = 0; u < 4; u++)             // index clamped: every lane issues all four loads
                e[u] = __builtin_nontemporal_load((const v8h *)(er + (size_t)min(c0 + u * 64, nchunk - 1) * 8));
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int c = c0 + u * 64;
                if (c < nchunk) {
#pragma unroll
                    for (int j = 0; j < 8; j++) acc += (double)(float)e[u][j] * ad[j * nchunk + c];
                }
            }
        }
        const double s = wave_sum(acc);
        if (lane == 0 && logits) logits[v] = (float)s;
        take_better(best, s, v);
    }
    if (lane == 0) wbest[wave] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
        Best r = wbest[0];
        for (int w = 1; w < LM_WAVES; w++) take_better(r, wbest[w].v, wbest[w].i);
        partial[blockIdx.x] = r;
    }
}

// Several rows of hidden states at once, exactly, on the int8 matrix instruction.  Every fp16 value is an integer
// multiple of 2^-24, so with balanced 8-bit digits x = 2^-24 sum_j 256^j d_j, d_j in [-128, 127], four digits cover
// |x| < 127.5.  A product of two such values is the sum over the digit pairs (i, j) of 256^(i + j) d_i d_j: the pairs
// with the same i + j share an int32 accumulator (at most 4 * 2^14 * 16384 = 2^30), and the seven sums (nine, see below) meet in fp64
// once per logit - a few roundings of 2^-53 instead of one per column.
//
// The matrix is streamed once per 32 hidden rows: a wave owns WN tiles of 16 matrix rows (A operand) and walks their columns
// 64 at a time.  What bounds it are the bytes of the matrix, if the memory sees long pieces: with every lane loading its own
// operands (16 rows x 64 bytes per instruction) 250880 x 4096 at 8 rows took 398 us a call, and the arithmetic taken out
// changed nothing.  So the pieces are copied to LDS asynchronously, 256 consecutive bytes of a row at a time, and read
// from there in operand order (360 us; then the arithmetic counts: without it 326).  The wave cuts its values into digits
// itself, 13 instructions per four values and one per pair for the largest magnitude, two pieces of 64 columns in one
// straight line so that the matrix unit has work beside that (342 us, 6.0 TB/s; 14336 columns at 2 rows 1440 -> 1155;
// 17 to 32 rows, where a digit read from LDS meets one matrix tile only and products and arithmetic are the bound, 484 ->
// 470).  Every workgroup starts at another chunk: from column 0 on all of them fall on a few memory channels (417 us).
// A piece with a value of 0.246 and more takes a fourth digit, a third more products and twice the arithmetic; a multiply-add
// straight from fp16 is worth 5 % there (250880 x 4096, values of 0.3, 8 and 32 rows: 449 -> 426 and 636 -> 615 us; values of 0.02
// take 333 and 486; two pieces in a straight line there as well: 428 and 614, and the others 341).
// Two matrix tiles per wave also for 17 to 32 rows: 75 spilled registers, 731 us.  The hidden rows' digits (k_lm_prepare)
// go through LDS as well, shared by the 8 waves, one barrier per chunk.
//
// Hidden values of 127.5 and more (a feature that dominates its row) have two digits more: a 64-column
// piece in which any row has one is read a second time, for its products with digits 4 and 5; with the whole product on the fp64
// instruction instead one such feature made a call of 398 us one of 1000.  A tile of the matrix with a value of 127 or
// more, and every tile if a hidden row holds an infinity or NaN, is done again on the fp64 matrix instruction, where nothing
// bounds the values.
constexpr int LMD_CH = 2;                  // 64-column pieces per chunk
constexpr uint32_t LMD_BIG = 0x57f8;       // fp16 bits of 127.5: from here on a hidden value takes digits 4 and 5
constexpr uint32_t LMD_BIG_E = 0x57f0;     // fp16 bits of 127: from here on a matrix value takes more than four digits (it is moved by 1/4)
constexpr uint32_t LMD_SMALL = 0x33e0;     // fp16 bits of 0.246: below it three digits do, and lm_planes_small holds
constexpr int LMD_SHIFT = 0x400000;        // 1/4 in units of 2^-24

// Matrix values are cut into digits after 1/4 has been added, so that the third digit of a small one is positive and comes out of
// the sum below as it is; what that adds to the products, 64 times the sums of the hidden rows' digits, is taken off again,
// exactly, before the sums meet.
// Three planes of four values below LMD_SMALL in magnitude (two words of two halves).  x * 2^24 + 2^23 + 0x408080 is
// exact in fp32 and its low bytes are the digits of x + 1/4 plus 0x80, 0x80 and 0: one multiply-add straight from fp16,
// then byte permutations.
__device__ __forceinline__ void lm_planes_small(uint32_t w0, uint32_t w1, int (&p)[4]) {
    const uint32_t hb[4] = {w0 & 0xffffu, w0 >> 16, w1 & 0xffffu, w1 >> 16};
    uint32_t u[4];
#pragma unroll
    for (int i = 0; i < 4; i++)
        u[i] = __float_as_uint(fmaf(__half2float(__ushort_as_half((unsigned short)hb[i])), 16777216.0f, 8388608.0f + (LMD_SHIFT + 0x8080)));
    const uint32_t a = __builtin_amdgcn_perm(u[1], u[0], 0x05010400), b = __builtin_amdgcn_perm(u[3], u[2], 0x05010400);
    const uint32_t c = __builtin_amdgcn_perm(u[1], u[0], 0x0c0c0602), d = __builtin_amdgcn_perm(u[3], u[2], 0x0c0c0602);
    p[0] = (int)(__builtin_amdgcn_perm(b, a, 0x05040100) ^ 0x80808080u);
    p[1] = (int)(__builtin_amdgcn_perm(b, a, 0x07060302) ^ 0x80808080u);
    p[2] = (int)__builtin_amdgcn_perm(d, c, 0x05040100);                   // 1 .. 0x7f
}

template <int SHIFT = 0>
__device__ __forceinline__ uint32_t lm_digits(float f) {       // bytes = the four digits of f (+ SHIFT * 2^-24), below 127.5 in magnitude
    return ((uint32_t)(int)fmaf(f, 16777216.0f, 0.0f) + (0x80808080u + SHIFT)) ^ 0x80808080u;
}
// four values' digit words -> one word per plane (byte k = value k)
__device__ __forceinline__ void lm_planes(const uint32_t (&u)[4], int (&p)[4]) {
    const uint32_t a = __builtin_amdgcn_perm(u[1], u[0], 0x05010400), b = __builtin_amdgcn_perm(u[3], u[2], 0x05010400);
    const uint32_t c = __builtin_amdgcn_perm(u[1], u[0], 0x07030602), d = __builtin_amdgcn_perm(u[3], u[2], 0x07030602);
    p[0] = (int)__builtin_amdgcn_perm(b, a, 0x05040100);
    p[1] = (int)__builtin_amdgcn_perm(b, a, 0x07060302);
    p[2] = (int)__builtin_amdgcn_perm(d, c, 0x05040100);
    p[3] = (int)__builtin_amdgcn_perm(d, c, 0x07060302);
}

// digits 0 to 3 of a finite value of 127.5 or more in magnitude, and its digits 4 and 5: x = low + 256 y, low in
// [-128.5, 127.5) and a multiple of 1/16, |y| <= 256
__device__ __forceinline__ uint32_t lm_digits_wide(float f, int &d4, int &d5) {
    const float y = floorf(fmaf(f, 0.00390625f, 0.501953125f));
    d4 = (((int)y + 128) & 255) - 128;
    d5 = ((int)y - d4) >> 8;
    return (((uint32_t)(int)(fmaf(y, -256.0f, f) * 16.0f) << 20) + 0x80808080u) ^ 0x80808080u;
}

// What k_lm_prepare says of a hidden row: whether it holds an infinity or NaN, whether any value needs digits 4 and 5,
// the 64-column pieces with such values, and the sums of its digits.
constexpr int LM_PIECE_WORDS = LM_MAX_HIDDEN / 64 / 32;
enum { LM_NONFINITE = 1, LM_WIDE = 2 };
struct LmRow {
    int flags;
    uint32_t wide[LM_PIECE_WORDS];
    int sum[4];                // of the row's digits 0 to 3, plane by plane
};

// LayerNorm of one hidden row per workgroup: the fp16 row to a (what the fp64 form reads), its digit planes 0 to 3 to
// dig[(kt * 4 + plane) * MT + row tile][lane][16 bytes], planes 4 and 5 to dig2[(kt * 2 + plane - 4) * MT + row tile].
// Rows beyond `rows` (up to the end of the row tile) get zero digits.
template <int PER>
__global__ void __launch_bounds__(512) k_lm_prepare(const __half *__restrict__ x, const __half *__restrict__ g,
                                                    const __half *__restrict__ b, float eps, int rows, int H, int MT,
                                                    __half *__restrict__ a, uint8_t *__restrict__ dig, uint8_t *__restrict__ dig2,
                                                    LmRow *__restrict__ info) {
    constexpr int NT = 512;
    __shared__ double sm[NT / 64];
    __shared__ LmRow here;
    if (threadIdx.x < sizeof(LmRow) / 4) ((uint32_t *)&here)[threadIdx.x] = 0u;
    __syncthreads();
    const int t = blockIdx.x, mt = t >> 4, row = t & 15;
    const __half *xr = x + (size_t)t * H;
    const bool live = t < rows;
    v8h v[PER];
    double s = 0.0, q = 0.0, mean = 0.0, inv = 0.0;
    int sum[4] = {0, 0, 0, 0};
    if (live) {
#pragma unroll
        for (int i = 0; i < PER; i++) {
            const int k = (threadIdx.x + i * NT) * 8;
            if (k < H) {
                v[i] = *(const v8h_any *)(xr + k);
#pragma unroll
                for (int e = 0; e < 8; e++) s += (double)(float)v[i][e];
            }
        }
        mean = block_sum<NT / 64>(s, sm) / (double)H;
#pragma unroll
        for (int i = 0; i < PER; i++) {
            if ((int)(threadIdx.x + i * NT) * 8 < H) {
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    const double d = (double)(float)v[i][e] - mean;
                    q += d * d;
                }
            }
        }
        inv = 1.0 / sqrt(block_sum<NT / 64>(q, sm) / (double)H + (double)eps);
    }
#pragma unroll
    for (int i = 0; i < PER; i++) {
        const int k = (threadIdx.x + i * NT) * 8;
        if (k < H) {
            // columns 64 kt + 32 h + 8 g .. +8: bytes 8 h .. +8 of lane (g, row)
            const int kt = k >> 6, h = (k >> 5) & 1, gg = (k >> 3) & 3;
            __half out[8];
            int lo[4] = {0, 0, 0, 0}, hi[4] = {0, 0, 0, 0};
            uint32_t up[2][2] = {{0u, 0u}, {0u, 0u}};            // digits 4 and 5, packed like the planes
            if (live) {
                const v8h gv = *(const v8h_any *)(g + k), bv = *(const v8h_any *)(b + k);
                uint32_t u[2][4];
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    out[e] = d2h_rn(((double)(float)v[i][e] - mean) * inv * (double)(float)gv[e] + (double)(float)bv[e]);
                    u[e >> 2][e & 3] = lm_digits(__half2float(out[e]));
                    const uint32_t bits = __half_as_ushort(out[e]) & 0x7fffu;
                    if (bits >= LMD_BIG) {                       // rare
                        int d4, d5;
                        u[e >> 2][e & 3] = lm_digits_wide(__half2float(out[e]), d4, d5);
                        up[0][e >> 2] |= (uint32_t)(d4 & 255) << (8 * (e & 3));
                        up[1][e >> 2] |= (uint32_t)(d5 & 255) << (8 * (e & 3));
                        atomicOr(&here.flags, bits >= 0x7c00u ? LM_NONFINITE : LM_WIDE);
                        atomicOr(&here.wide[kt >> 5], 1u << (kt & 31));
                    }
                }
                *(v8h *)(a + (size_t)t * H + k) = *(const v8h *)out;
                lm_planes(u[0], lo);
                lm_planes(u[1], hi);
#pragma unroll
                for (int pl = 0; pl < 4; pl++)
                    sum[pl] = __builtin_amdgcn_sdot4(hi[pl], 0x01010101, __builtin_amdgcn_sdot4(lo[pl], 0x01010101, sum[pl], false), false);
            }
#pragma unroll
            for (int pl = 0; pl < 4; pl++)
                *(v2i *)(dig + (((size_t)(kt * 4 + pl) * MT + mt) * 64 + gg * 16 + row) * 16 + h * 8) = (v2i){lo[pl], hi[pl]};
#pragma unroll
            for (int pl = 0; pl < 2; pl++)
                *(v2i *)(dig2 + (((size_t)(kt * 2 + pl) * MT + mt) * 64 + gg * 16 + row) * 16 + h * 8) = (v2i){(int)up[pl][0], (int)up[pl][1]};
        }
    }
#pragma unroll
    for (int pl = 0; pl < 4; pl++) {
        const int w = (int)wave_sum((float)sum[pl]);          // at most 64 x 32 x 128: exact
        if ((threadIdx.x & 63) == 0) atomicAdd(&here.sum[pl], w);
    }
    __syncthreads();
    if (threadIdx.x < sizeof(LmRow) / 4) ((uint32_t *)&info[t])[threadIdx.x] = ((const uint32_t *)&here)[threadIdx.x];
}

// the fp64 form of one wave's products: 16 matrix rows x MT tiles of 16 hidden rows.  Lane (row l%16, group l/16)
// feeds 8 consecutive values of its matrix row and of its hidden row to 8 instructions - any pairing of the
// contraction index works as long as both operands use the same one.  Register r of lane (g, c): matrix row 4r + g.
template <int MT>
__device__ __forceinline__ void lm_tile_f64(const __half *__restrict__ er, const __half *__restrict__ a, int rows, int H,
                                                      v4d (&acc)[MT]) {
    const int lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
#pragma unroll
    for (int j = 0; j < MT; j++) acc[j] = (v4d){0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int k = 0; k < H; k += 32) {
        const v8h e = *(const v8h *)(er + k);
#pragma unroll
        for (int j = 0; j < MT; j++) {
            const v8h x = *(const v8h *)(a + (size_t)min(j * 16 + c, rows - 1) * H + g * 8 + k);
#pragma unroll
            for (int q = 0; q < 8; q++)
                acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)(float)e[q], (double)(float)x[q], acc[j], 0, 0, 0);
        }
    }
}

// LDS of k_lm_head_digits: per wave a ring of matrix pieces (16 WN rows x LMD_CH * 128 bytes each), then a ring of the hidden
// rows' digits for as many pieces, shared by the workgroup.  64 to 128 KB of the matrix are in flight per compute unit.
template <int WN, int MT>
struct LmLds {
    static constexpr int SLOT = WN * 16 * LMD_CH * 128, RING = WN == 2 ? 2 : 3;
    static constexpr int DIGITS = LMD_CH * 4 * MT * 1024, BYTES = RING * (8 * SLOT + DIGITS);
};

typedef _Float16 v2h __attribute__((ext_vector_type(2)));
__device__ __forceinline__ v2h lm_max_abs(v2h m, v2h x) {     // one instruction; NaN wins
    return __builtin_elementwise_maximum(__builtin_elementwise_maximum(m, x), -x);
}
// one asynchronous copy of 64 x 16 bytes to LDS, in the order of the lanes; zeros from `bytes` on
template <int AUX>
__device__ __forceinline__ void lm_copy16(const void *base, int bytes, unsigned char *to, uint32_t offset) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void *)base, 0, bytes, 0x00020000),
                                             (__attribute__((address_space(3))) void *)to, 16, offset, 0, 0, AUX);
}

template <int WN, int MT>
__global__ void __launch_bounds__(512, 2) k_lm_head_digits(const __half *__restrict__ a, const uint8_t *__restrict__ dig,
                                                           const uint8_t *__restrict__ dig2, const LmRow *__restrict__ info, int rows,
                                                           const __half *__restrict__ E,
                                                           int V, int H, float *__restrict__ logits, Best *__restrict__ partial) {
    constexpr int CH = LMD_CH, RING = LmLds<WN, MT>::RING, SLOT = LmLds<WN, MT>::SLOT, DIGITS = LmLds<WN, MT>::DIGITS;
    constexpr int NE = SLOT / 1024, ND = DIGITS / 8192;      // copies a wave asks for per chunk: matrix, digits
    constexpr int SEGS = CH * 8, RPI = 64 / SEGS;            // 16-byte segments of a row in a slot, rows per copy
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ Best wbest[8][MT * 16];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
    unsigned char *ring = lds + wave * (RING * SLOT), *dstage = lds + 8 * RING * SLOT;
    const int KT = H >> 6, nch = (KT + CH - 1) / CH, ntiles = (V + 15) >> 4;
    __shared__ uint32_t wide[LM_PIECE_WORDS];                // pieces of any row with digits 4 and 5
    __shared__ int dsum[MT * 16][4];                         // 64 times the sums of the hidden rows' digits (read behind many barriers)
    if (threadIdx.x < MT * 64) dsum[threadIdx.x >> 2][threadIdx.x & 3] = info[threadIdx.x >> 2].sum[threadIdx.x & 3] * (LMD_SHIFT >> 16);
    const int flags = lane < rows ? info[lane].flags : 0;    // (every wave by itself: no barrier in front of the first requests)
    const bool all_f64 = __any(flags & LM_NONFINITE), any_wide = __any(flags & LM_WIDE);
    if (any_wide) {                                          // rare; the same in all waves
        if (threadIdx.x < LM_PIECE_WORDS) {
            uint32_t w = 0;
            for (int t = 0; t < rows; t++) w |= info[t].wide[threadIdx.x];
            wide[threadIdx.x] = w;
        }
        __syncthreads();
    }
    const bool wide_store = logits && V % 4 == 0 && ((uintptr_t)logits & 15) == 0;
    Best best[MT];
#pragma unroll
    for (int j = 0; j < MT; j++) best[j] = Best{-INFINITY, 0x7fffffff};

    // Copies: one takes RPI rows x SEGS segments of a slot, in the order of the lanes; segment s of row r lies at position
    // s ^ (r & SEGS - 1) of the row, so that the 16 rows a lane group reads one segment of do not share banks.  Rows beyond
    // the matrix and chunks beyond the last round are out of the descriptor's bounds and read as zeros, the columns behind a
    // ragged last piece are not used.  (Offsets sit in the vector operand: the check against the bounds is sure to see them.)
    uint32_t voff[NE];
#pragma unroll
    for (int j = 0; j < NE; j++) {
        const int r = j * RPI + lane / SEGS;
        voff[j] = (uint32_t)r * (uint32_t)(H * 2) + (((lane & (SEGS - 1)) ^ (r & (SEGS - 1))) << 4);
    }
    const __half *pbase = E;                                 // this wave's rows of the round that is being requested, and their bytes
    int pbytes = 0;
    auto rows_of = [&](int grp) {
        const long long row0 = (long long)(grp * 8 + wave) * (WN * 16), left = grp * 8 * WN < ntiles ? (long long)V - row0 : 0;
        pbase = E + (left > 0 ? row0 : 0) * H;
        pbytes = left > 0 ? (int)min(left, (long long)WN * 16) * H * 2 : 0;
    };
    auto load_e = [&](int slot, int ch) {
#pragma unroll
        for (int j = 0; j < NE; j++)
            lm_copy16<2 /* non-temporal */>(pbase, pbytes, ring + slot * SLOT + j * 1024, voff[j] + ch * (CH * 128));
    };
    auto load_d = [&](int buf, int ch) {
#pragma unroll
        for (int j = 0; j < ND; j++)
            lm_copy16<0>(dig, KT * 4 * MT * 1024, dstage + buf * DIGITS + (wave + 8 * j) * 1024, ch * DIGITS + (wave + 8 * j) * 1024 + lane * 16);
    };
    // Every workgroup starts its rows at another chunk and wraps around: rows are a power of two or so of bytes apart,
    // and with all workgroups at the same column the requests of the whole device fall on a few memory channels.
    const int rot = (blockIdx.x >> 3) % nch;
    // The ring runs through the rounds of a workgroup without draining.  (pg, pi, pch): round, index and chunk that the next
    // request of matrix pieces is for, dch: the chunk of digits that is, slot: the place of the chunk at hand in both rings.
    int pg = blockIdx.x, pi = 0, pch = rot, dch = rot, slot = 0;
    rows_of(pg);
    auto request = [&](int s) {
        load_e(s, pch);
        pch = pch + 1 == nch ? 0 : pch + 1;
        if (++pi == nch) { pi = 0; pch = rot; pg += gridDim.x; rows_of(pg); }
    };
    auto request_digits = [&](int s) {
        load_d(s, dch);
        dch = dch + 1 == nch ? 0 : dch + 1;
    };
    if (!all_f64) {
#pragma unroll
        for (int s = 0; s < RING; s++) {
            if (s < RING - 1) request_digits(s);
            request(s);
        }
    }
    for (int grp = blockIdx.x; grp * 8 * WN < ntiles; grp += gridDim.x) {       // the same rounds for the whole workgroup
        const int vt0 = (grp * 8 + wave) * WN;
        v4i acc[WN][MT][9];
#pragma unroll
        for (int p = 0; p < WN; p++)
#pragma unroll
            for (int j = 0; j < MT; j++)
#pragma unroll
                for (int s = 0; s < 9; s++) acc[p][j][s] = (v4i){0, 0, 0, 0};
        bool slow = all_f64;
        if (!all_f64) {
            int ch = rot;
            for (int i_ch = 0; i_ch < nch; i_ch++) {
                // This chunk has landed: matrix pieces are asked for RING chunks ahead, digits RING - 1 (before the pieces of
                // the same step), so behind this chunk's digits there are RING - 1 chunks' pieces and RING - 2 chunks' digits
                // in flight.  Later stores only make the wait longer.
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(NE + (RING - 2) * (NE + ND)) : "memory");
                __builtin_amdgcn_s_barrier();    // ... in all waves, and everybody is done with the digits of the chunk before
                asm volatile("" ::: "memory");
                request_digits(slot == 0 ? RING - 1 : slot - 1);
                v4i e[CH][WN][2];
#pragma unroll
                for (int u = 0; u < CH; u++)
#pragma unroll
                    for (int p = 0; p < WN; p++)
#pragma unroll
                        for (int h = 0; h < 2; h++)
                            e[u][p][h] = *(const v4i *)(ring + slot * SLOT + (p * 16 + c) * (CH * 128) + (((u * 8 + h * 4 + g) ^ ((p * 16 + c) & (SEGS - 1))) << 4));
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // the slot is free again
                request(slot);
                const unsigned char *sb = dstage + slot * DIGITS + lane * 16;
                v2h big[CH];                             // largest magnitudes of this lane's values (NaN if there is one)
#pragma unroll
                for (int u = 0; u < CH; u++) {
                    big[u] = (v2h){(_Float16)0.0f, (_Float16)0.0f};
#pragma unroll
                    for (int p = 0; p < WN; p++)
#pragma unroll
                        for (int i = 0; i < 8; i++) {
                            const int word = e[u][p][i >> 2][i & 3];
                            big[u] = lm_max_abs(big[u], *(const v2h *)&word);
                        }
                }
                static_assert(CH == 2, "pieces of a chunk");
                const v2h both = lm_max_abs(big[0], big[1]);
                const uint32_t bits = *(const uint32_t *)&both & 0x7fff7fffu;
                const bool full = ch * CH + CH <= KT;
                if (full && !__any(max(bits & 0xffffu, bits >> 16) >= LMD_SMALL)) {
                    // nearly always: straight-line, so that one piece's arithmetic runs beside the other's products
#pragma unroll
                    for (int u = 0; u < CH; u++) {
                        v4i d[WN][3];
#pragma unroll
                        for (int p = 0; p < WN; p++)
#pragma unroll
                            for (int q = 0; q < 4; q++) {        // values 4 q .. +4 of this lane's 16
                                int pl[4];
                                lm_planes_small((uint32_t)e[u][p][q >> 1][2 * (q & 1)], (uint32_t)e[u][p][q >> 1][2 * (q & 1) + 1], pl);
#pragma unroll
                                for (int i = 0; i < 3; i++) d[p][i][q] = pl[i];
                            }
#pragma unroll
                        for (int j = 0; j < 4; j++)
#pragma unroll
                            for (int m = 0; m < MT; m++) {
                                const v4i xb = *(const v4i *)(sb + ((u * 4 + j) * MT + m) * 1024);
#pragma unroll
                                for (int i = 0; i < 3; i++)
#pragma unroll
                                    for (int p = 0; p < WN; p++)
                                        acc[p][m][i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(d[p][i], xb, acc[p][m][i + j], 0, 0, 0);
                            }
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < CH; u++) {
                        if (ch * CH + u >= KT) continue;         // ragged last chunk
                        const uint32_t ub = *(const uint32_t *)&big[u] & 0x7fff7fffu;
                        slow |= (bool)__any(max(ub & 0xffffu, ub >> 16) >= LMD_BIG_E);
                        v4i d[WN][4];
#pragma unroll
                        for (int p = 0; p < WN; p++)
#pragma unroll
                            for (int q = 0; q < 4; q++) {
                                const uint32_t w0 = (uint32_t)e[u][p][q >> 1][2 * (q & 1)], w1 = (uint32_t)e[u][p][q >> 1][2 * (q & 1) + 1];
                                const uint32_t hb[4] = {w0 & 0xffffu, w0 >> 16, w1 & 0xffffu, w1 >> 16};
                                uint32_t dw[4];
                                int pl[4];
#pragma unroll
                                for (int i = 0; i < 4; i++) dw[i] = lm_digits<LMD_SHIFT>(__half2float(__ushort_as_half((unsigned short)hb[i])));
                                lm_planes(dw, pl);
#pragma unroll
                                for (int i = 0; i < 4; i++) d[p][i][q] = pl[i];
                            }
#pragma unroll
                        for (int j = 0; j < 4; j++)
#pragma unroll
                            for (int m = 0; m < MT; m++) {
                                const v4i xb = *(const v4i *)(sb + ((u * 4 + j) * MT + m) * 1024);
#pragma unroll
                                for (int i = 0; i < 4; i++)
#pragma unroll
                                    for (int p = 0; p < WN; p++)
                                        acc[p][m][i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(d[p][i], xb, acc[p][m][i + j], 0, 0, 0);
                            }
                    }
                }
                ch = ch + 1 == nch ? 0 : ch + 1;         // behind the last chunk comes the first of the next round
                slot = slot + 1 == RING ? 0 : slot + 1;
            }
            if (any_wide) {                                  // digits 4 and 5 of the hidden rows, piece by piece
                for (int wi = 0; wi < LM_PIECE_WORDS; wi++)
                    for (uint32_t left = __builtin_amdgcn_readfirstlane(wide[wi]); left; left &= left - 1u) {
                        const int kt = wi * 32 + __ffs((int)left) - 1;
#pragma unroll
                        for (int p = 0; p < WN; p++) {
                            const __half *er = E + (size_t)min((vt0 + p) * 16 + c, V - 1) * H + g * 8;
                            v4i d[4];
#pragma unroll
                            for (int h = 0; h < 2; h++) {
                                const v4i w = *(const v4i *)(er + (size_t)kt * 64 + h * 32);
#pragma unroll
                                for (int q = 0; q < 2; q++) {
                                    const uint32_t w0 = (uint32_t)w[2 * q], w1 = (uint32_t)w[2 * q + 1];
                                    const uint32_t hb[4] = {w0 & 0xffffu, w0 >> 16, w1 & 0xffffu, w1 >> 16};
                                    uint32_t dw[4];
                                    int pl[4];
#pragma unroll
                                    for (int i = 0; i < 4; i++) dw[i] = lm_digits(__half2float(__ushort_as_half((unsigned short)hb[i])));
                                    lm_planes(dw, pl);
#pragma unroll
                                    for (int i = 0; i < 4; i++) d[i][2 * h + q] = pl[i];
                                }
                            }
#pragma unroll
                            for (int j = 0; j < 2; j++)
#pragma unroll
                                for (int m = 0; m < MT; m++) {
                                    const v4i xb = *(const v4i *)(dig2 + ((size_t)(kt * 2 + j) * MT + m) * 1024 + lane * 16);
#pragma unroll
                                    for (int i = 0; i < 4; i++)
                                        acc[p][m][4 + i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(d[i], xb, acc[p][m][4 + i + j], 0, 0, 0);
                                }
                        }
                    }
            }
        }
#pragma unroll
        for (int p = 0; p < WN; p++) {
            if (vt0 + p >= ntiles) continue;                 // wave-uniform
            v4d val[MT];
            if (slow) {
                lm_tile_f64<MT>(E + (size_t)min((vt0 + p) * 16 + c, V - 1) * H + g * 8, a, rows, H, val);
            } else {
#pragma unroll
                for (int j = 0; j < MT; j++)
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        double t = (double)acc[p][j][8][r];
#pragma unroll
                        for (int s = 7; s >= 0; s--) t = t * 256.0 + (double)(acc[p][j][s][r] - (s >= 2 && s < 6 ? dsum[j * 16 + c][s - 2] : 0));
                        val[j][r] = t * 0x1p-48;
                    }
            }
#pragma unroll
            for (int j = 0; j < MT; j++) {
                const int t = j * 16 + c;
                if (t >= rows) continue;
                // the fp64 instruction returns matrix row 4r + g in register r of lane group g, the int8 one 4g + r
                const int v0 = (vt0 + p) * 16 + (slow ? g : 4 * g), dv = slow ? 4 : 1;
                if (wide_store && !slow && v0 < V)
                    *(v4f *)(logits + (size_t)t * V + v0) = (v4f){(float)val[j][0], (float)val[j][1], (float)val[j][2], (float)val[j][3]};
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const int v = v0 + r * dv;
                    if (v >= V) continue;
                    if (logits && (slow || !wide_store)) logits[(size_t)t * V + v] = (float)val[j][r];
                    take_better(best[j], val[j][r], v);
                }
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // nothing may land in LDS after the workgroup's end
    // the four lane groups of a wave hold candidates of the same hidden rows, then the waves
#pragma unroll
    for (int j = 0; j < MT; j++) {
#pragma unroll
        for (int off = 16; off < 64; off <<= 1) {
            const double v2 = __shfl_xor(best[j].v, off);
            const int i2 = __shfl_xor(best[j].i, off);
            take_better(best[j], v2, i2);
        }
        if (g == 0) wbest[wave][j * 16 + c] = best[j];
    }
    __syncthreads();
    if (threadIdx.x < MT * 16 && (int)threadIdx.x < rows) {
        Best r = wbest[0][threadIdx.x];
        for (int w2 = 1; w2 < 8; w2++) take_better(r, wbest[w2][threadIdx.x].v, wbest[w2][threadIdx.x].i);
        partial[threadIdx.x * LM_GROUPS + blockIdx.x] = r;
    }
}

template <int WN, int MT>
hipError_t lm_head_digits(int groups, const __half *a, const uint8_t *dig, const uint8_t *dig2, const LmRow *info, int rows,
                          const __half *E, int V, int H, float *logits, Best *partial, hipStream_t st) {
    constexpr int lds = LmLds<WN, MT>::BYTES;
    auto kern = k_lm_head_digits<WN, MT>;
    static std::mutex attr_lock;
    static bool attr_set = false;
    {
        std::lock_guard<std::mutex> hold(attr_lock);
        if (!attr_set) {
            hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
    }
    kern<<<groups, 512, lds, st>>>(a, dig, dig2, info, rows, E, V, H, logits, partial);
    return hipGetLastError();
}

// the best of the workgroups' candidates of each hidden row
__global__ void __launch_bounds__(64) k_lm_pick(const Best *__restrict__ partial, int ngroups, int32_t *__restrict__ next) {
    const Best *p = partial + (size_t)blockIdx.x * LM_GROUPS;
    Best r = Best{-INFINITY, 0x7fffffff};
    for (int i = threadIdx.x; i < ngroups; i += 64) take_better(r, p[i].v, p[i].i);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double v = __shfl_xor(r.v, off);
        const int i = __shfl_xor(r.i, off);
        take_better(r, v, i);
    }
    if (threadIdx.x == 0) next[blockIdx.x] = r.i;
}

size_t align_up(size_t v) { return (v + 255) & ~(size_t)255; }

}  // namespace

// ------------------------------------------------------------------------------------------------
// Choice of the next token by temperature / top-k sampling with the caller's uniform numbers.
// One workgroup of 16 waves per row of logits.  Wave w owns the contiguous indices [w Cw, (w+1) Cw); in
// iteration j its lanes read 4 x 64 consecutive floats (index = start + 256 j + 64 e + lane, e = 0..3), so every
// load instruction is 256 contiguous bytes and "index order" is the order (wave, j, e, lane).  Whatever depends
// on that order (which of several equal logits at the top-k boundary stay in play; whose running sum first
// exceeds the target) is resolved level by level: waves, then iterations of one wave, then the 256 elements of
// one iteration, with ballots and ordered scans.
namespace {

// unsigned keys that order like the floats they come from (-0 counts as +0)
__device__ __forceinline__ uint32_t order_key(float f) {
    const uint32_t u = __float_as_uint(f + 0.0f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// One radix step, done by the first wave: the bin b (from 255 downwards) in which the running count of keys reaches
// `remaining`, and how many of that bin's keys are still needed.  hist: 256 counts; lane L takes bins 4L .. 4L+3.
__device__ __forceinline__ void radix_pick_bin(const int *hist, int remaining, int lane, uint32_t &bin, int &need) {
    const int h0 = hist[4 * lane], h1 = hist[4 * lane + 1], h2 = hist[4 * lane + 2], h3 = hist[4 * lane + 3];
    int suf = h0 + h1 + h2 + h3;                                 // becomes the count of this lane's and all higher bins
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_down(suf, off);
        if (lane + off < 64) suf += o;
    }
    const int above = __shfl_down(suf, 1);
    int cum = lane < 63 ? above : 0;                             // keys in bins above this lane's
    const bool mine = suf >= remaining && cum < remaining;       // exactly one lane, if remaining <= total
    int b = 4 * lane + 3, n = remaining - cum;
    if (cum + h3 < remaining) { cum += h3; b = 4 * lane + 2; n = remaining - cum;
        if (cum + h2 < remaining) { cum += h2; b = 4 * lane + 1; n = remaining - cum;
            if (cum + h1 < remaining) { cum += h1; b = 4 * lane; n = remaining - cum; } } }
    const unsigned long long who = __ballot(mine);
    const int src = who ? __ffsll((long long)who) - 1 : 0;       // lane 0 (bin 0 .. 3) if the counts fall short
    bin = (uint32_t)__shfl(b, src);
    need = __shfl(n, src);
}

__device__ __forceinline__ double wave_scan_incl(double v, int lane) {
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const double o = __shfl_up(v, off);
        if (lane >= off) v += o;
    }
    return v;
}

__global__ void __launch_bounds__(1024) k_sample(const float *__restrict__ logits, int V, float temperature, int top_k,
                                                 const float *__restrict__ uni, int32_t *__restrict__ next) {
    __shared__ uint32_t s_key[16];
    __shared__ int s_idx[16], s_eq[16], hist[256];
    __shared__ double s_sum[16];
    __shared__ uint32_t sh_prefix;
    __shared__ int sh_need;
    const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float *l = logits + (size_t)row * V;
    const int Cw = (((V + 15) / 16) + 255) / 256 * 256;
    const int seg0 = min(V, wave * Cw), seg1 = min(V, seg0 + Cw), nit = (seg1 - seg0 + 255) / 256;
    const unsigned long long lt = (1ull << lane) - 1ull;               // lanes below this one

    // 1. the largest logit, lowest index first (a thread meets its indices in ascending order)
    uint32_t bk = 0;
    int bi = 0x7fffffff;
    for (int j0 = 0; j0 < nit; j0 += 4) {                 // 16 loads in flight: the pass is bound by their latency
        float f[16];
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const int v = seg0 + j0 * 256 + i * 64 + lane;
            f[i] = v < seg1 ? l[v] : -INFINITY;
        }
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const int v = seg0 + j0 * 256 + i * 64 + lane;
            const uint32_t k = order_key(f[i]);
            if (v < seg1 && k > bk) { bk = k; bi = v; }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t k2 = (uint32_t)__shfl_xor((int)bk, off);
        const int i2 = __shfl_xor(bi, off);
        if (k2 > bk || (k2 == bk && i2 < bi)) { bk = k2; bi = i2; }
    }
    if (lane == 0) { s_key[wave] = bk; s_idx[wave] = bi; }
    __syncthreads();
    bk = s_key[0]; bi = s_idx[0];
    for (int w = 1; w < 16; w++)
        if (s_key[w] > bk || (s_key[w] == bk && s_idx[w] < bi)) { bk = s_key[w]; bi = s_idx[w]; }
    const int best = min(bi, V - 1);                        // (a row of nothing but NaN patterns has no best: stay in bounds)
    if (temperature == 0.0f || top_k == 1) {               // the greedy choice (uniform over the workgroup)
        if (tid == 0) next[row] = best;
        return;
    }

    // 2. key of the top_k-th largest logit by a radix select over the four bytes of the keys
    const bool all = top_k <= 0 || top_k >= V;
    uint32_t thr = 0;
    int need_eq = 0;                                        // in play: key > thr, and the first need_eq with key == thr
    if (!all) {
        uint32_t prefix = 0;
        int remaining = top_k;
        for (int pass = 3; pass >= 0; pass--) {
            for (int i = tid; i < 256; i += 1024) hist[i] = 0;
            __syncthreads();
            const int shift = pass * 8;
            for (int j = 0; j < nit; j++)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const int v = seg0 + j * 256 + e * 64 + lane;
                    bool in = v < seg1;
                    uint32_t k = 0;
                    if (in) {
                        k = order_key(l[v]);
                        in = pass == 3 || (k >> (shift + 8)) == prefix;
                    }
                    // lanes of a wave that hit the same bin add once: the high bytes of logits crowd a few bins
                    uint32_t bin = (k >> shift) & 255u;
                    if (pass < 3) {                          // few keys share the prefix by now
                        if (in) atomicAdd(&hist[bin], 1);
                        continue;
                    }
                    unsigned long long todo = __ballot(in);
                    while (todo) {
                        const int first = __ffsll((long long)todo) - 1;
                        const uint32_t b0 = (uint32_t)__shfl((int)bin, first);
                        const unsigned long long same = __ballot(in && bin == b0);
                        if (lane == first) atomicAdd(&hist[b0], __popcll(same));
                        todo &= ~same;
                    }
                }
            __syncthreads();
            if (wave == 0) {
                uint32_t b;
                int n;
                radix_pick_bin(hist, remaining, lane, b, n);
                if (lane == 0) { sh_prefix = (prefix << 8) | b; sh_need = n; }
            }
            __syncthreads();
            prefix = sh_prefix;
            remaining = sh_need;
        }
        thr = prefix;
        need_eq = remaining;
    }

    // 3. one pass: per wave the number of logits equal to the threshold and the sum of
    //    p = exp((l - l_max) / temperature) over its logits in play, given how many equal ones precede the wave.
    //    The count comes first (its own pass) because the sum needs it.
    int eq_wave = 0;
    if (!all) {
        for (int j = 0; j < nit; j++)
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const int v = seg0 + j * 256 + e * 64 + lane;
                eq_wave += __popcll(__ballot(v < seg1 && order_key(l[v]) == thr));
            }
        if (lane == 0) s_eq[wave] = eq_wave;
        __syncthreads();
    }
    int eq_before_wave = 0;
    if (!all)
        for (int w = 0; w < wave; w++) eq_before_wave += s_eq[w];

    const double Td = (double)temperature, lm = (double)l[best];
    // p of the element (j, e) of this lane, 0 if it is not in play; eq_seen = equal ones before iteration j's
    // element group e in this wave (updated here)
    auto weight = [&](int j, int e, int &eq_seen) -> double {
        const int v = seg0 + j * 256 + e * 64 + lane;
        const bool valid = v < seg1;
        const float lv = valid ? l[v] : 0.0f;
        bool keep = valid;
        if (!all) {
            const uint32_t k = order_key(lv);
            const bool eq = valid && k == thr;
            const unsigned long long m = __ballot(eq);
            keep = valid && (k > thr || (eq && eq_seen + __popcll(m & lt) < need_eq));
            eq_seen += __popcll(m);
        }
        return keep ? exp(((double)lv - lm) / Td) : 0.0;
    };
    double sum = 0.0;
    {
        int eq_seen = eq_before_wave;
        for (int j = 0; j < nit; j++)
#pragma unroll
            for (int e = 0; e < 4; e++) sum += weight(j, e, eq_seen);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
    if (lane == 0) s_sum[wave] = sum;
    __syncthreads();
    double total = 0.0;
    for (int w = 0; w < 16; w++) total += s_sum[w];
    const double target = (double)uni[row] * total;

    // 4. the wave whose segment holds the target (the last wave with anything in play if rounding leaves none)
    int wstar = -1, wlast = -1;
    double before = 0.0;
    {
        double c = 0.0;
        for (int w = 0; w < 16; w++) {
            if (s_sum[w] > 0.0) wlast = w;
            if (wstar < 0 && s_sum[w] > 0.0 && c + s_sum[w] > target) { wstar = w; before = c; }
            if (wstar < 0) c += s_sum[w];
        }
        if (wstar < 0) { wstar = wlast; before = c - (wlast >= 0 ? s_sum[wlast] : 0.0); }
    }
    if (wstar < 0) {                                        // no wave has a positive sum (logits that are not numbers):
        if (threadIdx.x == 0) next[row] = min(max(best, 0), V - 1);   // the same in-range answer the segmented kernels give
        return;
    }
    if (wave != wstar) return;                              // whole waves leave; no barrier follows

    // 5. inside that wave: walk the iterations, then the four groups of the iteration, then the lanes
    int eq_seen = eq_before_wave, pick = -1, last_in_play = -1;
    double c = before;
    for (int j = 0; j < nit && pick < 0; j++) {
#pragma unroll
        for (int e = 0; e < 4; e++) {
            if (pick >= 0) break;
            const double p = weight(j, e, eq_seen);
            const unsigned long long has = __ballot(p > 0.0);
            if (!has) continue;
            last_in_play = seg0 + j * 256 + e * 64 + (63 - __clzll((long long)has));
            const double incl = wave_scan_incl(p, lane);
            const unsigned long long over = __ballot(p > 0.0 && c + incl > target);
            if (over) pick = seg0 + j * 256 + e * 64 + (__ffsll((long long)over) - 1);
            c += __shfl(incl, 63);
        }
    }
    if (lane == 0) next[row] = pick >= 0 ? pick : last_in_play;
}

// The same choice with a row spread over many workgroups, for the two cases that need no top-k selection (greedy;
// all tokens in play): segments of SAMPLE_SEG consecutive logits, one workgroup each.
//   k_sample_segmax   largest logit of every segment (lowest index first)
//   k_sample_segsum   every workgroup reduces those to the row's largest logit, then sums p over its segment
//   k_sample_pick     one wave per row: greedy answer, or the segment that holds the target and the walk through it
constexpr int SAMPLE_SEG = 4096;
struct SegStat {
    uint32_t key;
    int idx;
    double sum;
};

// (key, index) of the best of the workgroup's candidates, lowest index among equal keys; all threads get it
template <int NWV>
__device__ __forceinline__ void block_best(uint32_t &bk, int &bi, uint32_t *s_key, int *s_idx) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t k2 = (uint32_t)__shfl_xor((int)bk, off);
        const int i2 = __shfl_xor(bi, off);
        if (k2 > bk || (k2 == bk && i2 < bi)) { bk = k2; bi = i2; }
    }
    if (lane == 0) { s_key[wave] = bk; s_idx[wave] = bi; }
    __syncthreads();
    bk = s_key[0]; bi = s_idx[0];
#pragma unroll
    for (int w = 1; w < NWV; w++)
        if (s_key[w] > bk || (s_key[w] == bk && s_idx[w] < bi)) { bk = s_key[w]; bi = s_idx[w]; }
    __syncthreads();
}

__global__ void __launch_bounds__(256) k_sample_segmax(const float *__restrict__ logits, int V, SegStat *__restrict__ st) {
    __shared__ uint32_t s_key[4];
    __shared__ int s_idx[4];
    const int g = blockIdx.x, row = blockIdx.y, G = gridDim.x;
    const float *l = logits + (size_t)row * V;
    const int base = g * SAMPLE_SEG, end = min(V, base + SAMPLE_SEG);
    float f[SAMPLE_SEG / 256];
#pragma unroll
    for (int i = 0; i < SAMPLE_SEG / 256; i++) {
        const int v = base + i * 256 + threadIdx.x;
        f[i] = v < end ? l[v] : -INFINITY;
    }
    uint32_t bk = 0;
    int bi = 0x7fffffff;
#pragma unroll
    for (int i = 0; i < SAMPLE_SEG / 256; i++) {
        const int v = base + i * 256 + threadIdx.x;
        const uint32_t k = order_key(f[i]);
        if (v < end && k > bk) { bk = k; bi = v; }
    }
    block_best<4>(bk, bi, s_key, s_idx);
    if (threadIdx.x == 0) { st[(size_t)row * G + g].key = bk; st[(size_t)row * G + g].idx = bi; }
}

// the row's best (key, index) from the G segment results; all threads of the workgroup get it
template <int NWV>
__device__ __forceinline__ void row_best(const SegStat *__restrict__ st, int G, uint32_t &bk, int &bi, uint32_t *s_key,
                                         int *s_idx) {
    bk = 0;
    bi = 0x7fffffff;
    for (int i = threadIdx.x; i < G; i += 64 * NWV) {
        const uint32_t k = st[i].key;
        const int v = st[i].idx;
        if (k > bk || (k == bk && v < bi)) { bk = k; bi = v; }
    }
    block_best<NWV>(bk, bi, s_key, s_idx);
}

__global__ void __launch_bounds__(256) k_sample_segsum(const float *__restrict__ logits, int V, float temperature,
                                                        SegStat *__restrict__ st) {
    __shared__ uint32_t s_key[4];
    __shared__ int s_idx[4];
    __shared__ double s_sum[4];
    const int g = blockIdx.x, row = blockIdx.y, G = gridDim.x;
    const float *l = logits + (size_t)row * V;
    uint32_t bk;
    int bi;
    row_best<4>(st + (size_t)row * G, G, bk, bi, s_key, s_idx);
    bi = min(bi, V - 1);                                     // stays in bounds whatever the logits hold
    const double lm = (double)l[bi], Td = (double)temperature;
    const int base = g * SAMPLE_SEG, end = min(V, base + SAMPLE_SEG);
    double sum = 0.0;
#pragma unroll
    for (int i = 0; i < SAMPLE_SEG / 256; i++) {
        const int v = base + i * 256 + threadIdx.x;
        if (v < end) sum += exp(((double)l[v] - lm) / Td);
    }
    sum = wave_sum(sum);
    if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) st[(size_t)row * G + g].sum = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
}

__global__ void __launch_bounds__(64) k_sample_pick(const float *__restrict__ logits, int V, float temperature, int G,
                                                    const SegStat *__restrict__ st_all, const float *__restrict__ uni,
                                                    int32_t *__restrict__ next) {
    __shared__ uint32_t s_key[1];
    __shared__ int s_idx[1];
    const int row = blockIdx.x, lane = threadIdx.x;
    const float *l = logits + (size_t)row * V;
    const SegStat *st = st_all + (size_t)row * G;
    uint32_t bk;
    int bi;
    row_best<1>(st, G, bk, bi, s_key, s_idx);
    bi = min(bi, V - 1);                                     // stays in bounds whatever the logits hold
    if (temperature == 0.0f) {
        if (lane == 0) next[row] = bi;
        return;
    }
    // running sum over the segments in order, 64 at a time
    double total = 0.0;
    for (int g0 = 0; g0 < G; g0 += 64) {
        const double v = g0 + lane < G ? st[g0 + lane].sum : 0.0;
        total += __shfl(wave_scan_incl(v, lane), 63);
    }
    const double target = (double)uni[row] * total;
    int gstar = -1, glast = -1;
    double before = 0.0, c = 0.0;
    for (int g0 = 0; g0 < G && gstar < 0; g0 += 64) {
        const double v = g0 + lane < G ? st[g0 + lane].sum : 0.0;
        const double incl = wave_scan_incl(v, lane);
        const unsigned long long has = __ballot(v > 0.0);
        if (has) glast = g0 + 63 - __clzll((long long)has);
        const unsigned long long over = __ballot(v > 0.0 && c + incl > target);
        if (over) {
            const int k = __ffsll((long long)over) - 1;
            gstar = g0 + k;
            before = c + __shfl(incl - v, k);
        }
        c += __shfl(incl, 63);
    }
    if (gstar < 0) {                                        // rounding left no segment above the target: the last one
        if (glast < 0) glast = G - 1;                       // (no positive sum at all: logits that are not numbers)
        gstar = glast;
        before = total - st[glast].sum;
    }
    // walk the segment in index order: 16 iterations of 4 groups of 64 consecutive logits
    const double lm = (double)l[bi], Td = (double)temperature;
    const int base = gstar * SAMPLE_SEG, end = min(V, base + SAMPLE_SEG);
    int pick = -1;
    c = before;
    for (int v0 = base; v0 < end && pick < 0; v0 += 64) {
        const int v = v0 + lane;
        const double p = v < end ? exp(((double)l[v] - lm) / Td) : 0.0;
        const double incl = wave_scan_incl(p, lane);
        const unsigned long long over = __ballot(v < end && c + incl > target);
        if (over) pick = v0 + __ffsll((long long)over) - 1;
        c += __shfl(incl, 63);
    }
    if (lane == 0) next[row] = pick >= 0 ? pick : end - 1;
}

// Top-k sampling with k <= SAMPLE_KMAX, a row again spread over segments: the k largest of the row are among the
// k largest of every segment, so k_sample_segtop writes each segment's k largest (in index order) and
// k_sample_pick_topk, one workgroup per row, selects among those few thousand candidates.
constexpr int SAMPLE_KMAX = 64;
struct Cand {
    uint32_t key;
    int idx;
};

// 256 threads hold NPT keys each, in the order (i, wave, lane).  Marks the k largest (equal keys: earlier first) in
// take (bit i) and gives each marked key its position among the marked, in that order.  LDS: hist[256], grp[64],
// two words sh.  Every thread of the workgroup must call it; k >= 1 and at most the number of valid keys.
template <int NPT>
__device__ __forceinline__ void block_topk_ordered(const uint32_t (&key)[NPT], uint32_t valid, int k, int *hist, int *grp,
                                                   uint32_t *sh, uint32_t &take, int (&pos)[NPT]) {
    static_assert(NPT <= 16, "64 (i, wave) groups are scanned by one wave");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned long long lt = (1ull << lane) - 1ull;
    uint32_t prefix = 0;
    int remaining = k;
    for (int pass = 3; pass >= 0; pass--) {
        hist[tid] = 0;
        __syncthreads();
        const int shift = pass * 8;
#pragma unroll
        for (int i = 0; i < NPT; i++) {
            const bool in = ((valid >> i) & 1u) && (pass == 3 || (key[i] >> (shift + 8)) == prefix);
            const uint32_t bin = (key[i] >> shift) & 255u;
            // (the high bytes of logits crowd a few bins: 64 lanes on one LDS word still take fewer clocks than finding
            // out by ballots which lanes share a bin)
            if (in) atomicAdd(&hist[bin], 1);
        }
        __syncthreads();
        if (wave == 0) {
            uint32_t b;
            int n;
            radix_pick_bin(hist, remaining, lane, b, n);
            if (lane == 0) { sh[0] = (prefix << 8) | b; sh[1] = (uint32_t)n; }
        }
        __syncthreads();
        prefix = sh[0];
        remaining = (int)sh[1];
        __syncthreads();
    }
    const uint32_t thr = prefix;
    const int need = remaining;
    // ordered rank of the keys equal to thr, then ordered position of the marked keys: per (i, wave) group a
    // count, an exclusive scan of the 4 NPT counts by the first wave, and the lanes below within the group
    auto ordered = [&](auto flag, int (&out)[NPT]) {
#pragma unroll
        for (int i = 0; i < NPT; i++) {
            const unsigned long long m = __ballot(flag(i));
            if (lane == 0) grp[i * 4 + wave] = __popcll(m);
            out[i] = __popcll(m & lt);
        }
        __syncthreads();
        if (wave == 0) {
            const int c = lane < NPT * 4 ? grp[lane] : 0;
            int inc = c;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int o = __shfl_up(inc, off);
                if (lane >= off) inc += o;
            }
            if (lane < NPT * 4) grp[lane] = inc - c;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NPT; i++) out[i] += grp[i * 4 + wave];
        __syncthreads();
    };
    int rank[NPT];
    ordered([&](int i) { return ((valid >> i) & 1u) && key[i] == thr; }, rank);
    take = 0;
#pragma unroll
    for (int i = 0; i < NPT; i++)
        if (((valid >> i) & 1u) && (key[i] > thr || (key[i] == thr && rank[i] < need))) take |= 1u << i;
    ordered([&](int i) { return (take >> i) & 1u; }, pos);
}

__global__ void __launch_bounds__(256) k_sample_segtop(const float *__restrict__ logits, int V, int top_k,
                                                       Cand *__restrict__ cand) {
    constexpr int NPT = SAMPLE_SEG / 256;
    __shared__ int hist[256], grp[64];
    __shared__ uint32_t sh[2];
    const int g = blockIdx.x, row = blockIdx.y, G = gridDim.x;
    const float *l = logits + (size_t)row * V;
    const int base = g * SAMPLE_SEG, end = min(V, base + SAMPLE_SEG);
    uint32_t key[NPT], valid = 0;
#pragma unroll
    for (int i = 0; i < NPT; i++) {
        const int v = base + i * 256 + threadIdx.x;
        key[i] = 0;
        if (v < end) { key[i] = order_key(l[v]); valid |= 1u << i; }
    }
    uint32_t take;
    int pos[NPT];
    block_topk_ordered<NPT>(key, valid, min(top_k, end - base), hist, grp, sh, take, pos);
    Cand *out = cand + ((size_t)row * G + g) * SAMPLE_KMAX;
#pragma unroll
    for (int i = 0; i < NPT; i++)
        if ((take >> i) & 1u) out[pos[i]] = Cand{key[i], base + i * 256 + (int)threadIdx.x};
}

__global__ void __launch_bounds__(256) k_sample_pick_topk(const float *__restrict__ logits, int V, float temperature,
                                                          int top_k, int G, const Cand *__restrict__ cand_all,
                                                          const float *__restrict__ uni, int32_t *__restrict__ next) {
    constexpr int NPT = 16;                                  // 4096 candidates at most: 64 segments x 64
    __shared__ int hist[256], grp[64], play_idx[SAMPLE_KMAX];
    __shared__ uint32_t sh[2], s_key[4];
    __shared__ int s_idx[4];
    const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const float *l = logits + (size_t)row * V;
    const Cand *cand = cand_all + (size_t)row * G * SAMPLE_KMAX;
    // candidate j = (segment, position): every segment gave min(top_k, its size); only the last can be short
    const int per = min(top_k, SAMPLE_SEG), n_last = min(top_k, V - (G - 1) * SAMPLE_SEG), Nc = (G - 1) * per + n_last;
    uint32_t key[NPT], valid = 0;
    int idx[NPT];
    uint32_t bk = 0;
    int bi = 0x7fffffff;
#pragma unroll
    for (int i = 0; i < NPT; i++) {
        const int j = i * 256 + tid;
        key[i] = 0;
        idx[i] = 0;
        if (j < Nc) {
            const int g = min(j / per, G - 1);
            const Cand c = cand[(size_t)g * SAMPLE_KMAX + (j - g * per)];
            key[i] = c.key;
            idx[i] = c.idx;
            valid |= 1u << i;
            if (c.key > bk) { bk = c.key; bi = c.idx; }      // a thread meets its candidates in index order
        }
    }
    block_best<4>(bk, bi, s_key, s_idx);
    bi = min(bi, V - 1);                                     // stays in bounds whatever the logits hold
    uint32_t take;
    int pos[NPT];
    block_topk_ordered<NPT>(key, valid, top_k, hist, grp, sh, take, pos);
#pragma unroll
    for (int i = 0; i < NPT; i++)
        if ((take >> i) & 1u) play_idx[pos[i]] = idx[i];
    __syncthreads();
    if (tid >= 64) return;
    // the top_k tokens in play, in index order, one per lane
    const int v = lane < top_k ? play_idx[lane] : 0;
    const double p = lane < top_k ? exp(((double)l[v] - (double)l[bi]) / (double)temperature) : 0.0;
    const double incl = wave_scan_incl(p, lane);
    const double target = (double)uni[row] * __shfl(incl, 63);
    const unsigned long long over = __ballot(lane < top_k && incl > target);
    const int which = over ? __ffsll((long long)over) - 1 : top_k - 1;
    if (lane == 0) next[row] = play_idx[which];
}

}  // namespace

struct petals_client {
    petals_client_config cfg;
    petals_client_params p;
    __half *a;          // LayerNorm output of the rows of one lm_head call
    Best *partial;      // [LM_MAX_ROWS][LM_GROUPS]
    uint8_t *dig, *dig2;   // digit planes of up to LM_MAX_ROWS hidden rows: [H / 64][4 and 2][row tiles][1024]
    LmRow *info;           // [LM_MAX_ROWS]
    SegStat *seg;       // [max_rows_per_call][segments of the vocabulary]: per-segment results of the sampler
    Cand *cand;         // [max_rows_per_call][segments][SAMPLE_KMAX]: per-segment candidates of top-k sampling
};

namespace {
int check_client_config(const petals_client_config *c) {
    if (!c) return ps_fail(PETALS_ERR_INVALID_ARG, "config is null");
    if (c->vocab < 1 || c->hidden < 1 || c->max_rows_per_call < 1)
        return ps_fail(PETALS_ERR_INVALID_ARG, "config fields must be positive");
    if (c->hidden % 64 || c->hidden > LM_MAX_HIDDEN) return ps_fail(PETALS_ERR_UNSUPPORTED, "hidden must be a multiple of 64, at most 16384");
    if (!(c->ln_eps > 0.0f)) return ps_fail(PETALS_ERR_INVALID_ARG, "ln_eps must be positive");
    return PETALS_OK;
}
}  // namespace

extern "C" {

int petals_client_workspace_bytes(const petals_client_config *cfg, size_t *bytes) {
    if (!bytes) return ps_fail(PETALS_ERR_INVALID_ARG, "null pointer");
    if (int rc = check_client_config(cfg)) return rc;
    *bytes = align_up((size_t)cfg->max_rows_per_call * cfg->hidden * 2) + align_up(sizeof(Best) * LM_MAX_ROWS * LM_GROUPS) +
             align_up((size_t)6 * LM_MAX_ROWS * cfg->hidden) + align_up(sizeof(LmRow) * LM_MAX_ROWS) +
             align_up(sizeof(SegStat) * (size_t)cfg->max_rows_per_call * ((cfg->vocab + SAMPLE_SEG - 1) / SAMPLE_SEG)) +
             align_up(sizeof(Cand) * SAMPLE_KMAX * (size_t)cfg->max_rows_per_call * ((cfg->vocab + SAMPLE_SEG - 1) / SAMPLE_SEG));
    return PETALS_OK;
}

int petals_client_create(const petals_client_config *cfg, const petals_client_params *params, void *dev_workspace,
                         petals_client **out) {
    if (!params || !dev_workspace || !out) return ps_fail(PETALS_ERR_INVALID_ARG, "null pointer");
    if (int rc = check_client_config(cfg)) return rc;
    if (!params->embeddings || !params->emb_ln_g || !params->emb_ln_b || !params->final_ln_g || !params->final_ln_b)
        return ps_fail(PETALS_ERR_INVALID_ARG, "a parameter pointer is null");
    if ((uintptr_t)dev_workspace & 255) return ps_fail(PETALS_ERR_INVALID_ARG, "workspace must be 256-byte aligned");
    if ((uintptr_t)params->embeddings & 15) return ps_fail(PETALS_ERR_INVALID_ARG, "embeddings must be 16-byte aligned");
    petals_client *c = new (std::nothrow) petals_client;
    if (!c) return ps_fail(PETALS_ERR_INVALID_ARG, "out of host memory");
    c->cfg = *cfg;
    c->p = *params;
    c->a = (__half *)dev_workspace;
    c->partial = (Best *)((uint8_t *)dev_workspace + align_up((size_t)cfg->max_rows_per_call * cfg->hidden * 2));
    c->dig = (uint8_t *)c->partial + align_up(sizeof(Best) * LM_MAX_ROWS * LM_GROUPS);
    c->dig2 = c->dig + (size_t)4 * LM_MAX_ROWS * cfg->hidden;
    c->info = (LmRow *)(c->dig + align_up((size_t)6 * LM_MAX_ROWS * cfg->hidden));
    c->seg = (SegStat *)((uint8_t *)c->info + align_up(sizeof(LmRow) * LM_MAX_ROWS));
    c->cand = (Cand *)((uint8_t *)c->seg + align_up(sizeof(SegStat) * (size_t)cfg->max_rows_per_call *
                                                     ((cfg->vocab + SAMPLE_SEG - 1) / SAMPLE_SEG)));
    *out = c;
    return PETALS_OK;
}

int petals_client_destroy(petals_client *client) {
    if (!client) return ps_fail(PETALS_ERR_INVALID_ARG, "null pointer");
    delete client;
    return PETALS_OK;
}

int petals_client_embed(petals_client *c, const int32_t *token_ids, int32_t M, void *hidden_out, void *stream) {
    if (!c || !token_ids || !hidden_out) return ps_fail(PETALS_ERR_INVALID_ARG, "null pointer");
    if (M < 1) return ps_fail(PETALS_ERR_INVALID_ARG, "M must be positive");
    if (M > c->cfg.max_rows_per_call) return ps_fail(PETALS_ERR_CAPACITY, "%d rows exceed max_rows_per_call %d", M, c->cfg.max_rows_per_call);
    hipStream_t st = (hipStream_t)stream;
    const __half *E = (const __half *)c->p.embeddings;
    if (c->cfg.hidden >= 4096)
        k_embed_ln<1024><<<M, 1024, 0, st>>>(token_ids, E, c->cfg.vocab, c->cfg.hidden, (const __half *)c->p.emb_ln_g,
                                             (const __half *)c->p.emb_ln_b, c->cfg.ln_eps, (__half *)hidden_out);
    else
        k_embed_ln<256><<<M, 256, 0, st>>>(token_ids, E, c->cfg.vocab, c->cfg.hidden, (const __half *)c->p.emb_ln_g,
                                           (const __half *)c->p.emb_ln_b, c->cfg.ln_eps, (__half *)hidden_out);
    HIP_TRY(hipGetLastError());
    return PETALS_OK;
}

int petals_client_lm_head(petals_client *c, const void *hidden_in, int32_t M, float *logits_out, int32_t *next_token_out,
                          void *stream) {
    if (!c || !hidden_in) return ps_fail(PETALS_ERR_INVALID_ARG, "null pointer");
    if (!logits_out && !next_token_out) return ps_fail(PETALS_ERR_INVALID_ARG, "neither logits nor next tokens requested");
    if (M < 1) return ps_fail(PETALS_ERR_INVALID_ARG, "M must be positive");
    if (M > c->cfg.max_rows_per_call) return ps_fail(PETALS_ERR_CAPACITY, "%d rows exceed max_rows_per_call %d", M, c->cfg.max_rows_per_call);
    hipStream_t st = (hipStream_t)stream;
    const int H = c->cfg.hidden, V = c->cfg.vocab;
    const __half *E = (const __half *)c->p.embeddings, *x = (const __half *)hidden_in;
    const __half *lng = (const __half *)c->p.final_ln_g, *lnb = (const __half *)c->p.final_ln_b;
    if (M == 1) {
        // one row: the matrix streams at 6.6 TB/s past one fp64 multiply-add per value
        HIP_TRY(ps_layernorm(x, lng, lnb, c->cfg.ln_eps, 1, H, c->a, nullptr, 0.0f, st));
        const size_t lds = (size_t)H * 8;
        {   // the limit belongs to the function, for all clients of the process: set once, to the widest row there is
            static std::mutex attr_lock;
            static bool attr_set = false;
            std::lock_guard<std::mutex> hold(attr_lock);
            if (!attr_set) {
                HIP_TRY(hipFuncSetAttribute((const void *)k_lm_head, hipFuncAttributeMaxDynamicSharedMemorySize, LM_MAX_HIDDEN * 8));
                attr_set = true;
            }
        }
        const int groups = min(LM_GROUPS, (V + LM_WAVES - 1) / LM_WAVES);
        k_lm_head<<<groups, LM_THREADS, lds, st>>>(c->a, E, V, H, logits_out, c->partial);
        HIP_TRY(hipGetLastError());
        if (next_token_out) {
            k_lm_pick<<<1, 64, 0, st>>>(c->partial, groups, next_token_out);
            HIP_TRY(hipGetLastError());
        }
        return PETALS_OK;
    }
    const int ntiles = (V + 15) / 16;
    for (int m0 = 0; m0 < M; m0 += LM_MAX_ROWS) {
        const int rows = min(LM_MAX_ROWS, M - m0), mt = rows > 16 ? 2 : 1;
        const __half *xr = x + (size_t)m0 * H;
        __half *a = c->a + (size_t)m0 * H;
        float *lg = logits_out ? logits_out + (size_t)m0 * V : nullptr;
        // up to 16 rows: two matrix tiles per wave (the digits read from LDS then serve both) once that leaves every
        // compute unit a workgroup of 8 waves; with 17 to 32 rows two tiles need more registers than there are
        const int wn = mt == 1 && ntiles >= 256 * 16 ? 2 : 1, groups = min(LM_GROUPS, (ntiles + 8 * wn - 1) / (8 * wn));
        if (H <= 4096) k_lm_prepare<1><<<16 * mt, 512, 0, st>>>(xr, lng, lnb, c->cfg.ln_eps, rows, H, mt, a, c->dig, c->dig2, c->info);
        else k_lm_prepare<4><<<16 * mt, 512, 0, st>>>(xr, lng, lnb, c->cfg.ln_eps, rows, H, mt, a, c->dig, c->dig2, c->info);
        HIP_TRY(hipGetLastError());
        hipError_t e = wn == 2   ? lm_head_digits<2, 1>(groups, a, c->dig, c->dig2, c->info, rows, E, V, H, lg, c->partial, st)
                       : mt == 2 ? lm_head_digits<1, 2>(groups, a, c->dig, c->dig2, c->info, rows, E, V, H, lg, c->partial, st)
                                 : lm_head_digits<1, 1>(groups, a, c->dig, c->dig2, c->info, rows, E, V, H, lg, c->partial, st);
        HIP_TRY(e);
        if (next_token_out) {
            k_lm_pick<<<rows, 64, 0, st>>>(c->partial, groups, next_token_out + m0);
            HIP_TRY(hipGetLastError());
        }
    }
    return PETALS_OK;
}

int petals_client_sample(petals_client *c, const float *logits, int32_t M, float temperature, int32_t top_k,
                         const float *uniforms, int32_t *next_token_out, void *stream) {
    if (!c || !logits || !uniforms || !next_token_out) return ps_fail(PETALS_ERR_INVALID_ARG, "null pointer");
    if (M < 1) return ps_fail(PETALS_ERR_INVALID_ARG, "M must be positive");
    if (!(temperature >= 0.0f)) return ps_fail(PETALS_ERR_INVALID_ARG, "temperature must be zero (greedy) or positive");
    hipStream_t st = (hipStream_t)stream;
    const int V = c->cfg.vocab, G = (V + SAMPLE_SEG - 1) / SAMPLE_SEG;
    const bool greedy = temperature == 0.0f || top_k == 1, all = top_k <= 0 || top_k >= V;
    if ((greedy || all) && M <= c->cfg.max_rows_per_call && M <= 65535) {
        // no top-k selection: the row is spread over G workgroups (per-segment results in the workspace)
        k_sample_segmax<<<dim3(G, M), 256, 0, st>>>(logits, V, c->seg);
        if (!greedy) k_sample_segsum<<<dim3(G, M), 256, 0, st>>>(logits, V, temperature, c->seg);
        k_sample_pick<<<M, 64, 0, st>>>(logits, V, greedy ? 0.0f : temperature, G, c->seg, uniforms, next_token_out);
    } else if (top_k <= SAMPLE_KMAX && G <= 64 && M <= c->cfg.max_rows_per_call && M <= 65535) {
        // a small k: every segment hands in its k largest, one workgroup per row selects among those
        k_sample_segtop<<<dim3(G, M), 256, 0, st>>>(logits, V, top_k, c->cand);
        k_sample_pick_topk<<<M, 256, 0, st>>>(logits, V, temperature, top_k, G, c->cand, uniforms, next_token_out);
    } else {
        k_sample<<<M, 1024, 0, st>>>(logits, V, temperature, top_k, uniforms, next_token_out);
    }
    HIP_TRY(hipGetLastError());
    return PETALS_OK;
}

}  // extern "C"

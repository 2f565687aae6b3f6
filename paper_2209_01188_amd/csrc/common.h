// Shared declarations of the span library's kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <type_traits>
#include <utility>

#include "f64math.h"

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
// eight halves at any address (callers' tensors carry no alignment promise; the hardware loads them in one piece)
typedef _Float16 v8h_any __attribute__((ext_vector_type(8), aligned(2)));
typedef double v4d __attribute__((ext_vector_type(4)));

#define PS_MAX_SESSIONS 64
#define PS_MAX_HEADS 256

// int8 weights of one linear in streaming tile order: tiles of 16 output rows x 64
// input columns, 1024 bytes each; tile (nt, kt) starts at ((nt * K/64) + kt) * 1024;
// inside a tile lane l (0..63) owns bytes [16 l, 16 l + 16): row nt*16 + l%16,
// columns kt*64 + (l/16)*16 + 0..15.  This is exactly the per-lane operand of
// v_mfma_i32_16x16x64_i8, and a wave reads one tile as 1 KB of consecutive bytes.
struct LinearW {
    const int8_t *wt;
    const float *sw;      // [N] row scales (row absmax)
    const __half *bias;   // [N]
    int N, K;
};

// Per-call table in device memory: key/value memory of the sessions of the call and
// the ALiBi slopes.  len[s]: tokens cached BEFORE this call.
struct SessTable {
    __half *kv[PS_MAX_SESSIONS];   // session base: [block][key|value][head][cap][d]
    int len[PS_MAX_SESSIONS];
    int cap[PS_MAX_SESSIONS];
    double slopes[PS_MAX_HEADS];   // ALiBi slope per head
};

// Where a linear's result goes and what is fused before the fp16 rounding.
struct OutDesc {
    int scatter;          // 0: y is [M,N] row-major; 1: fused-QKV scatter (q -> y [M,H], k/v -> caches)
    __half *y;
    int epilogue;         // 0 none, 1 tanh-GeLU, 2 + resid
    const __half *resid;  // [M,N]
    int32_t *acc_out;     // optional int32 [M,N] copy of the integer accumulators
    int T, nh, d, blk;    // scatter: row t belongs to session t / T at position len + t % T of block blk
    int t0;               // scatter: the launch's row 0 is row t0 of the call (a call may be split over launches)
    uint32_t *next_mask;  // optional (scatter == 0): outlier-column bit mask [N/32] of the linear that reads y
    float next_theta;     // a column of y is flagged when any |y| >= next_theta
    __half *pre_out;      // optional (scatter == 0): [M,N] copy of the sum BEFORE the fused GeLU / residual
};

struct CodeTable { float code[256]; };
// The 256 entries of the 8-bit dynamic data type of the hidden-state codec, ascending: per decade 10^-e
// (e = 0..6) the centres of 2^(6-e) equal buckets spanning [0.1, 1.0], both signs, plus 0 and 1.0.
// constexpr: host code and device-side constant tables are built from the same evaluation.
constexpr CodeTable ps_make_code_table() {
    CodeTable tab{};
    const double decade[7] = {1.0, 1e-1, 1e-2, 1e-3, 1e-4, 1e-5, 1e-6};
    float pos[127] = {};
    int n = 0;
    for (int e = 6; e >= 0; e--) {          // ascending: decades from small to large, buckets ascending inside a decade
        const int cnt = 64 >> e;
        for (int j = 0; j < cnt; j++) pos[n++] = (float)(decade[e] * (0.1 + 0.9 * (j + 0.5) / cnt));
    }
    int k = 0;
    for (int i = n - 1; i >= 0; i--) tab.code[k++] = -pos[i];
    tab.code[k++] = 0.0f;
    for (int i = 0; i < n; i++) tab.code[k++] = pos[i];
    tab.code[k++] = 1.0f;
    return tab;
}

// Hidden states that arrive as blockwise 8-bit codes and are decoded by the first LayerNorm of a call:
// value i = fp16(table[q[i]] * absmax[i / block]) over the flat [M, H] buffer.  x_out receives the decoded
// fp16 rows (the first block's residual reads them).
struct QuantIn {
    const uint8_t *q;
    const float *absmax;
    int block;
    __half *x_out;
};

// Up to so many outlier columns the fp16 part of a linear in output blocks goes through fp64 matrix instructions on compacted
// operands, beyond that through the digit products, which cost the same for 53 columns as for 200.  Calls of up to 1024 rows are few
// blocks, whose units do the fp64 products alone (192 rows of 9216 x 3072: 43 us without, 62 with 40, 73 with 64 columns, 61 in
// digits; 72 rows of 19968 x 6656: 57, 80, 92, 83; 256 rows 72, 103, 123, 111).  Where a unit has no more than 16 of the 16 x 16 tiles
// fp64 stays ahead (352 rows of 2560 x 2560, 64 columns 41 against 52), and so it does in larger calls, which would write and read
// more fp64 sums than that saves (1400 rows of 16384 x 4096: 237 against 281, 4096 rows 520 against 755).
#define PS_EXACT_OUTLIERS 64
#define PS_OUTLIER_CHUNKS (PS_EXACT_OUTLIERS / 4)
__host__ __device__ inline int ps_exact_outliers(int N, int M) { return M <= 1024 && (N / 16) * ((M + 15) / 16) > 3600 ? 52 : PS_EXACT_OUTLIERS; }
// Compacted outlier operands of one linear call, in v_mfma_f64_16x16x4_f64 lane order:
// chunk c of tile r holds 64 doubles, lane l = column list[4c + l/16] of row 16r + l%16
// (weight rows permuted inside a tile, see outlier_prep_wave).
struct OutlierSet {
    const int *count;       // [0] number of outlier columns of this call, [1] digit planes its activations need
    const double *wd64;     // [N/16][PS_OUTLIER_CHUNKS][64] dequantized fp16 weights
    const double *x64;      // [ceil(M/16)][PS_OUTLIER_CHUNKS][64] fp16 activations
};

// --- launchers (all enqueue on `st` and return the launch status) ---------------
hipError_t ps_quantize_weight(const float *W, int N, int K, int8_t *wt, float *sw, hipStream_t st);
hipError_t ps_untile_weight(const int8_t *wt, int N, int K, int8_t *wq_rowmajor, hipStream_t st);
hipError_t ps_fill_u32(uint32_t *p, size_t n, uint32_t v, hipStream_t st);
hipError_t ps_copy_bytes(const void *src, void *dst, size_t n, hipStream_t st);
// flags (null, or zeroed): one byte per column, set to 1 where a row reaches theta
hipError_t ps_layernorm(const __half *x, const __half *g, const __half *b, float eps, int M, int H,
                        __half *y, uint8_t *flags, float theta, hipStream_t st);
// LayerNorm of rows that arrive as 8-bit codes (also writes the decoded rows to qin.x_out)
hipError_t ps_layernorm_q8(const QuantIn &qin, const __half *g, const __half *b, float eps, int M,
                           int H, __half *y, uint8_t *flags, float theta, hipStream_t st);
hipError_t ps_colmask(const __half *X, int M, int K, float theta, uint32_t *mask, hipStream_t st);
// M rows -> tiled int8 codes (rows padded to 16 with zeros), row scales; mask given, or (flags not null) given as one byte
// per column and then written to mask
// xo_tiled (may be null): same tile order, 16 bytes per (token, 16-column group) = the fp16 values of the
// group's first 8 outlier columns in ascending order; groups without outliers are not written
// pr (pr.count may be null): the linear's outlier columns are counted and, if they are few, compacted in the same launch
// rd (rd.xd may be null): if the call has many outlier columns, their digits for ps_gemm, and what became of each row
struct OutlierPrep;
struct RowDigits {
    int8_t *xd;          // [ceil(M/16)][K/64][4 digits][1024], tiles in the order of xq_tiled
    int *rowstate;       // [M]
    int *done;           // [PS_DIGIT_DONE], cleared
};
#define PS_ROWS_IN_DIGITS 1       // the row's digits are written; a call is taken as digits if all its rows say so
hipError_t ps_rowquant_tiled(const __half *X, int M, int K, uint32_t *mask, const uint8_t *flags, int8_t *xq_tiled,
                             int8_t *xo_tiled, float *sx, int8_t *xq_rowmajor_dbg, const OutlierPrep &pr, const RowDigits &rd,
                             hipStream_t st);
// LayerNorm and row quantizer of a call of 2 to PS_NORM_ROWS_MAX rows in one launch (quant.hip): y, the mask (whose bits need not
// be cleared) and all that ps_rowquant_tiled writes.  qin (may be null): the rows arrive as 8-bit codes, x is ignored
#define PS_NORM_ROWS_MAX 128
#define PS_NORM_RECORD_WORDS 16   // 32-bit words of a row's record
struct NormExchange {
    uint64_t *records;           // [PS_NORM_ROWS_MAX] records, no word of which holds the tag
    uint32_t *masks;             // [PS_NORM_ROWS_MAX][H / 32]
    uint32_t tag;                // 1 to 65535
    uint32_t patience;           // ticks of the 100 MHz clock that a row waits for the others; 0: it does without them
};
hipError_t ps_layernorm_codes(const __half *x, const QuantIn *qin, const __half *g, const __half *b, float eps, int M, int H, __half *y,
                              uint32_t *mask, int8_t *xq_tiled, int8_t *xo_tiled, float *sx, int8_t *xq_dbg, float theta,
                              const NormExchange &ex, hipStream_t st);
hipError_t ps_mask_to_bytes(const uint32_t *mask, int K, uint8_t *out, hipStream_t st);
hipError_t ps_mask_count(const uint32_t *masks, int n_masks, int words, int32_t *out, hipStream_t st);

// Scratch of the outlier-heavy case of a prefill-size call (more than ps_exact_outliers columns): the fp16
// product over the outlier columns is taken exactly, as int8 digit products (see gemm_lds.hip)
#define PS_X_DIGITS 6            // balanced 8-bit digits of an fp16 activation in units of 2^-24 (4 cover |x| < 127.5)
struct ManyOutliers {
    int *list;      // [K] outlier column indices, ascending, padded with -1 to a multiple of 64
    int *regular;   // [K] the other columns, likewise, where ps_regular_compacted
    int8_t *xl;     // digit tiles of the activations [PS_X_DIGITS][ceil(M/16)][ceil(n_out/64)][1024], behind them the codes
    int8_t *wd;     // digit tiles of the dequantized weights [2][N/16][ceil(n_out/64)][1024] of the regular columns (rows, weights)
    double *od;     // [M, N] the outlier product
    size_t wd_bytes;   // room at wd: once the digit products are done it holds the partial sums of a split contraction
};
// Where many columns are outliers, the codes of the other ones are gathered beside the digits and the int8 product walks only
// these (its codes of outlier columns are zero).  Gathering a column costs what multiplying some 2000 rows takes: 2048 rows
// with half of the columns -1 to +2 %, with seven in ten -4 % (8192 wide), with nine in ten -7 %; 1024 rows with seven in ten
// -2 to -4 %; 4096 rows of a 14336-wide block with 84 and 61 % 1.05 times as fast altogether.
__host__ __device__ inline bool ps_regular_compacted(int n_out, int K, int M) {
    return n_out > PS_EXACT_OUTLIERS && n_out < K && (long long)n_out * M >= (long long)(K - n_out) * 2000;
}
// LDS-staged linear for M > 64 rows (any number of outlier columns)
hipError_t ps_gemm_lds(const LinearW &w, const int8_t *xq_tiled, const uint32_t *mask, const __half *X, const float *sx,
                       int M, const OutlierSet &os, const ManyOutliers &mo, const OutDesc &o, const SessTable *sess,
                       hipStream_t st);
// optional copies of the one-row path's intermediates for tests (each may be null)
struct RowDebug {
    __half *a_out;       // LayerNorm output [K]
    int8_t *xq_out;      // int8 codes [K]
    uint32_t *mask_out;  // outlier bit mask [K/32]
    float *sx_out;       // row scale
};
// y = mixed int8/fp16 linear of ONE fp16 row x[K] (decode, batch 1); with ln_g/ln_b non-null the row
// first goes through LayerNorm.  Outlier detection and int8 quantization happen inside the kernel.
// qin (may be null; needs ln_g): the row arrives as 8-bit codes, x is ignored
hipError_t ps_gemv_row(const LinearW &w, const __half *x, const __half *ln_g, const __half *ln_b, float eps,
                       float theta, const RowDebug &dbg, const OutDesc &o, const SessTable *sess, const QuantIn *qin,
                       hipStream_t st);
// One token of one session through all blocks of a narrow span, one launch (decode_row.hip).  lin, ln*: block 0's; block b's lie
// b * stride bytes further.
struct StepArgs {
    LinearW lin[4];
    const __half *ln1g, *ln1b, *ln2g, *ln2b;
    size_t stride;
    int n_blocks, H, F, nh;
    float eps;
    uint32_t theta_bits;
    const __half *x;             // input row, or (q8 not null) its codes
    const uint8_t *q8;
    const float *q8_absmax;
    int q8_block;
    __half *out;
    const SessTable *sess;
    uint32_t *words;             // [PS_STEP_WORDS(H, F)], cleared before the launch: rows on their way, then ticket and done
    int *ticket;                 // next work item; [1] not zero: a reader has given up
    uint32_t patience;           // polls after which one does
    int *done;                   // [PS_MAX_HEADS] key ranges that have been summed up
    double *partials;
    int ranges;                  // of keys per head (this and what follows set by the launcher)
    double inv_h;                // 1 / H
};
#define PS_STEP_WORDS(H, F) ((size_t)6 * (H) + (F) + 64 + PS_MAX_HEADS)
bool ps_decode_row_applies(int H, int F, int d, int n_blocks);
hipError_t ps_decode_row(const StepArgs &s, int d, int max_keys, hipStream_t st);
hipError_t ps_steps_given_up(int *dev_count, hipStream_t st);     // on this device, since the library was loaded
#define PS_CHUNKED_ROWS_MAX 512
// batched-decode linear, 2 <= M <= PS_CHUNKED_ROWS_MAX rows, up to 64 per workgroup (int8 MFMA, outlier columns exactly on fp64 MFMA inside the
// loop); xq_tiled and xo_tiled as written by ps_rowquant_tiled
// dc (dc.xd may be null): for calls of 17 to 64 rows on wide matrices, whose outlier columns are then taken as digits if the row
// quantizer has written them for all rows, see gemm_digits.h.  (That is known on the device only: both forms are in one launch.)
struct DigitCall;
hipError_t ps_gemm(const LinearW &w, const int8_t *xq_tiled, const int8_t *xo_tiled, const uint32_t *mask,
                   const __half *X, const float *sx, int M, const OutDesc &o, const SessTable *sess, const DigitCall &dc,
                   hipStream_t st);
#define PS_DIGIT_SPLITS 4         // workgroups that share the contraction
#define PS_DIGIT_DONE 1024        // pieces of the output that they finish: 512 pairs of panels, for each half of the tokens
struct DigitCall {
    const int8_t *xd;             // RowDigits
    const int *rowstate;
    int *done;                    // [PS_DIGIT_DONE], cleared by the row quantizer: shares whose sums are in memory
    double *part;                 // [split][token half][pair of panels][16][64 lanes]: the outlier product in units of u_n 2^-24
    int *part_acc;                // the same of the regular columns' sums
};
bool ps_gemm_digits_applies(int N, int K, int M);
// Calls of more than 64 rows that are better served by ps_gemm, 32 or 64 rows per workgroup (the weights are streamed once
// per 32 or 64 rows, with every compute unit busy) than by the output blocks of ps_gemm_lds with their kernels for
// outlier columns.  PS_CHUNKED_ROWS_MAX bounds such calls.
bool ps_gemm_prefers_chunks(const LinearW &w, int M);
double ps_gemm_lds_us(int N, int K, int M);       // estimate of a linear of M > 64 rows in output blocks, with its row kernels

// attention of M = B*T query rows against the caches (new keys/values already appended)
// the call's table, and (n_masks, n_more > 0) its outlier masks and what else starts from zero cleared
hipError_t ps_call_setup(const SessTable &host_table, SessTable *dev_table, uint32_t *masks, size_t n_masks, uint32_t *more, size_t n_more, hipStream_t st);
#define PS_ATTN_MAX_SPLITS 16
#define PS_ATTN_PARTIAL_SLOTS 8192   // (row, head, split) triples that may need a partial result
// mask (may be null): outlier-column bits of ctx are ORed into it (|ctx| >= theta)
// lse, ctx32 (both null, or both given): for the backward pass, fp32 [nh][M] log of the softmax denominator of
// every (head, row) and fp32 [M, nh*d] context before its fp16 rounding
hipError_t ps_attention(const __half *q, const SessTable *sess, int blk, int M, int T, int nh, int d, int max_keys,
                        double *partials, __half *ctx, uint32_t *mask, float theta, float *lse, float *ctx32,
                        hipStream_t st);

// --- backward pass (gradients w.r.t. activations) ---
// fp16 [M,N] row-major -> 16 x 32 tiles in v_mfma_f32_16x16x32_f16 operand order, rows padded to 16 with zeros
hipError_t ps_tile_rows(const __half *X, int M, int N, __half *tiles, hipStream_t st);
// the linear's dequantized fp16 weights, transposed, in the same tile order: [K/16][N/32][512 halves]
hipError_t ps_transpose_w(const LinearW &w, __half *wt16, hipStream_t st);
// out[M, n_feat] (fp32) = token tiles [ceil(M/16)][ktiles] x feature tiles [n_feat/16][ktiles], contraction 32 * ktiles.
// With gelu_pre ([M, n_feat] fp16, n_feat % 32 == 0) the result is not stored as fp32: fp16(result * GeLU'(gelu_pre))
// goes to tile_out in token-tile order [ceil(M/16)][n_feat/32][512 halves], rows beyond M zero (out is unused).
hipError_t ps_gemm_f16_tiles(const __half *feat_tiles, const __half *tok_tiles, int ktiles, int M, int n_feat,
                             float *out, const __half *gelu_pre, __half *tile_out, hipStream_t st);
// tiles (may be null): the result again in token-tile order [ceil(M/16)][H/32][512 halves], rows beyond M zero
hipError_t ps_ln_bwd(const float *dz, const __half *x, const __half *g, const __half *dres, float eps, int M, int H,
                     __half *dx, __half *tiles, hipStream_t st);
hipError_t ps_attn_bwd_prep(const float *dctx, const float *ctx32, int M, int nh, int d, __half *dO, float *Dv,
                            hipStream_t st);
// QT, KT, dOT: scratch [B][nh][d][ceil(T/32)*32] halves each; dqkv [B*T, 3*nh*d] in the fused-QKV column order
hipError_t ps_attention_bwd(const __half *q, const SessTable *sess, int blk, int B, int T, int nh, int d, const __half *dO,
                            __half *QT, __half *KT, __half *dOT, const float *lse, const float *Dv, __half *dqkv,
                            hipStream_t st);

hipError_t ps_hidden_quantize(const __half *x, size_t n, int block, const CodeTable &tab, uint8_t *q, float *absmax,
                              hipStream_t st);
hipError_t ps_hidden_dequantize(const uint8_t *q, const float *absmax, size_t n, int block, const CodeTable &tab,
                                __half *y, hipStream_t st);
hipError_t ps_kv_export(const __half *kv, int nh, int cap, int d, int len, __half *out, hipStream_t st);
hipError_t ps_kv_import(__half *kv, int nh, int cap, int d, int len, const __half *in, hipStream_t st);

// --- small device helpers ---------------------------------------------------------
// Producer side of the outlier-column detection: ORs the bits of flagged columns into mask.
// Bits are only ever set between two clears, so a stale read of the word can at worst cause a
// redundant atomic.
__device__ __forceinline__ void flag_outlier_bits(uint32_t *mask, int word, uint32_t bits) {
    if (bits && (mask[word] & bits) != bits) atomicOr(&mask[word], bits);
}
__device__ __forceinline__ void flag_outlier(uint32_t *mask, float theta, int k, __half v) {
    if (mask && fabsf(__half2float(v)) >= theta) flag_outlier_bits(mask, k >> 5, 1u << (k & 31));
}
// The same for the LayerNorms of calls of more than 64 rows, with a byte per column: an outlier feature is one in every
// row, and the memory takes 7 ns per atomic on one address (351 rows of 4096 with four outlier columns: 10.1 us, 5.1
// with bytes).  Plain stores of a 1 need no order, meet in the XCD's own L2, and L2s write back only the bytes that were
// written.
__device__ __forceinline__ void flag_outlier_bytes(uint8_t *flags, int k, uint32_t bits) {
    while (bits) {
        flags[k + __ffs(bits) - 1] = 1;
        bits &= bits - 1;
    }
}
// 16 such bytes as bits
__device__ __forceinline__ uint32_t flag_bits16(const v4i &f) {
    const uint32_t lo = __builtin_amdgcn_udot4((uint32_t)f[1], 0x80402010u, __builtin_amdgcn_udot4((uint32_t)f[0], 0x08040201u, 0u, false), false);
    const uint32_t hi = __builtin_amdgcn_udot4((uint32_t)f[3], 0x80402010u, __builtin_amdgcn_udot4((uint32_t)f[2], 0x08040201u, 0u, false), false);
    return lo | hi << 8;
}
// the outlier bits of columns 16 c .. 16 c + 15, from flags if there are any
__device__ __forceinline__ uint32_t chunk_outliers(const uint32_t *mask, const uint8_t *flags, int c) {
    return flags ? flag_bits16(*(const v4i *)(flags + (size_t)c * 16)) : ((const uint16_t *)mask)[c];
}
// Wave-wide reductions on the data-parallel-primitive moves (a few clocks a step; an exchange through LDS takes some
// sixty, and a row kernel of a few microseconds waits for six of them in a row): four shifted steps inside the rows of
// 16 lanes, two row broadcasts, the result in lane 63.  All 64 lanes must be active.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_move(uint32_t old, uint32_t v) {     // lanes without a source keep `old`
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_move(float old, float v) {
    return __uint_as_float(dpp_move<CTRL, ROWS>(__float_as_uint(old), __float_as_uint(v)));
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_move(double old, double v) {
    const uint64_t o = (uint64_t)__double_as_longlong(old), u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = dpp_move<CTRL, ROWS>((uint32_t)o, (uint32_t)u), hi = dpp_move<CTRL, ROWS>((uint32_t)(o >> 32), (uint32_t)(u >> 32));
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}
__device__ __forceinline__ uint32_t lane63(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, 63); }
__device__ __forceinline__ float lane63(float v) { return __uint_as_float(lane63(__float_as_uint(v))); }
__device__ __forceinline__ double lane63(double v) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    return __longlong_as_double((long long)((uint64_t)lane63((uint32_t)(u >> 32)) << 32 | lane63((uint32_t)u)));
}
template <typename T, typename OP>
__device__ __forceinline__ T wave_reduce(T v, T none, OP op) {               // none: what a lane without a partner combines with
    v = op(v, dpp_move<0x111, 0xf>(none, v));     // row_shr 1, 2, 4, 8
    v = op(v, dpp_move<0x112, 0xf>(none, v));
    v = op(v, dpp_move<0x114, 0xf>(none, v));
    v = op(v, dpp_move<0x118, 0xf>(none, v));
    v = op(v, dpp_move<0x142, 0xa>(none, v));     // row_bcast 15 into rows 1 and 3
    v = op(v, dpp_move<0x143, 0xc>(none, v));     // row_bcast 31 into rows 2 and 3
    return lane63(v);
}
__device__ __forceinline__ float wave_max(float v) {
    return wave_reduce(v, -INFINITY, [](float a, float b) { return fmaxf(a, b); });
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
    return wave_reduce(v, 0u, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
}
__device__ __forceinline__ float wave_sum(float v) {
    return wave_reduce(v, 0.0f, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ double wave_sum(double v) {
    return wave_reduce(v, 0.0, [](double a, double b) { return a + b; });
}
// The same within groups of GROUP (2, 4, 8, 16) neighbouring lanes, every lane getting the result: exchanges inside
// quads, then mirrored halves and rows (which hold one value per half or row by then).
template <int GROUP, typename T, typename OP>
__device__ __forceinline__ T group_reduce(T v, OP op) {
    if constexpr (GROUP >= 2) v = op(v, dpp_move<0xb1, 0xf>(v, v));          // quad_perm 1 0 3 2
    if constexpr (GROUP >= 4) v = op(v, dpp_move<0x4e, 0xf>(v, v));          // quad_perm 2 3 0 1
    if constexpr (GROUP >= 8) v = op(v, dpp_move<0x141, 0xf>(v, v));         // row_half_mirror
    if constexpr (GROUP >= 16) v = op(v, dpp_move<0x140, 0xf>(v, v));        // row_mirror
    return v;
}
// lane n of every group of GROUP (8 or 16) neighbouring lanes, n a constant
template <int GROUP, int N>
__device__ __forceinline__ double group_bcast(double v) {
    static_assert(GROUP == 8 || GROUP == 16, "groups of half a row or a row");
    const double a = dpp_move<0x150 + N, 0xf>(v, v);                         // row_newbcast
    if constexpr (GROUP == 16) return a;
    const double b = dpp_move<0x150 + N + 8, 0xf>(v, v);
    return (threadIdx.x & 8) ? b : a;
}
// the value of the lane 16 or 32 lanes away (rows or halves of the wave swapped), for symmetric operations: returns
// op(own, other) in every lane
template <int DIST, typename OP>
__device__ __forceinline__ double swap_reduce(double v, OP op) {
    static_assert(DIST == 16 || DIST == 32, "row or half");
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)u, hi = (uint32_t)(u >> 32);
    uint32_t a[2], b[2];
    if constexpr (DIST == 16) {
        const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false), h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        a[0] = l[0]; a[1] = h[0]; b[0] = l[1]; b[1] = h[1];
    } else {
        const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false), h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        a[0] = l[0]; a[1] = h[0]; b[0] = l[1]; b[1] = h[1];
    }
    return op(__longlong_as_double((long long)((uint64_t)a[1] << 32 | a[0])), __longlong_as_double((long long)((uint64_t)b[1] << 32 | b[0])));
}
template <int DIST>
__device__ __forceinline__ int swap_sum(int v) {
    if constexpr (DIST == 16) {
        const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
        return (int)(l[0] + l[1]);
    } else {
        const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
        return (int)(l[0] + l[1]);
    }
}
__device__ __forceinline__ double add_f64(double a, double b) { return a + b; }
__device__ __forceinline__ double max_f64(double a, double b) { return fmax(a, b); }
// workgroup reductions over NW waves; sm: NW floats of LDS; sums are added in a fixed order
template <int NW>
__device__ __forceinline__ float block_max(float v, float *sm) {
    v = wave_max(v);
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
    __syncthreads();
    float r = sm[0];
#pragma unroll
    for (int i = 1; i < NW; i++) r = fmaxf(r, sm[i]);
    __syncthreads();
    return r;
}
template <int NW>
__device__ __forceinline__ double block_sum(double v, double *sm) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
    __syncthreads();
    double r = sm[0];
#pragma unroll
    for (int i = 1; i < NW; i++) r += sm[i];
    __syncthreads();
    return r;
}
template <int NW>
__device__ __forceinline__ float block_sum(float v, float *sm) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = v;
    __syncthreads();
    float r = sm[0];
#pragma unroll
    for (int i = 1; i < NW; i++) r += sm[i];
    __syncthreads();
    return r;
}
// Workgroup barrier that orders the LDS traffic only.  (__syncthreads() would also wait for
// every load from global memory in flight, e.g. for weights requested ahead.)
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}
// Keeps an fp32 value in a register as fp32: the compiler may otherwise fold "fp32 multiply,
// then convert to fp16" into one mixed-precision instruction that rounds the exact product
// once, which differs from the two-step result on double-rounding cases.
__device__ __forceinline__ float keep_f32(float v) {
    asm volatile("" : "+v"(v));
    return v;
}
// one decoded hidden-state value: fp32 product, one rounding to fp16
__device__ __forceinline__ __half decode_q8(const float *table, uint32_t code, float absmax) {
    return __float2half_rn(keep_f32(table[code] * absmax));
}
// double -> fp16 with ONE rounding (to nearest even): the value is first rounded to odd at the 20 mantissa bits of
// its high word (the low word only says whether anything lies below them), which is exact in fp32 and keeps enough
// for the rounding to fp16 to be the only one.  (keep_f32: the compiler would otherwise see one conversion from fp64
// to fp16, for which there is no instruction, and expand it into forty.)
__device__ __forceinline__ __half d2h_rn(double v) {
    const uint64_t u = __double_as_longlong(v);
    const uint32_t lo = (uint32_t)u, hi = (uint32_t)(u >> 32) | min(lo, 1u);
    return __float2half_rn(keep_f32((float)__longlong_as_double((long long)((uint64_t)hi << 32))));
}
__device__ __forceinline__ uint32_t pk_max_u16(uint32_t a, uint32_t b) {     // of the two halves of a word
    typedef unsigned short us2 __attribute__((ext_vector_type(2)));
    const us2 r = __builtin_elementwise_max(*(us2 *)&a, *(us2 *)&b);
    return *(const uint32_t *)&r;
}
template <typename F, int... I>
__device__ __forceinline__ void for_constants(F f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>()), ...);
}
// smallest non-negative fp16 bit pattern whose value is >= theta (fp16 magnitudes order like their bits)
inline uint32_t ps_theta_to_bits(float theta) {
    if (!(theta > 0.0f)) return 0u;
    _Float16 h = (_Float16)theta;          // round to nearest
    unsigned short b;
    memcpy(&b, &h, 2);
    if ((float)h < theta) b++;             // next pattern up (0x7bff + 1 = 0x7c00 = +inf)
    return b;
}
// int8 code of one activation/weight: fp32 product, round half to even, clamp
__device__ __forceinline__ int q8(float x, float r) {
    float q = rintf(x * r);
    q = fminf(fmaxf(q, -127.0f), 127.0f);
    return (int)q;
}
__device__ __forceinline__ int pack4(int a, int b, int c, int d) {
    return (a & 0xff) | ((b & 0xff) << 8) | ((c & 0xff) << 16) | ((d & 0xff) << 24);
}

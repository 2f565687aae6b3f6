// Prefill-size linear (M > 64 rows) on the matrix cores with LDS-staged operand tiles.
//
// Regular columns: int8 x int8 -> int32 with v_mfma_i32_16x16x64_i8.  Both operands already sit
// in HBM in 16x64 tiles whose 1024 bytes are in the lane order of that instruction, so a tile
// travels global -> LDS -> registers as plain 16-byte per-lane copies (bank-conflict free, no
// transposition).  A workgroup computes a block of the output, 256 x 256 in large calls; k-tiles move
// through a 4-slot LDS ring filled by asynchronous global->LDS copies.
//
// Outlier columns: up to ps_exact_outliers of them are added exactly in the epilogue (fp64 matrix
// instruction on compacted operands, see outlier_prep.h).  More than that: the fp16 x fp16 product over the
// outlier columns is computed EXACTLY in integer arithmetic on the int8 matrix cores.  Every fp16 value
// is an integer multiple of 2^-24, so an activation is x = 2^-24 * sum_j 256^j * L_j with balanced
// 8-bit digits L_j (4 of them up to |x| < 127.5, at most 6); a dequantized weight of output row n,
// Wd = fp16(code * a_n), is u_n * (m_n * code + r) with u_n the fp16 spacing at a_n, m_n = a_n / u_n
// rounded to an integer (11 bits) and a remainder r that always fits 8 bits.  The gathered digit
// matrices [digits * M, n_out] and [2 * N, n_out] go through the same pipeline as the regular
// columns (int32 sums: exact), and each wave reassembles
//   sum_k x * Wd = u_n * 2^-24 * (m_n * sum_j 256^j * A_c[j] + sum_j 256^j * A_r[j])
// in fp64 for the int8 kernel's epilogue to add.  (The fp16 matrix instruction with its fp32 sums
// lands one fp16 rounding step off in about one output of 300 at 57344 columns, and a neighbouring
// value is enough to move a row maximum or cross the outlier threshold downstream.)
//
// The fp16 form of the pipeline serves the backward pass as a plain product of two tile arrays
// (ps_gemm_f16_tiles): fp32 result, or for the down linear fp16(result * GeLU') in the tile order of the
// next product.
#include <mutex>

#include "common.h"
#include "digits.h"
#include "epilogue.h"

namespace {

constexpr int PS_KSPLIT_MAX = 8;   // workgroups that share one output block's contraction, at most

// ---------------------------------------------------------------------------------------------
// outlier column list and fp16 gathers (only do work when the call has > ps_exact_outliers)

// Digit tiles of the outlier columns, in the int8 operand order (16 rows x 64 compacted columns = 1024 bytes, lane l owns row
// l%16 and columns (l/16)*16 .. +16), one wave per tile or run of tiles.
//
// Activations: digit j of token tile mt, column tile ct at ((j * MTT + mt) * CT + ct) * 1024.  All PS_X_DIGITS digit planes
// are written; count[1] receives the number of planes that hold anything (at least 4), which is what the product walks.
// Weights: digit 0 (the int8 codes) of panel nt, column tile ct at ((nt) * CT + ct) * 1024, digit 1 (the remainders) at
// ((NT + nt) * CT + ct) * 1024.
__device__ __forceinline__ void store_x_digits(__half (&x)[16], bool live, int8_t *__restrict__ xl, size_t plane, size_t tile, int &need) {
    const int lane = threadIdx.x & 63;
    bool big = false;
#pragma unroll
    for (int e = 0; e < 16; e++) {
        uint32_t b = __half_as_ushort(x[e]);
        if (!live || (b & 0x7fffu) >= 0x7c00u) b = 0;               // not a number / infinite: unspecified, stay defined
        big |= (b & 0x7fffu) >= DIGITS_BIG;
        x[e] = __ushort_as_half((unsigned short)b);
    }
    v4i dig[PS_X_DIGITS];
#pragma unroll
    for (int p = 0; p < PS_X_DIGITS; p++) dig[p] = (v4i){0, 0, 0, 0};
    if (!__any(big)) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
            int p4[4];
            digit_planes4(*(const __half(*)[4])(x + 4 * q), p4);
#pragma unroll
            for (int p = 0; p < 4; p++) dig[p][q] = p4[p];
        }
    } else {                                                        // values that take more than four digits: in 64 bits
#pragma unroll
        for (int e = 0; e < 16; e++) {
            long long I = (long long)((double)__half2float(x[e]) * 16777216.0);     // exact: every fp16 value is a multiple of 2^-24
#pragma unroll
            for (int p = 0; p < PS_X_DIGITS; p++) {
                const int d = (int)((I + 128) & 255) - 128;         // balanced digit in [-128, 127]
                I = (I - d) >> 8;
                dig[p][e >> 2] |= (d & 0xff) << (8 * (e & 3));
                if (d != 0) need = max(need, p + 1);
            }
            __builtin_amdgcn_sched_barrier(0);                      // one after the other: side by side they take 90 registers
        }
    }
#pragma unroll
    for (int p = 0; p < PS_X_DIGITS; p++) *(v4i *)(xl + ((p * plane + tile) * 64 + lane) * 16) = dig[p];
}
__device__ __forceinline__ void store_w_digits(const v4i &codes, float sw, int8_t *__restrict__ wd, size_t plane, size_t tile) {
    const int lane = threadIdx.x & 63;
    float a;
    int E, m;
    const bool scaled = digit_scale(sw, a, E, m);
    v4i rem = digit_remainders(codes, a, (_Float16)a, (_Float16)ldexpf(1.5f, E));
    if (!(sw <= 65504.0f)) {                                        // some weight of the row may overflow fp16: those count as their codes
#pragma unroll
        for (int q = 0; q < 4; q++) {
            rem[q] = 0;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const int c = (int)(int8_t)(codes[q] >> (8 * e));
                int r = 0;
                if (scaled) {
                    const float v = dequant_w16(c, a);
                    if (fabsf(v) <= 65504.0f) r = (int)ldexpf(v, 10 - E) - m * c;
                }
                rem[q] |= (min(max(r, -128), 127) & 0xff) << (8 * e);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    *(v4i *)(wd + (tile * 64 + lane) * 16) = codes;
    *(v4i *)(wd + ((plane + tile) * 64 + lane) * 16) = rem;
}

// One column at a time.  The weights always: 64 columns of a panel's codes lie within a few cache lines, which the lanes share
// (a linear of 65 rows at half of its columns, 14336 x 57344, 4096 x 16384 and 16384 x 4096: 1007, 175 and 117 us; with the
// codes compacted as below 1228, 201 and 141; at three quarters 1426, 231 and 144 against 1422, 240 and 150; only with nearly
// all columns of the largest it is 1 to 4 % behind).
__device__ __forceinline__ void weight_digits(const LinearW &w, const int *__restrict__ list, int8_t *__restrict__ wd, int n_out, int bid, int nblk) {
    const int CT = (n_out + 63) >> 6, NT = w.N >> 4, KT = w.K >> 6, lane = threadIdx.x & 63, row = lane & 15;
    for (int item = bid; item < NT * CT; item += nblk) {
        const int nt = item / CT, ct = item - nt * CT;
        int id[16], c[16];
#pragma unroll
        for (int q = 0; q < 4; q++) *(int4 *)(id + 4 * q) = ((const int4 *)(list + ct * 64 + (lane >> 4) * 16))[q];
#pragma unroll
        for (int e = 0; e < 16; e++) {
            const int k = max(id[e], 0);
            c[e] = w.wt[((size_t)nt * KT + (k >> 6)) * 1024 + (((k & 63) >> 4) * 16 + row) * 16 + (k & 15)];
        }
        v4i codes;
#pragma unroll
        for (int q = 0; q < 4; q++)
            codes[q] = pack4(id[4 * q] < 0 ? 0 : c[4 * q], id[4 * q + 1] < 0 ? 0 : c[4 * q + 1], id[4 * q + 2] < 0 ? 0 : c[4 * q + 2], id[4 * q + 3] < 0 ? 0 : c[4 * q + 3]);
        store_w_digits(codes, w.sw[nt * 16 + row], wd, (size_t)NT * CT, (size_t)nt * CT + ct);
    }
}
__device__ __forceinline__ void token_digits_gathered(const __half *__restrict__ X, int M, int K, const int *__restrict__ list,
                                                      int8_t *__restrict__ xl, int n_out, int bid, int nblk, int &need) {
    const int CT = (n_out + 63) >> 6, MTT = (M + 15) >> 4, lane = threadIdx.x & 63;
    for (int item = bid; item < MTT * CT; item += nblk) {
        const int mt = item / CT, ct = item - mt * CT, t = mt * 16 + (lane & 15);
        int id[16];
#pragma unroll
        for (int q = 0; q < 4; q++) *(int4 *)(id + 4 * q) = ((const int4 *)(list + ct * 64 + (lane >> 4) * 16))[q];
        const __half *xr = X + (size_t)min(t, M - 1) * K;
        __half x[16];
#pragma unroll
        for (int e = 0; e < 16; e++) x[e] = xr[max(id[e], 0)];                  // always in bounds
#pragma unroll
        for (int e = 0; e < 16; e++)
            if (id[e] < 0) x[e] = __ushort_as_half(0);
        store_x_digits(x, t < M, xl, (size_t)MTT * CT, (size_t)mt * CT + ct, need);
    }
}

// Most columns: a wave makes up to DT_TILES consecutive tiles of one row tile at a time.  It reads the rows as they lie (a lane
// 16 columns, DT_AHEAD k-tiles at once: with one it waits for each in turn) and drops the outlier columns into its piece of
// LDS in the order of the tiles.  From four columns in seven on: there the columns of DT_TILES tiles lie within DT_AHEAD
// k-tiles (1024 x 16384 at 8192 rows with half of the columns 974 us by column and 999 this way, with five in eight 1115 and
// 1049; 200 rows with 400 of 32768 columns 460 and 689).
constexpr int DT_TILES = 4, DT_AHEAD = 8;

// what the lanes of a wave have written to LDS is there for its other lanes
__device__ __forceinline__ void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ void token_digits_compacted(const __half *__restrict__ X, int M, int K, const uint64_t *__restrict__ mask64,
                                                       const int *__restrict__ list, int8_t *__restrict__ xl, int n_out, __half *st,
                                                       int bid, int nblk, int &need) {
    const int CT = (n_out + 63) >> 6, MTT = (M + 15) >> 4, lane = threadIdx.x & 63, row = lane & 15, g = lane >> 4;
    const int ranges = (CT + DT_TILES - 1) / DT_TILES;
    for (int item = bid; item < MTT * ranges; item += nblk) {
        const int mt = item / ranges, ct0 = (item - mt * ranges) * DT_TILES, t = mt * 16 + row;
        const __half *src = X + (size_t)min(t, M - 1) * K + g * 16;
        // the outlier columns of ranks [64 ct0, 64 (ct0 + DT_TILES)) into st[tile][lane][16], zero where there is none
        const int k0 = list[ct0 * 64], kt1 = list[min(n_out, (ct0 + DT_TILES) * 64) - 1] >> 6;   // uniform; ascending
#pragma unroll
        for (int i = 0; i < DT_TILES * 2; i++) ((v4i *)st)[i * 64 + lane] = (v4i){0, 0, 0, 0};
        wave_sync_lds();
        int base = -__popcll(mask64[k0 >> 6] & ((1ull << (k0 & 63)) - 1));          // rank of the k-tile's first outlier, from 64 ct0
        for (int kt = k0 >> 6; kt <= kt1; kt += DT_AHEAD) {
            uint64_t bits[DT_AHEAD];
            __half v[DT_AHEAD][16];
#pragma unroll
            for (int u = 0; u < DT_AHEAD; u++) {
                const __half *from = src + (size_t)min(kt + u, kt1) * 64;
                bits[u] = kt + u <= kt1 ? mask64[kt + u] : 0;
                *(v8h *)v[u] = *(const v8h *)from;
                *(v8h *)(v[u] + 8) = *(const v8h *)(from + 8);
            }
#pragma unroll
            for (int u = 0; u < DT_AHEAD; u++) {
                const uint32_t mine = (uint32_t)(bits[u] >> (16 * g)) & 0xffffu;
                int pos = base + __popcll(bits[u] & ((1ull << (16 * g)) - 1));
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    if ((mine >> e) & 1u) {
                        if ((uint32_t)pos < 64u * DT_TILES) st[((pos >> 6) * 64 + row + 16 * ((pos >> 4) & 3)) * 16 + (pos & 15)] = v[u][e];
                        pos++;
                    }
                }
                base += __popcll(bits[u]);
            }
        }
        wave_sync_lds();
        for (int j = 0; j < DT_TILES && ct0 + j < CT; j++) {
            __half x[16];
            *(v8h *)x = *(const v8h *)(st + (j * 64 + lane) * 16);
            *(v8h *)(x + 8) = *(const v8h *)(st + (j * 64 + lane) * 16 + 8);
            store_x_digits(x, t < M, xl, (size_t)MTT * CT, (size_t)mt * CT + ct0 + j, need);
        }
        wave_sync_lds();                 // read before the next item's zeros
    }
}

// ---------------------------------------------------------------------------------------------
// the tile pipeline

struct GemmArgs {
    const unsigned char *a_tiles;   // weight-side tiles: [rows][KTILES][1024]
    const unsigned char *b_tiles;   // token-side tiles:  [rows][KTILES][1024]
    const unsigned char *a_regular, *b_regular;     // int8: ManyOutliers' wd and xl
    int ktiles;                     // int8: K/64.  fp16: the plain product's tile count.  digits: derived from the outlier count
    int M, N;
    int exact;                      // ps_exact_outliers
    int nb_n, nb_m;                 // output blocks of this launch along the features and along the tokens
    int nb_n0;                      // first feature block of this launch (a linear may be split over two launches)
    // plain fp16 product only: instead of the fp32 result, store fp16(result * GeLU'(gelu_pre)) in the tile order
    // of the next product's token-side operand (16 x 32 tiles, rows beyond M zero)
    const __half *gelu_pre;   // [M, N] fp16, or null
    __half *tile_out;
    double *od;               // digit product only: [M, N] fp64, the product over the outlier columns
    // int8 product with EPI_PARTIAL only: the k-tiles are shared out over ksplit workgroups per output block, each of
    // which stores its raw sums to part[split][weight panel][token tile][lane]; k_split_finish adds and finishes them
    int ksplit;
    v4i *part;
    float *f32_out;           // plain fp16 product: [M, N] fp32 result
};

// Tiles [rows][tiles of `list`][1024] of the listed columns of src, which has KT tiles to a row; 0 where the list has -1.
__device__ __forceinline__ void gather_codes(const int8_t *__restrict__ src, int rows, int KT, const int *__restrict__ list, int n,
                                             int8_t *__restrict__ dst, int bid, int nblk) {
    const int RT = (n + 63) >> 6, lane = threadIdx.x & 63, row = lane & 15;
    for (int item = bid; item < rows * RT; item += nblk) {
        const int r = item / RT, rt = item - r * RT;
        int id[16], c[16];
#pragma unroll
        for (int q = 0; q < 4; q++) *(int4 *)(id + 4 * q) = ((const int4 *)(list + rt * 64 + (lane >> 4) * 16))[q];
#pragma unroll
        for (int e = 0; e < 16; e++) {
            const int k = max(id[e], 0);
            c[e] = src[((size_t)r * KT + (k >> 6)) * 1024 + (((k & 63) >> 4) * 16 + row) * 16 + (k & 15)];
        }
        v4i codes;
#pragma unroll
        for (int q = 0; q < 4; q++)
            codes[q] = pack4(id[4 * q] < 0 ? 0 : c[4 * q], id[4 * q + 1] < 0 ? 0 : c[4 * q + 1], id[4 * q + 2] < 0 ? 0 : c[4 * q + 2], id[4 * q + 3] < 0 ? 0 : c[4 * q + 3]);
        *(v4i *)(dst + ((size_t)item * 64 + lane) * 16) = codes;
    }
}

// Both kinds of digit tiles in one launch (a launch costs as much as the work of a call with few tiles): the first NBX waves
// cut the activations, the rest the weights.  Workgroups of four waves, which share nothing: a launch that finds nothing to
// do costs by its number of workgroups.  Does nothing unless the call has more outlier columns than the fp64 path takes.
__global__ void __launch_bounds__(256) k_digit_tiles(const __half *__restrict__ X, int M, LinearW w, const uint32_t *__restrict__ mask,
                                                      int *__restrict__ count, const int *__restrict__ list,
                                                      int8_t *__restrict__ xl, int8_t *__restrict__ wd, int NBX,
                                                      const int8_t *__restrict__ xq_tiled, const int *__restrict__ regular) {
    __shared__ __align__(16) __half stage[4][DT_TILES * 64 * 16];
    const int n_out = count[0];
    if (n_out <= ps_exact_outliers(w.N, M)) return;
    const int wave = threadIdx.x >> 6, wv = (int)blockIdx.x * 4 + wave, KT = w.K >> 6, CT = (n_out + 63) >> 6;
    const bool gather = regular && ps_regular_compacted(n_out, w.K, M);
    if (wv >= NBX) {
        const int NT = w.N >> 4;
        weight_digits(w, list, wd, n_out, wv - NBX, (int)gridDim.x * 4 - NBX);
        if (gather) gather_codes(w.wt, NT, KT, regular, w.K - n_out, wd + (size_t)2 * NT * CT * 1024, wv - NBX, (int)gridDim.x * 4 - NBX);
        return;
    }
    if (gather) {
        const int MTT = (M + 15) >> 4;
        gather_codes(xq_tiled, MTT, KT, regular, w.K - n_out, xl + (size_t)PS_X_DIGITS * MTT * CT * 1024, wv, NBX);
    }
    int need = 0;
    if (n_out * 7 >= w.K * 4) token_digits_compacted(X, M, w.K, (const uint64_t *)mask, list, xl, n_out, stage[wave], wv, NBX, need);
    else token_digits_gathered(X, M, w.K, list, xl, n_out, wv, NBX, need);
    if (need > 4) atomicMax(count + 1, need);
}

enum { GEMM_INT8 = 0, GEMM_F16 = 1, GEMM_DIGITS = 2 };
constexpr int EPI_PARTIAL = 3;

// MODE GEMM_INT8: the regular columns with the full epilogue.  GEMM_F16: plain fp16 product (backward pass).
// GEMM_DIGITS: int8 digit products of the outlier columns, reassembled per wave into the fp64 product.  A
// wave's 8 x 4 accumulator tiles are then 2 weight digits x 4 panels against the 4 digit planes of ONE token
// tile, so every lane holds all eight partial sums of its 16 outputs and nothing has to meet in memory.
// NSLOT: LDS ring slots (NSLOT - 1 stages are requested ahead).
// EPI (GEMM_INT8 only): what is fused before the fp16 rounding, 0 nothing, 1 tanh-GeLU, 2 + residual; a template
// argument because the tail's arithmetic must be straight-line code for the 16 outputs a lane finishes at a time
// to overlap (with run-time switches inside, every output's chain of dependent fp64 operations ran on its own).
template <int MODE, int WVN, int WVM, int TN, int TM, int NSLOT, int EPI>
__global__ void __launch_bounds__(64 * WVN * WVM, TN * TM <= 8 ? 4 : 2)   // waves per SIMD: at most 256 registers, small blocks 128
k_gemm_lds(GemmArgs ga, LinearW w, const float *__restrict__ sx, OutlierSet os, const double *__restrict__ outl, OutDesc o,
           const SessTable *__restrict__ sess) {
    constexpr bool F16 = MODE == GEMM_F16, DIG = MODE == GEMM_DIGITS;
    constexpr int NW = WVN * WVM, BN = WVN * TN, BM = WVM * TM, STAGE = BN + BM, LOADS = (STAGE + NW - 1) / NW;
    constexpr int FULL = STAGE % NW;                 // waves that copy LOADS tiles per stage, the others one less (0: all copy LOADS)
    constexpr int PD = NSLOT - 1;                    // stages requested ahead
    extern __shared__ __align__(16) unsigned char lds[];
    const int n_out = F16 ? ga.ktiles * 32 : os.count[0];
    const bool many = F16 || n_out > ga.exact;
    if (DIG && !many) return;
    if constexpr (DIG) __builtin_assume(n_out > 0);  // there is a k-tile (not told so, the loop takes 0.5 % longer)
    // k-tiles to walk (64 int8 or 32 fp16 columns each).  If EVERY column is an outlier all int8 codes are
    // zero: the int8 product is skipped and only the epilogue runs.
    int KTILES = F16 ? ga.ktiles : DIG ? (n_out + 63) >> 6 : ga.ktiles;       // tiles per row of the operands
    const unsigned char *a_tiles = ga.a_tiles, *b_tiles = ga.b_tiles;
    if constexpr (MODE == GEMM_INT8 && EPI != EPI_PARTIAL) {
        if (many && ps_regular_compacted(n_out, ga.ktiles * 64, ga.M)) {        // the regular columns' codes by themselves
            KTILES = ga.ktiles - (n_out >> 6);
            a_tiles = ga.a_regular + (size_t)2 * (ga.N >> 4) * ((n_out + 63) >> 6) * 1024;
            b_tiles = ga.b_regular + (size_t)PS_X_DIGITS * ((ga.M + 15) >> 4) * ((n_out + 63) >> 6) * 1024;
        }
    }
    int NS = !F16 && !DIG && n_out == ga.ktiles * 64 ? 0 : KTILES;

    // Workgroup -> output block.  Consecutive workgroup ids land on different XCDs (8 of them, each
    // with its own L2); give each XCD a contiguous run of blocks, ordered in strips of up to STRIP
    // m-blocks, so that the blocks an XCD works on at one time share weight and token tiles in its L2.
    // Small blocks: strips of about the same width; in one of a single m-block an XCD reads the weights of its
    // whole run of feature blocks by itself (3072 x 3072 at 300 rows, 5 m-blocks as 4 + 1 39 us, as 3 + 2 31).  Wider
    // strips: 2048 x 2048 at 1024 rows 35 -> 42.
    const int nb_n = ga.nb_n, nb_m = ga.nb_m, ksplit = EPI == EPI_PARTIAL ? ga.ksplit : 1;
    const int total = nb_n * nb_m * ksplit, per_xcd = (total + 7) >> 3;
    int ord = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_xcd || ord >= total) return;
    int split = 0, s_first = 0;                      // this workgroup's k-tiles: [s_first, s_first + NS)
    if constexpr (EPI == EPI_PARTIAL) {
        split = ord / (nb_n * nb_m);
        ord -= split * nb_n * nb_m;
        s_first = (int)((long long)NS * split / ksplit);
        NS = (int)((long long)NS * (split + 1) / ksplit) - s_first;
    }
    constexpr int STRIP = 4;
    const int nstrips = (nb_m + STRIP - 1) / STRIP, width = BN + BM < 24 ? (nb_m + nstrips - 1) / nstrips : STRIP;
    const int strip = min(ord / (width * nb_n), nstrips - 1);
    const int rem = ord - strip * width * nb_n, sw_this = min(width, nb_m - strip * width);
    const int bn = rem / sw_this, bm = strip * width + rem % sw_this;

    // Digit product: planes 0..3 first, then, only when some outlier value reaches 127.5 in magnitude, planes 4.. as a
    // second pass over the same block, which adds to what the first one stored (as a launch of its own the second pass
    // cost every linear 2.4 us of finding nothing to do).  Everything that depends on the thread is worked out again in
    // each pass: kept over the loop it cost 18 spilled registers.
    const int groups = DIG ? (os.count[1] + 3) >> 2 : 1;
#pragma unroll 1
    for (int pg = 0; pg < groups; pg++) {
    int tid = threadIdx.x;
    if constexpr (DIG) {
        asm volatile("" : "+v"(tid));
        if (pg) {                                             // every wave is done with the slots of the first pass
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
    }
    const int M = ga.M, N = ga.N, NT = N >> 4, MTT = (M + 15) >> 4;
    // (the wave's number as a scalar: six to eight fewer registers, but the digit product's schedule gets slower by it, 29.0
    // against 29.3 ms for a prefill call of 8 x 512 tokens of a 14336-wide block)
    const int wave = DIG ? tid >> 6 : __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, row = lane & 15, kg = lane >> 4;
    const int wn = wave / WVM, wm = wave % WVM;
    const int nt0 = (ga.nb_n0 + bn) * BN, mt0 = bm * BM;

    // the stage tiles this wave copies: s = wave + NW*j; s < BN: weight tile, else token tile
    const unsigned char *src[LOADS];
#pragma unroll
    for (int j = 0; j < LOADS; j++) {
        const int s = wave + NW * j;
        if constexpr (DIG) {
            static_assert(MODE != GEMM_DIGITS || (TN == 8 && TM == 4), "digit slots: 2 digits x 4 panels, 4 planes of one token tile");
            if (s < BN) {                    // slot: wave column s / 8, digit (s % 8) / 4, panel 4 * (2 bn + s / 8) + s % 4
                const int panel = min((bn * WVN + s / TN) * 4 + (s & 3), NT - 1);
                src[j] = ga.a_tiles + ((size_t)((s % TN) / 4) * NT + panel) * KTILES * 1024 + lane * 16;
            } else {                         // slot: wave row t / 4 = token tile, plane t % 4 of the group
                const int t = s - BN, plane = min(pg * 4 + (t & 3), PS_X_DIGITS - 1);
                src[j] = ga.b_tiles + ((size_t)plane * MTT + min(bm * WVM + t / TM, MTT - 1)) * KTILES * 1024 + lane * 16;
            }
        } else {
            if (s < BN) src[j] = a_tiles + ((size_t)min(nt0 + s, NT - 1) * KTILES + s_first) * 1024 + lane * 16;
            else src[j] = b_tiles + ((size_t)min(mt0 + s - BN, MTT - 1) * KTILES + s_first) * 1024 + lane * 16;
        }
    }

    typedef typename std::conditional<F16, v4f, v4i>::type acc_t;
    acc_t acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; i++)
#pragma unroll
        for (int j = 0; j < TM; j++) acc[i][j] = (acc_t){0, 0, 0, 0};

    // k-tiles travel global -> LDS with the asynchronous global_load_lds instruction (no staging
    // registers): one instruction copies one 1 KB tile, lane l supplying the address of bytes
    // [16 l, 16 l + 16) and the hardware writing them to tile base + 16 l.  The ring holds PD stages
    // in flight, which covers the latency of an L2 miss.  Copies of one wave complete in order, so
    // "stage s has landed" is "at most LOADS * (stages requested after s) copies outstanding".
    auto dma_part = [&](int s, int j0, int j1) {
        unsigned char *slot = lds + (size_t)(s % NSLOT) * STAGE * 1024;
#pragma unroll
        for (int j = j0; j < j1; j++) {
            if (FULL && j == LOADS - 1 && wave >= FULL) break;
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void *)(src[j] + (size_t)s * 1024),
                (__attribute__((address_space(3))) void *)(slot + (size_t)(wave + NW * j) * 1024), 16, 0, 0);
        }
    };
    auto wait_own = [&](int in_flight_after) {
        if (FULL && wave >= FULL) {
            if (in_flight_after >= 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS * 2 - 2) : "memory");
            else if (in_flight_after == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS - 1) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        } else if (in_flight_after >= 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS * 2) : "memory");
        else if (in_flight_after == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    static_assert(PD <= 3 && PD >= 2, "wait_own distinguishes at most two stages in flight behind the awaited one");
    auto frag_load = [&](int s, v4i *fa, v4i *fb) {
        const unsigned char *base = lds + (size_t)(s % NSLOT) * STAGE * 1024 + lane * 16;
#pragma unroll
        for (int i = 0; i < TN; i++) fa[i] = *(const v4i *)(base + (size_t)(wn * TN + i) * 1024);
#pragma unroll
        for (int j = 0; j < TM; j++) fb[j] = *(const v4i *)(base + (size_t)(BN + wm * TM + j) * 1024);
    };
    for (int s = 0; s < PD && s < NS; s++) dma_part(s, 0, LOADS);

    // Fragments are double buffered in registers: while stage s is multiplied, the fragments of stage
    // s + 1 are read from LDS.  So at the barrier of iteration s, stage s + 1 must have landed.
    v4i fa0[TN], fb0[TM], fa1[TN], fb1[TM];
    if (NS > 0) {
        wait_own(min(NS - 1, PD - 1));              // stage 0 of this wave
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        frag_load(0, fa0, fb0);
    }
    auto multiply = [&](const v4i *ca, const v4i *cb, int e0, int e1) {     // eighths [e0, e1) of a stage
#pragma unroll
        for (int q = TN * TM * e0 / 8; q < TN * TM * e1 / 8; q++) {
            const int i = q / TM, j = q % TM;
            if constexpr (F16)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(*(const v8h *)&ca[i], *(const v8h *)&cb[j], acc[i][j], 0, 0, 0);
            else
                acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ca[i], cb[j], acc[i][j], 0, 0, 0);
        }
    };
    // The fragment reads of stage s + 1 are issued in the middle of the multiplications of stage s, so they
    // have half a stage to complete before the wait that precedes their first use.  No branch may separate
    // them from the multiplications: where two paths with different numbers of LDS reads in flight meet, the
    // compiler waits for all of them.  So the last stage goes through the same motions (its barrier is one
    // too many, its fragment reads fetch its own stage again).
    // pieces of the next stage's fragment reads, to be spread between the multiplications
    auto frag_part = [&](int s, v4i *fa, v4i *fb, int part) {           // part 0: token side, 1 / 2: halves of the weight side
        const unsigned char *base = lds + (size_t)(s % NSLOT) * STAGE * 1024 + lane * 16;
        if (part == 0) {
#pragma unroll
            for (int j = 0; j < TM; j++) fb[j] = *(const v4i *)(base + (size_t)(BN + wm * TM + j) * 1024);
        } else {
#pragma unroll
            for (int i = part == 1 ? 0 : TN / 2; i < (part == 1 ? TN / 2 : TN); i++)
                fa[i] = *(const v4i *)(base + (size_t)(wn * TN + i) * 1024);
        }
    };
    auto step = [&](int s, const v4i *ca, const v4i *cb, v4i *na, v4i *nb) {
        wait_own(max(0, min(NS - s - 2, PD - 2)));  // stage s + 1 of this wave (stages up to s + PD - 1 are requested)
        __builtin_amdgcn_s_barrier();               // everybody's stage s + 1 visible; everybody done reading stage s - 1
        asm volatile("" ::: "memory");
        // the copy requests (into the slot of stage s - 1) and the fragment reads are issued a few at a time
        // while the matrix pipe is busy, not in front of it
        const bool more = s + PD < NS;
        const int sn = min(s + 1, NS - 1);
        multiply(ca, cb, 0, 1);
        __builtin_amdgcn_sched_barrier(0);
        if (more) dma_part(s + PD, 0, LOADS / 2);
        __builtin_amdgcn_sched_barrier(0);
        multiply(ca, cb, 1, 2);
        __builtin_amdgcn_sched_barrier(0);
        if (more) dma_part(s + PD, LOADS / 2, LOADS);
        __builtin_amdgcn_sched_barrier(0);
        multiply(ca, cb, 2, 3);
        __builtin_amdgcn_sched_barrier(0);
        frag_part(sn, na, nb, 0);
        __builtin_amdgcn_sched_barrier(0);
        multiply(ca, cb, 3, 4);
        __builtin_amdgcn_sched_barrier(0);
        frag_part(sn, na, nb, 1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(ca, cb, 4, 5);
        __builtin_amdgcn_sched_barrier(0);
        frag_part(sn, na, nb, 2);
        __builtin_amdgcn_sched_barrier(0);
        multiply(ca, cb, 5, 8);
    };
    for (int s = 0; s < NS; s += 2) {
        step(s, fa0, fb0, fa1, fb1);
        if (s + 1 < NS) step(s + 1, fa1, fb1, fa0, fb0);
    }
    // all copies have landed (vmcnt(0) when the last stage was awaited); wait for every wave to finish
    // reading the last stage before the slots are reused below
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    // Epilogue.  D[lane][r] = output row 4*(l/16)+r of the weight tile, token l%16 of the token tile.
    // The accumulators go through LDS (each lane parks and re-reads only its own values, half of
    // the wave's tiles at a time) so that the tail is a rolled loop over weight panels instead of
    // TN*TM inlined copies.  What depends only on the output column (weight scale / 127, bias, where a
    // fused-QKV column goes) is tabulated in LDS once per block; what depends only on the token (row
    // scale / 127, row addresses) sits in registers: the loop body has no division left.
    constexpr int NPARK = TN % 2 ? 1 : 2, QN = TN / NPARK;               // weight panels parked at a time
    static_assert(BN % 2 == 0, "a block begins at a whole word of the outlier mask");
    acc_t *mine = (acc_t *)lds + (size_t)wave * (QN * TM * 64) + lane;
    if constexpr (DIG) {
        // acc[digit * 4 + p][j]: lane (token row l%16, features 4 * (l/16) + r) of panel p, weight digit, plane j.
        // sum_k x * Wd = u_n * 2^-24 * (m_n * sum_j 256^j A_code[j] + sum_j 256^j A_rem[j]), taken in fp64 from the top
        // plane down: exact below 2^53, i.e. up to the last step, and good to 1 part in 2^53 after it.
        const int tt = bm * WVM + wm, t = tt * 16 + row;
        const int live = min(4, os.count[1] - pg * 4);       // planes 6, 7 do not exist
        if (tt < MTT) {                                                  // wave-uniform
#pragma unroll
            for (int p = 0; p < 4; p++) {
                const int panel = (bn * WVN + wn) * 4 + p;
                if (panel >= NT) continue;                               // wave-uniform
                const int n0 = panel * 16 + 4 * kg;
                const float4 s4 = *(const float4 *)(w.sw + n0);
                const float sv[4] = {s4.x, s4.y, s4.z, s4.w};
                v4d res;
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    double tc = 0.0, tr = 0.0;
#pragma unroll
                    for (int j = 3; j >= 0; j--) {
                        if (j < live) {
                            tc = tc * 256.0 + (double)acc[p][j][r];
                            tr = tr * 256.0 + (double)acc[4 + p][j][r];
                        }
                    }
                    float a;
                    int E, m;
                    digit_scale(sv[r], a, E, m);
                    res[r] = ldexp((double)m * tc + tr, E - 34 + 32 * pg);   // u = 2^(E-10), activations in units of 2^-24
                }
                if (t < M) {
                    double *dst = ga.od + (size_t)t * N + n0;
                    if (pg) res += *(const v4d *)dst;
                    *(v4d *)dst = res;
                }
            }
        }
    } else if constexpr (F16) {
#pragma unroll
        for (int p = 0; p < NPARK; p++) {
#pragma unroll
            for (int i = 0; i < QN; i++)
#pragma unroll
                for (int j = 0; j < TM; j++) mine[(i * TM + j) * 64] = acc[p * QN + i][j];
#pragma unroll 1
            for (int idx = 0; idx < QN * TM; idx++) {
                const int nt = nt0 + wn * TN + p * QN + idx / TM, mt = mt0 + wm * TM + idx % TM;
                if (nt >= NT || mt >= MTT) continue;                    // wave-uniform
                const int t = mt * 16 + row, n0 = nt * 16 + 4 * kg;
                if (ga.gelu_pre) {
                    v4h du = {(_Float16)0, (_Float16)0, (_Float16)0, (_Float16)0};
                    if (t < M) {
                        const v4f a = mine[idx * 64];
                        const v4h pre = *(const v4h *)(ga.gelu_pre + (size_t)t * N + n0);
#pragma unroll
                        for (int r = 0; r < 4; r++) du[r] = (_Float16)(a[r] * gelu_tanh_grad((float)pre[r]));
                    }
                    *(v4h *)(ga.tile_out + (((size_t)mt * (N >> 5) + (n0 >> 5)) * 64 + row + 16 * ((n0 & 31) >> 3)) * 8 + (n0 & 7)) = du;
                } else if (t < M) {
                    *(v4f *)(ga.f32_out + (size_t)t * N + n0) = mine[idx * 64];
                }
            }
        }
    } else if constexpr (EPI == EPI_PARTIAL) {
#pragma unroll
        for (int i = 0; i < TN; i++)
#pragma unroll
            for (int j = 0; j < TM; j++) {
                const int nt = nt0 + wn * TN + i, mt = mt0 + wm * TM + j;
                if (nt < NT && mt < MTT) ga.part[(((size_t)split * NT + nt) * MTT + mt) * 64 + lane] = acc[i][j];
            }
    } else {
        constexpr size_t PARK = (size_t)NW * QN * TM * 1024;
        double *col_swd = (double *)(lds + PARK);                        // [BN * 16] weight scale / 127
        double *col_bias = col_swd + BN * 16;                            // [BN * 16]
        int2 *col_sc = (int2 *)(col_bias + BN * 16);                     // [BN * 4] fused-QKV: where 4 columns go
        uint32_t *col_flag = (uint32_t *)(col_sc + BN * 4);              // [BN / 2] outlier bits of this block's columns
        if (threadIdx.x < BN / 2) col_flag[threadIdx.x] = 0u;
        for (int i = threadIdx.x; i < BN * 16; i += 64 * NW) {
            const int n = nt0 * 16 + i;
            col_swd[i] = n < N ? (double)(w.sw[n] / 127.0f) : 0.0;
            col_bias[i] = n < N ? (double)__half2float(w.bias[n]) : 0.0;
        }
        if (o.scatter) {
            for (int i = threadIdx.x; i < BN * 4; i += 64 * NW) {
                // output row n = h*3d + p*d + j: queries to y[M, nh*d], keys/values into the caches
                const int n0 = nt0 * 16 + 4 * i, d = o.d, h = n0 / (3 * d), rem = n0 - h * 3 * d, p = rem / d, j = rem - p * d;
                col_sc[i] = p == 0 ? make_int2(-1, h * d + j) : make_int2((o.blk * 2 + (p == 2 ? 1 : 0)) * o.nh + h, j);
            }
        }
        // per token row of this lane (TM token tiles)
        double sxd[TM];
        __half *yrow[TM];            // plain: y row; fused QKV: query row
        __half *kvrow[TM];           // fused QKV: session cache + position * d
        int capd[TM];
        int trow[TM];
#pragma unroll
        for (int j = 0; j < TM; j++) {
            const int mt = mt0 + wm * TM + j, t = mt * 16 + row;
            const bool ok = mt < MTT && t < M;
            trow[j] = ok ? t : -1;
            const int tc = ok ? t : 0;
            sxd[j] = (double)(sx[tc] / 127.0f);
            kvrow[j] = nullptr;
            capd[j] = 0;
            if (!o.scatter) {
                yrow[j] = o.y + (size_t)tc * N;
            } else {
                const int sidx = tc / o.T, cap = sess->cap[sidx], pos = sess->len[sidx] + (tc - sidx * o.T);
                yrow[j] = o.y + (size_t)tc * (o.nh * o.d);
                kvrow[j] = sess->kv[sidx] + (size_t)pos * o.d;
                capd[j] = cap * o.d;
            }
        }
        // exact outlier part: the token-side operands of the first XC chunks stay in registers; the rest comes XR chunks at a time,
        // for all token tiles at once (one tile after the other, a weight operand and a latency for each: 4096 rows of 16384 x 4096
        // with 64 outlier columns 655 -> 528 us, 351 rows 116 -> 105).  No further ahead: 16 columns there 348 -> 428.
        constexpr int XC = TM == 1 ? 8 : 2, XR = TM == 1 ? 4 : 2;
        const int nch = many ? 0 : (n_out + 3) >> 2;
        double xw[TM][XC];
        if (nch > 0)
#pragma unroll
            for (int j = 0; j < TM; j++)
#pragma unroll
                for (int c = 0; c < XC; c++)
                    xw[j][c] = os.x64[((size_t)min(mt0 + wm * TM + j, MTT - 1) * PS_OUTLIER_CHUNKS + min(c, nch - 1)) * 64 + lane];
        __syncthreads();                                                 // tables visible

#pragma unroll
        for (int p = 0; p < NPARK; p++) {
#pragma unroll
            for (int i = 0; i < QN; i++)
#pragma unroll
                for (int j = 0; j < TM; j++) mine[(i * TM + j) * 64] = acc[p * QN + i][j];
#pragma unroll 1
            for (int i = 0; i < QN; i++) {
                const int ntl = wn * TN + p * QN + i, nt = nt0 + ntl;
                if (nt >= NT) continue;                                  // wave-uniform
                const int n0 = nt * 16 + 4 * kg;
                const v4d swd4 = *(const v4d *)(col_swd + ntl * 16 + 4 * kg);
                const v4d bias4 = *(const v4d *)(col_bias + ntl * 16 + 4 * kg);
                const int2 sc = o.scatter ? col_sc[ntl * 4 + kg] : make_int2(-1, n0);
                const double *ap = os.wd64 + (size_t)nt * PS_OUTLIER_CHUNKS * 64 + lane;
                double aw[XC];
                if (nch > 0)
#pragma unroll
                    for (int c = 0; c < XC; c++) aw[c] = ap[min(c, nch - 1) * 64];
                // 1. operands of the TM token tiles of this panel: parked sums, residuals, the outlier part
                v4i a4[TM];
                v4h r4[TM];
                v4d od[TM];
#pragma unroll
                for (int j = 0; j < TM; j++) {
                    a4[j] = mine[(i * TM + j) * 64];
                    if constexpr (EPI == 2) r4[j] = *(const v4h *)(o.resid + (size_t)max(trow[j], 0) * N + n0);   // rows out of range read row 0
                    od[j] = (v4d){0.0, 0.0, 0.0, 0.0};
                }
                if (many) {
#pragma unroll
                    for (int j = 0; j < TM; j++)
                        if (trow[j] >= 0) od[j] = *(const v4d *)(outl + (size_t)trow[j] * N + n0);
                } else if (nch > 0) {
#pragma unroll
                    for (int c = 0; c < XC; c++)
                        if (c < nch)
#pragma unroll
                            for (int j = 0; j < TM; j++) od[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(aw[c], xw[j][c], od[j], 0, 0, 0);
                    for (int c0 = XC; c0 < nch; c0 += XR) {
                        double a[XR], b[XR][TM];
#pragma unroll
                        for (int u = 0; u < XR; u++) {
                            const int c = min(c0 + u, nch - 1) * 64;
                            a[u] = ap[c];
#pragma unroll
                            for (int j = 0; j < TM; j++) b[u][j] = os.x64[(size_t)min(mt0 + wm * TM + j, MTT - 1) * PS_OUTLIER_CHUNKS * 64 + lane + c];
                        }
#pragma unroll
                        for (int u = 0; u < XR; u++)
                            if (c0 + u < nch)
#pragma unroll
                                for (int j = 0; j < TM; j++) od[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[u][j], od[j], 0, 0, 0);
                    }
                }
                // 2. the arithmetic of the 4 TM outputs, no branch inside, written one operation at a time over all of
                //    them so that consecutive instructions are independent (a wave issues in order)
                constexpr int NE = 4 * TM;
                double vv[NE];
#pragma unroll
                for (int e = 0; e < NE; e++) vv[e] = (double)a4[e >> 2][e & 3];
#pragma unroll
                for (int e = 0; e < NE; e++) vv[e] *= sxd[e >> 2];
#pragma unroll
                for (int e = 0; e < NE; e++) vv[e] = vv[e] * swd4[e & 3] + od[e >> 2][e & 3];
#pragma unroll
                for (int e = 0; e < NE; e++) vv[e] += bias4[e & 3];
                if constexpr (EPI == 1) {
#pragma unroll
                    for (int e = 0; e < NE; e++) vv[e] = gelu_tanh(vv[e]);
                } else if constexpr (EPI == 2) {
#pragma unroll
                    for (int e = 0; e < NE; e++) vv[e] += (double)(float)r4[e >> 2][e & 3];
                }
                // one rounding to fp16 (see d2h_rn)
                __half out[TM][4];
#pragma unroll
                for (int e = 0; e < NE; e++) out[e >> 2][e & 3] = d2h_rn(vv[e]);
                // (pins the arithmetic above this point: otherwise the compiler sinks each token tile's share of it
                // into that tile's conditional store below, and the chains no longer overlap)
                v2i packed[TM];
#pragma unroll
                for (int j = 0; j < TM; j++) {
                    packed[j] = *(const v2i *)out[j];
                    asm volatile("" : "+v"(packed[j][0]), "+v"(packed[j][1]));
                }
                // 3. stores and the optional by-products
#pragma unroll
                for (int j = 0; j < TM; j++) {
                    const int t = trow[j];
                    if (t < 0) continue;
                    if (o.acc_out) *(v4i *)(o.acc_out + (size_t)t * N + n0) = a4[j];
                    if (o.pre_out) {                     // the sum before the fused GeLU / residual (backward pass)
                        __half pre[4];
#pragma unroll
                        for (int r = 0; r < 4; r++) pre[r] = d2h_rn((double)a4[j][r] * sxd[j] * swd4[r] + od[j][r] + bias4[r]);
                        *(v2i *)(o.pre_out + (size_t)t * N + n0) = *(const v2i *)pre;
                    }
                    __half *dst;
                    if (sc.x < 0) {
                        dst = yrow[j] + sc.y;
                        if (o.next_mask) {               // collected per block in LDS, sent once below
                            uint32_t bits = 0;
#pragma unroll
                            for (int r = 0; r < 4; r++) {
                                const __half hv = __ushort_as_half((unsigned short)((uint32_t)packed[j][r >> 1] >> ((r & 1) * 16)));
                                if (fabsf(__half2float(hv)) >= o.next_theta) bits |= 1u << ((n0 + r) & 31);
                            }
                            if (bits) atomicOr(&col_flag[(ntl * 16 + 4 * kg) >> 5], bits);
                        }
                    } else {
                        dst = kvrow[j] + (size_t)sc.x * capd[j] + sc.y;
                    }
                    *(v2i *)dst = packed[j];
                }
            }
        }
        if (o.next_mask && !o.scatter) {
            __syncthreads();
            const int word = (nt0 * 16 >> 5) + threadIdx.x;
            if (threadIdx.x < BN / 2 && word < (N >> 5) && col_flag[threadIdx.x])
                atomicOr(&o.next_mask[word], col_flag[threadIdx.x]);
        }
    }
    }   // digit plane groups
}

// Second half of a split contraction: one wave per 16 x 16 output tile adds the partial sums, the outlier part and the
// linear's fused tail.
__global__ void __launch_bounds__(256) k_split_finish(GemmArgs ga, LinearW w, const float *__restrict__ sx, OutlierSet os,
                                                      const double *__restrict__ outl, OutDesc o,
                                                      const SessTable *__restrict__ sess) {
    const int NT = ga.N >> 4, MTT = (ga.M + 15) >> 4, lane = threadIdx.x & 63;
    const int item = blockIdx.x * 4 + (threadIdx.x >> 6), nt = item / MTT, mt = item - nt * MTT;
    if (nt >= NT) return;
    const int t = mt * 16 + (lane & 15), n0 = nt * 16 + 4 * (lane >> 4), n_out = os.count[0];
    v4i acc = {0, 0, 0, 0};
    for (int s = 0; s < ga.ksplit; s++) acc += ga.part[(((size_t)s * NT + nt) * MTT + mt) * 64 + lane];
    v4d od = {0.0, 0.0, 0.0, 0.0};
    if (n_out > ga.exact) {
        if (t < ga.M) od = *(const v4d *)(outl + (size_t)t * ga.N + n0);
    } else {
        const double *ap = os.wd64 + (size_t)nt * PS_OUTLIER_CHUNKS * 64 + lane, *bp = os.x64 + (size_t)mt * PS_OUTLIER_CHUNKS * 64 + lane;
        for (int c = 0; c < (n_out + 3) >> 2; c++) od = __builtin_amdgcn_mfma_f64_16x16x4f64(ap[c * 64], bp[c * 64], od, 0, 0, 0);
    }
    if (t < ga.M) emit_output4(o, sess, ga.N, t, n0, acc, od, sx[t] / 127.0f, w.sw, w.bias);
}

template <int MODE, int WVN, int WVM, int TN, int TM, int EPI = 0>
hipError_t launch_one(GemmArgs ga, const LinearW &w, const float *sx, const OutlierSet &os, const double *outl,
                      const OutDesc &o, const SessTable *sess, hipStream_t st) {
    constexpr int NSLOT = 4, BN = WVN * TN, BM = WVM * TM, QN = TN % 2 ? TN : TN / 2;   // a wave: 16 TN features x 16 TM tokens
    const int total = ga.nb_n * ga.nb_m * (EPI == EPI_PARTIAL ? ga.ksplit : 1);
    const size_t lds_stage = (size_t)NSLOT * (BN + BM) * 1024;
    const size_t lds_epi = (size_t)WVN * WVM * QN * TM * 1024 + (size_t)BN * 16 * 16 + (size_t)BN * 4 * 8 + (size_t)BN / 2 * 4;
    const size_t lds = lds_stage > lds_epi ? lds_stage : lds_epi;
    auto kern = k_gemm_lds<MODE, WVN, WVM, TN, TM, NSLOT, EPI>;
    static std::mutex attr_lock;
    static bool attr_set = false;
    {
        std::lock_guard<std::mutex> hold(attr_lock);
        if (!attr_set) {
            hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
    }
    kern<<<((total + 7) / 8) * 8, 64 * WVN * WVM, lds, st>>>(ga, w, sx, os, outl, o, sess);
    return hipGetLastError();
}

// The block forms of the int8 product: panels of 16 features x token tiles of 16.  What a launch takes, in microseconds,
// fitted to 310 linears (all four of blocks 1024 to 14336 wide, 80 to 4096 rows, every form; mean error 6 %, and the form it
// picks is 0.6 % behind the best one on average): workgroups go in rounds of 256 * resident; per k-tile a round takes
// stage + next * (further workgroups on the same unit), or its tiles at COPY if that is more; the first round costs `base` besides, a further one at least 2.
// What the rule is for: 256 compute units and few blocks.  With 256 x 128 blocks as the smallest, calls of 65 to 1500 rows
// left most of the units idle or split the contraction, which writes its sums and reads them again: 6144 x 2048 at 351 rows
// 51 us split, 34 in blocks of 128 x 128; 12288 x 4096 at 351 rows 64 -> 57 (96 x 192: 256 blocks instead of 144) and at 1400
// 142 -> 109 (192 x 192: 512 blocks instead of 288); 4096 x 1024 at 351 34 -> 28.  Deeper rings and another first k-tile
// for each workgroup cost all forms 1 to 15 %: it is neither latency nor memory channels that bound the stages of the small
// forms, but their copies (about 10 KB per microsecond and 256th of the chip) and the instructions around them.
struct BlockForm {
    int bn, bm, resident;
    double stage, next, base;
};
enum { FORM_16x16, FORM_16x8, FORM_12x12, FORM_6x12, FORM_8x8, FORM_4x4, FORMS };
constexpr BlockForm BLOCK_FORMS[FORMS] = {
    {16, 16, 1, 0.627, 0, 4.0}, {16, 8, 1, 0.438, 0, -0.9}, {12, 12, 1, 0.449, 0, 0.9},
    {6, 12, 1, 0.349, 0, -0.6}, {8, 8, 2, 0.320, 0.188, -1.0}, {4, 4, 1, 0.131, 0, -3.0},
};
constexpr double COPY = 16300;     // tiles per microsecond
constexpr int UNITS = 256;

int form_blocks(int form, int NT, int MTT) {
    const BlockForm &f = BLOCK_FORMS[form];
    return ((NT + f.bn - 1) / f.bn) * ((MTT + f.bm - 1) / f.bm);
}
double form_us(int form, int blocks, int ktiles) {
    const BlockForm &f = BLOCK_FORMS[form];
    const int cap = UNITS * f.resident, rounds = blocks / cap, rest = blocks % cap;
    auto round_us = [&](int n) { return ktiles * fmax(f.stage + f.next * ((n - 1) / UNITS), n * (f.bn + f.bm) / COPY); };
    return f.base + (rounds + (rest > 0) - 1) * fmax(f.base, 2.0) + rounds * round_us(cap) + (rest ? round_us(rest) : 0.0);
}

struct BlockPlan {
    int form, ksplit;       // ksplit > 1: FORM_16x8, the contraction split
    int tail_n;             // 256-feature blocks that go to a second launch in blocks of FORM_16x8
    double us;
};

// One workgroup per compute unit (128 KB of LDS): a launch of 256 x 256 blocks takes ceil(blocks / 256) rounds of
// equal length, and a last round that fills half of the units or less costs as much as a full one (896 blocks: 4
// rounds for the work of 3.5).  In that case the feature blocks of the last round can go to a second launch with
// blocks of half the token height, which fills all units for a shorter round (measured: 2 to 4 % of the linear's time;
// 4-wave workgroups with a 3-slot ring, two per unit, were slower).
int tail_blocks(int NT, int MTT) {
    const int nb_n = (NT + 15) / 16, nb_m = (MTT + 15) / 16, total = nb_n * nb_m, rest = total % UNITS;
    return total > UNITS && rest > 0 && rest <= UNITS / 2 && rest % nb_m == 0 ? rest / nb_m : 0;
}

// Workgroups that share the k-tiles of a 256 x 128 output block of a call that makes few blocks (351 rows of
// 4096 x 16384: 48 blocks on 256 compute units, 110 us; split five ways 32 us, and 9 us for
// adding up): as many as fill the compute units once, each with at least 16 k-tiles to walk.
int split_of(int NT, int ktiles, int MTT) {
    const int blocks = form_blocks(FORM_16x8, NT, MTT);
    return max(1, min(min(UNITS / blocks, ktiles / 16), PS_KSPLIT_MAX));
}

BlockPlan plan_blocks(int NT, int ktiles, int MTT, size_t part_bytes) {
    BlockPlan best = {FORM_16x16, 1, 0, form_us(FORM_16x16, form_blocks(FORM_16x16, NT, MTT), ktiles)};
    auto offer = [&](int form, int ksplit, int tail_n, double us) {
        if (us < best.us) best = {form, ksplit, tail_n, us};
    };
    if (const int tail = tail_blocks(NT, MTT))
        offer(FORM_16x16, 1, tail, form_us(FORM_16x16, form_blocks(FORM_16x16, NT - tail * 16, MTT), ktiles) +
                                   form_us(FORM_16x8, form_blocks(FORM_16x8, tail * 16, MTT), ktiles) + 2.0);
    for (int form = FORM_16x8; form < FORMS; form++) {
        const int blocks = form_blocks(form, NT, MTT);
        // 64 x 64: beyond one round, or with a long contraction, its times lie far above the estimate (8192 x 8192 at 80 rows
        // 58 us against 52 split)
        if (form == FORM_4x4 && (blocks > UNITS || ktiles > 64)) continue;
        offer(form, 1, 0, form_us(form, blocks, ktiles));
    }
    // split: the sums of all shares are written and read again (0.15 us per MB, and 11 us more from about 5 to 13 MB: the
    // kernels themselves hardly grow there, the gaps between them do); the weights stream at 5.6 TB/s at best
    int split = split_of(NT, ktiles, MTT);
    while (split > 1 && (size_t)split * NT * MTT * 1024 > part_bytes) split--;
    if (split > 1) {
        const double mb = 1.024e-3 * NT * MTT * split;
        const double share = (ktiles + split - 1) / split * fmax(0.485, split * form_blocks(FORM_16x8, NT, MTT) * 24 / COPY);
        offer(FORM_16x8, split, 0, -3.5 + 0.15 * mb + 11.4 * fmin(1.0, fmax(0.0, (mb - 5.0) / 8.0)) + fmax(share, NT * 1024.0 * ktiles / 5.6e6));
    }
    return best;
}

template <int MODE, int EPI>
hipError_t launch_form(int form, const GemmArgs &ga0, const LinearW &w, const float *sx, const OutlierSet &os, const double *outl,
                       const OutDesc &o, const SessTable *sess, hipStream_t st) {
    GemmArgs ga = ga0;
    const BlockForm &f = BLOCK_FORMS[form];
    if (!ga.nb_n) ga.nb_n = (ga.N / 16 + f.bn - 1) / f.bn;
    ga.nb_m = ((ga.M + 15) / 16 + f.bm - 1) / f.bm;
    if (form == FORM_16x16) return launch_one<MODE, 2, 4, 8, 4, EPI>(ga, w, sx, os, outl, o, sess, st);
    if (form == FORM_16x8) return launch_one<MODE, 4, 2, 4, 4, EPI>(ga, w, sx, os, outl, o, sess, st);
    if constexpr (MODE == GEMM_INT8) {
        if (form == FORM_12x12) return launch_one<MODE, 2, 4, 6, 3, EPI>(ga, w, sx, os, outl, o, sess, st);
        if (form == FORM_6x12) return launch_one<MODE, 2, 4, 3, 3, EPI>(ga, w, sx, os, outl, o, sess, st);
        if (form == FORM_8x8) return launch_one<MODE, 2, 4, 4, 2, EPI>(ga, w, sx, os, outl, o, sess, st);
        if (form == FORM_4x4) return launch_one<MODE, 2, 4, 2, 1, EPI>(ga, w, sx, os, outl, o, sess, st);
    }
    return hipErrorInvalidValue;
}
template <int MODE>
hipError_t launch_epi(int form, const GemmArgs &ga, const LinearW &w, const float *sx, const OutlierSet &os, const double *outl,
                      const OutDesc &o, const SessTable *sess, hipStream_t st) {
    if constexpr (MODE == GEMM_INT8) {
        if (o.epilogue == 1) return launch_form<MODE, 1>(form, ga, w, sx, os, outl, o, sess, st);
        if (o.epilogue == 2) return launch_form<MODE, 2>(form, ga, w, sx, os, outl, o, sess, st);
    }
    return launch_form<MODE, 0>(form, ga, w, sx, os, outl, o, sess, st);
}

template <int MODE>
hipError_t launch_lds(const GemmArgs &ga0, const LinearW &w, const float *sx, const OutlierSet &os, const double *outl,
                      const OutDesc &o, const SessTable *sess, hipStream_t st, size_t part_bytes = 0) {
    GemmArgs ga = ga0;
    const int NT = ga.N / 16, MTT = (ga.M + 15) / 16;
    ga.nb_n = ga.nb_n0 = 0;
    BlockPlan plan;
    if constexpr (MODE == GEMM_INT8) {
        plan = plan_blocks(NT, ga.ktiles, MTT, part_bytes);
        if (plan.ksplit > 1) {
            ga.ksplit = plan.ksplit;
            ga.nb_n = (NT + 15) / 16;
            ga.nb_m = (MTT + 7) / 8;
            hipError_t e = launch_one<MODE, 4, 2, 4, 4, EPI_PARTIAL>(ga, w, sx, os, outl, o, sess, st);
            if (e != hipSuccess) return e;
            k_split_finish<<<(NT * MTT + 3) / 4, 256, 0, st>>>(ga, w, sx, os, outl, o, sess);
            return hipGetLastError();
        }
    } else {
        // fp16 (the backward pass, 128 rows and more): blocks of half the height for at most 128 rows, or so few blocks
        // that half of the units would idle
        const bool half = MTT <= 8 || 2 * form_blocks(FORM_16x16, NT, MTT) <= UNITS;
        plan = {half ? FORM_16x8 : FORM_16x16, 1, half ? 0 : tail_blocks(NT, MTT), 0};
    }
    if (plan.tail_n) {
        GemmArgs gb = ga;
        gb.nb_n = plan.tail_n;
        ga.nb_n = (NT + 15) / 16 - plan.tail_n;
        gb.nb_n0 = ga.nb_n;
        hipError_t e = launch_epi<MODE>(FORM_16x16, ga, w, sx, os, outl, o, sess, st);
        if (e != hipSuccess) return e;
        return launch_epi<MODE>(FORM_16x8, gb, w, sx, os, outl, o, sess, st);
    }
    return launch_epi<MODE>(plan.form, ga, w, sx, os, outl, o, sess, st);
}

GemmArgs gemm_args(const void *a_tiles, const void *b_tiles, int ktiles, int M, int N) {
    GemmArgs g;
    memset(&g, 0, sizeof(g));
    g.a_tiles = (const unsigned char *)a_tiles;
    g.b_tiles = (const unsigned char *)b_tiles;
    g.ktiles = ktiles;
    g.M = M;
    g.N = N;
    g.exact = ps_exact_outliers(N, M);
    return g;
}

}  // namespace

// Rough microseconds of a linear of M rows in blocks with its row and digit kernels (see BLOCK_FORMS), to hold against the
// other forms of a call.
double ps_gemm_lds_us(int N, int K, int M) {
    const BlockPlan plan = plan_blocks(N / 16, K / 64, (M + 15) / 16, ~(size_t)0);
    return fmax(25.4 + 0.58e-6 * M * K + 1.4e-6 * M * N + plan.us, 25.0 + (double)N * K / 4.0e6);
}

hipError_t ps_gemm_f16_tiles(const __half *feat_tiles, const __half *tok_tiles, int ktiles, int M, int n_feat,
                             float *out, const __half *gelu_pre, __half *tile_out, hipStream_t st) {
    if (ktiles < 1 || M < 1 || n_feat < 16 || n_feat % 16) return hipErrorInvalidValue;
    if (gelu_pre && (!tile_out || n_feat % 32)) return hipErrorInvalidValue;
    GemmArgs ga = gemm_args(feat_tiles, tok_tiles, ktiles, M, n_feat);
    ga.gelu_pre = gelu_pre;
    ga.tile_out = tile_out;
    ga.f32_out = out;
    LinearW w;
    OutlierSet os;
    OutDesc o;
    memset(&w, 0, sizeof(w));
    memset(&os, 0, sizeof(os));
    memset(&o, 0, sizeof(o));
    return launch_lds<GEMM_F16>(ga, w, nullptr, os, nullptr, o, nullptr, st);
}

hipError_t ps_gemm_lds(const LinearW &w, const int8_t *xq_tiled, const uint32_t *mask, const __half *X, const float *sx,
                       int M, const OutlierSet &os, const ManyOutliers &mo, const OutDesc &o, const SessTable *sess,
                       hipStream_t st) {
    // The outlier-heavy case first (every kernel of it returns at once when the call has few outlier columns):
    // digit tiles of the activations and of the dequantized weights, the digit products.
    // (768 workgroups: those that are resident at once; twice as many cost a call that has nothing to cut 0.3 us more)
    // (a split product walks all columns: its sums go where the regular ones' codes would be)
    const bool split = plan_blocks(w.N / 16, w.K / 64, (M + 15) / 16, mo.wd_bytes).ksplit > 1;
    k_digit_tiles<<<768, 256, 0, st>>>(X, M, w, mask, (int *)os.count, mo.list, mo.xl, mo.wd, 1024, xq_tiled, split ? nullptr : mo.regular);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    GemmArgs gd = gemm_args(mo.wd, mo.xl, 0, M, w.N);
    gd.od = mo.od;
    gd.nb_n = (w.N / 16 + 7) / 8;                // 8 panels and 4 token tiles per block (times 2 digits, 4 planes)
    gd.nb_m = ((M + 15) / 16 + 3) / 4;
    e = launch_one<GEMM_DIGITS, 2, 4, 8, 4>(gd, w, sx, os, nullptr, o, sess, st);
    if (e != hipSuccess) return e;
    GemmArgs gi = gemm_args(w.wt, xq_tiled, w.K / 64, M, w.N);
    gi.a_regular = (const unsigned char *)mo.wd;
    gi.b_regular = (const unsigned char *)mo.xl;
    gi.part = (v4i *)mo.wd;                  // the digit tiles have been read when the int8 product starts
    return launch_lds<GEMM_INT8>(gi, w, sx, os, mo.od, o, sess, st, mo.wd_bytes);
}

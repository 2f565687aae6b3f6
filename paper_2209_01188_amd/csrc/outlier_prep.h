// Preparation of the outlier columns of a prefill-size linear, one wave at a time: part of the row quantizers' launch
// (it needs the column mask, the input rows and the weights, not the codes; as a launch of its own it cost 4.7 us per
// linear, whatever the data).
#pragma once
#include "epilogue.h"

struct OutlierPrep {
    LinearW w;
    int *count;          // null: nothing to prepare
    double *wd64, *x64;
    int *full_list;
};
// waves of work: one per 16 output rows, one per 16 tokens
__host__ __device__ inline int outlier_prep_items(const OutlierPrep &p, int M) { return p.count ? p.w.N / 16 + (M + 15) / 16 : 0; }

// Counts the outlier columns and, when there are at most PS_EXACT_OUTLIERS, gathers their
// dequantized weights (items [0, N/16)) and activations (the rest) as doubles in matrix-instruction lane order.
// Every wave rebuilds the short column list from the bit mask itself.  list: PS_EXACT_OUTLIERS ints of LDS of this wave.
__device__ __forceinline__ void outlier_prep_wave(const OutlierPrep &pr, const uint32_t *__restrict__ mask,
                                                  const __half *__restrict__ X, int M, int item, int *list) {
    const LinearW &w = pr.w;
    const int K = w.K, KT = K >> 6, nwords = K >> 5, lane = threadIdx.x & 63;
    const int wpt = (nwords + 63) / 64, w0 = min(nwords, lane * wpt), w1 = min(nwords, w0 + wpt);
    int cnt = 0;
    for (int i = w0; i < w1; i++) cnt += __popc(mask[i]);
    int incl = cnt;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int v = __shfl_up(incl, off);
        if (lane >= off) incl += v;
    }
    const int total = __shfl(incl, 63);
    if (item == 0 && lane == 0) { pr.count[0] = total; pr.count[1] = 4; }   // [1]: digit planes, raised by k_digit_tiles
    if (total > PS_EXACT_OUTLIERS && item == 0 && pr.full_list) {
        // more columns than the fp64 path takes: item 0 leaves their ascending list for the digit products,
        // padded with -1 up to the next multiple of 64
        int at = incl - cnt;
        for (int i = w0; i < w1; i++) {
            uint32_t b = mask[i];
            while (b) {
                const int j = __ffs(b) - 1;
                b &= b - 1;
                pr.full_list[at++] = i * 32 + j;
            }
        }
        const int padded = (total + 63) & ~63;
        for (int i = total + lane; i < padded; i += 64) pr.full_list[i] = -1;
    }
    if (total == 0 || total > PS_EXACT_OUTLIERS) return;
    int pos = incl - cnt;
    for (int i = w0; i < w1; i++) {
        uint32_t b = mask[i];
        while (b) {
            const int j = __ffs(b) - 1;
            b &= b - 1;
            list[pos++] = i * 32 + j;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int NT = w.N >> 4, row = lane & 15, kq = lane >> 4, nch = (total + 3) >> 2;
    if (item < NT) {
        // the fp64 matrix instruction returns row 4r + g in register r of lane group g, the int8 one
        // row 4g + r: store the weight rows permuted so both results line up in the same registers
        const int nt = item, nrow = 4 * (row & 3) + (row >> 2);
        const float swd = w.sw[nt * 16 + nrow] / 127.0f;
        for (int c = 0; c < nch; c++) {
            const int j = c * 4 + kq;
            double v = 0.0;
            if (j < total) {
                const int k = list[j];
                const int code = w.wt[((size_t)nt * KT + (k >> 6)) * 1024 + (((k & 63) >> 4) * 16 + nrow) * 16 + (k & 15)];
                v = (double)dequant_w16(code, swd);
            }
            pr.wd64[((size_t)nt * PS_OUTLIER_CHUNKS + c) * 64 + lane] = v;
        }
    } else {
        const int mt = item - NT, t = mt * 16 + row;
        for (int c = 0; c < nch; c++) {
            const int j = c * 4 + kq;
            double v = 0.0;
            if (j < total && t < M) v = (double)__half2float(X[(size_t)t * K + list[j]]);
            pr.x64[((size_t)mt * PS_OUTLIER_CHUNKS + c) * 64 + lane] = v;
        }
    }
}

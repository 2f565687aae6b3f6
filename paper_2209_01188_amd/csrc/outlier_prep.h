// Preparation of the outlier columns of a prefill-size linear, one wave at a time: part of the row quantizers' launch
// (it needs the column mask, the input rows and the weights, not the codes; as a launch of its own it cost 4.7 us per
// linear, whatever the data).
#pragma once
#include "epilogue.h"

struct OutlierPrep {
    LinearW w;
    int *count;          // null: nothing to prepare
    double *wd64, *x64;
    int *full_list, *regular_list;
};
// waves of work: one per 16 output rows and one per 16 tokens, and no fewer than the list has groups of 1024 columns (an
// output of 64 rows has four panels, its 65536 columns 64 groups)
__host__ __device__ inline int outlier_prep_items(const OutlierPrep &p, int M) {
    const int gathers = p.w.N / 16 + (M + 15) / 16, groups = (p.w.K + 1023) / 1024;
    return !p.count ? 0 : gathers > groups ? gathers : groups;
}

// Counts the outlier columns and, when there are at most ps_exact_outliers, gathers their
// dequantized weights (items [0, N/16)) and activations (the next ceil(M/16)) as doubles in matrix-instruction lane order.
// Every wave rebuilds the short column list from the bit mask itself.  list: PS_EXACT_OUTLIERS ints of LDS of this wave.
__device__ __forceinline__ void outlier_prep_wave(const OutlierPrep &pr, const uint32_t *__restrict__ mask, const uint8_t *__restrict__ flags,
                                                  const __half *__restrict__ X, int M, int item, int *list) {
    const LinearW &w = pr.w;
    // 16 columns per lane and step: groups of 1024 consecutive columns per wave, at most 64 of them (K <= 65536)
    const int K = w.K, KT = K >> 6, nchunk = K >> 4, lane = threadIdx.x & 63;
    auto chunk = [&](int c) -> uint32_t { return c < nchunk ? chunk_outliers(mask, flags, c) : 0u; };
    const auto sum = [](uint32_t a, uint32_t b) { return a + b; };
    uint32_t cnt = 0, before = 0;          // outlier columns in all groups, and in those in front of group `item`
    uint64_t used = 0;                     // groups that hold any
    for (int g0 = 0; g0 * 64 < nchunk; g0 += 8) {
        uint32_t b[8];
#pragma unroll
        for (int i = 0; i < 8; i++) b[i] = chunk((g0 + i) * 64 + lane);     // all requested before the first is looked at
#pragma unroll
        for (int i = 0; i < 8; i++) {
            cnt += __popc(b[i]);
            if (g0 + i < item) before += __popc(b[i]);
            used |= (uint64_t)(__ballot(b[i] != 0) != 0) << (g0 + i);
        }
    }
    const int total = (int)wave_reduce(cnt, 0u, sum);
    if (item == 0 && lane == 0) { pr.count[0] = total; pr.count[1] = 4; }   // [1]: digit planes, raised by k_digit_tiles
    const auto lanes_before = [&](uint32_t b) {     // of this lane's columns in its group
        const int n = __popc(b);
        int incl = n;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(incl, off);
            if (lane >= off) incl += v;
        }
        return incl - n;
    };
    if (total > ps_exact_outliers(w.N, M)) {
        // more columns than the fp64 path takes: their ascending list for the digit products, each group's part by the wave
        // of that number, padded with -1 up to the next multiple of 64.  (The whole list by one wave was what this launch
        // waited for: 200 rows of 32768 with 500 outlier columns 17 us.)
        if (item * 64 >= nchunk || !pr.full_list) return;
        uint32_t b = chunk(item * 64 + lane);
        int at = (int)wave_reduce(before, 0u, sum) + lanes_before(b);
        if (ps_regular_compacted(total, K, M)) {
            const int k0 = (item * 64 + lane) * 16;
            int to = k0 - at;
            if (k0 < K)
                for (int e = 0; e < 16; e++)
                    if (!((b >> e) & 1u)) pr.regular_list[to++] = k0 + e;
            if (item == 0 && lane < ((total - K) & 63)) pr.regular_list[K - total + lane] = -1;
        }
        while (b) {
            pr.full_list[at++] = (item * 64 + lane) * 16 + __ffs(b) - 1;
            b &= b - 1;
        }
        if (item == 0)
            for (int i = total + lane; i < ((total + 63) & ~63); i += 64) pr.full_list[i] = -1;
        return;
    }
    if (total == 0 || item >= (w.N >> 4) + ((M + 15) >> 4)) return;
    int base = 0;
    for (; used; used &= used - 1) {
        const int c = (__ffsll((unsigned long long)used) - 1) * 64 + lane;
        uint32_t b = chunk(c);
        int at = base + lanes_before(b);
        base += (int)wave_reduce((uint32_t)__popc(b), 0u, sum);
        while (b) {
            list[at++] = c * 16 + __ffs(b) - 1;
            b &= b - 1;
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

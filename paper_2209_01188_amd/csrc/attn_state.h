// Online softmax states of a decode attention: what the lane groups of a wave, and then the waves of a workgroup, have made of
// their keys.  head_dim / 8 = LPK neighbouring lanes share a key, lane `sub` of them holds dims 8 sub .. 8 sub + 8 of the sums o.
#pragma once
#include "common.h"

// One step of summing pairs of values over lanes 32, 16 or 8 apart: of a and b each half of the lanes is left with one (lanes
// with the bit set: b) - half the exchanges of summing both in all lanes.
template <int DIST>
__device__ __forceinline__ double sum_scatter(double a, double b) {
    const uint64_t ua = (uint64_t)__double_as_longlong(a), ub = (uint64_t)__double_as_longlong(b);
    if constexpr (DIST == 8) {
        const bool odd = threadIdx.x & 8;
        const double keep = odd ? b : a, send = odd ? a : b;
        return keep + dpp_move<0x128, 0xf>(send, send);              // row_ror 8
    } else {
        uint32_t x[2], y[2];
        if constexpr (DIST == 16) {
            const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)ua, (uint32_t)ub, false, false);
            const auto h = __builtin_amdgcn_permlane16_swap((uint32_t)(ua >> 32), (uint32_t)(ub >> 32), false, false);
            x[0] = l[0]; x[1] = h[0]; y[0] = l[1]; y[1] = h[1];
        } else {
            const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)ua, (uint32_t)ub, false, false);
            const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)(ua >> 32), (uint32_t)(ub >> 32), false, false);
            x[0] = l[0]; x[1] = h[0]; y[0] = l[1]; y[1] = h[1];
        }
        return __longlong_as_double((long long)((uint64_t)x[1] << 32 | x[0])) + __longlong_as_double((long long)((uint64_t)y[1] << 32 | y[0]));
    }
}

// The lane groups of a wave: its maximum first (m), then every group's sums scaled to it and added up (l in all lanes).  Of the
// sums over the keys every lane is left with LPK / 8 dims (one, from LPK = 8 down): those from merged_dim on.
template <int LPK>
__device__ __forceinline__ int merged_dim(int lane) {
    const int e = (lane >> 5 & 1) * 4 + (lane >> 4 & 1) * 2 + (LPK <= 8 ? lane >> 3 & 1 : 0);
    return lane % LPK * 8 + e;
}
template <int LPK>
__device__ __forceinline__ void merge_wave(double &m, double &l, double (&o)[8]) {
    double mw = m;
#pragma unroll
    for (int off = LPK; off < 8; off <<= 1) mw = fmax(mw, __shfl_xor(mw, off));
    if constexpr (LPK <= 8) mw = fmax(mw, dpp_move<0x128, 0xf>(mw, mw));
    mw = swap_reduce<32>(swap_reduce<16>(mw, max_f64), max_f64);
    const double f = (m == -INFINITY) ? 0.0 : exp_f64(m - mw);
    m = mw;
    l *= f;
#pragma unroll
    for (int off = LPK; off < 8; off <<= 1) l += __shfl_xor(l, off);
    if constexpr (LPK <= 8) l += dpp_move<0x128, 0xf>(l, l);
    l = swap_reduce<32>(swap_reduce<16>(l, add_f64), add_f64);
#pragma unroll
    for (int e = 0; e < 8; e++) {
        o[e] *= f;
#pragma unroll
        for (int off = LPK; off < 8; off <<= 1) o[e] += __shfl_xor(o[e], off);
    }
#pragma unroll
    for (int e = 0; e < 4; e++) o[e] = sum_scatter<32>(o[e], o[e + 4]);
#pragma unroll
    for (int e = 0; e < 2; e++) o[e] = sum_scatter<16>(o[e], o[e + 2]);
    if constexpr (LPK <= 8) o[0] = sum_scatter<8>(o[0], o[1]);
}

// The waves of a workgroup, from LDS: maximum m, denominator l and the sum over the keys of dim `dim` (one per lane).  Lane i of
// every NW scales the sums of wave i: one exponential instead of NW in a row.
template <int NW, int D>
__device__ __forceinline__ double merge_waves(const double (&red_m)[NW], const double (&red_l)[NW], const double (&red_o)[NW][D], int lane,
                                              int dim, double &m, double &l) {
    const double mine = red_m[lane % NW];
    m = group_reduce<NW>(mine, max_f64);
    const double f = (mine == -INFINITY) ? 0.0 : exp_f64(mine - m);
    l = group_reduce<NW>(f * red_l[lane % NW], add_f64);
    double o = 0.0;
    auto add = [&](auto wc) {
        constexpr int w = decltype(wc)::value;
        double fw;
        if constexpr (NW == 8) fw = group_bcast<8, w>(f);
        else fw = dpp_move<w * 0x55, 0xf>(f, f);                     // quad_perm w w w w
        o += fw * red_o[w][dim];
    };
    static_assert(NW == 4 || NW == 8, "lanes of a quad or of half a row");
    for_constants(add, std::make_integer_sequence<int, NW>());
    return o;
}

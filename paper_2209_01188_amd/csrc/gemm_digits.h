// Linear of 17 to 64 rows whose input has many outlier columns (the attention context and the GeLU output of a wide
// block: a third of 14336 and of 57344 columns at 32 rows).  The regular columns as in gemm.hip; the fp16 x fp16 product
// over the outlier columns exactly on the int8 matrix instruction, in the same pass over the weights: activations as four
// balanced 8-bit digits (written by the row quantizer, zero in regular columns), dequantized weights as
// u_n (m_n code + r) with the int8 code itself and a remainder r of 8 bits worked out in registers (see gemm_lds.hip).
//
// In gemm.hip every outlier column costs a 64-clock fp64 matrix instruction per panel and token tile (4 columns at a
// time); here a 64-column tile costs eight 16-clock int8 instructions per token tile and 80 vector instructions for its
// remainders, however many of its columns are outliers.
#pragma once
#include "digits.h"
#include "epilogue.h"

namespace {

constexpr int DIGIT_PAIRS = 8;        // waves of a workgroup, each with a pair of 16-row panels
constexpr int DIGIT_SLOTS = 6;        // of 10 KB of the LDS ring
typedef int v16i __attribute__((ext_vector_type(16)));

__device__ __forceinline__ v4i buffer_load16(const __amdgpu_buffer_rsrc_t r, int lane_offset, int offset) {
    const auto x = __builtin_amdgcn_raw_buffer_load_b128(r, lane_offset, offset, 2 /* non-temporal */);
    return (v4i){(int)x[0], (int)x[1], (int)x[2], (int)x[3]};
}
__device__ __forceinline__ void buffer_copy16(const __amdgpu_buffer_rsrc_t r, void *lds, int lane_offset, int offset) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)lds, 16, lane_offset, offset, 0, 0);
}

// One workgroup: 256 output rows, 32 tokens, and one of PS_DIGIT_SPLITS shares of the contraction.  A wave owns 32 output
// rows; its nine sums (v_mfma_i32_32x32x32_i8: 16 registers each, at most 2^14 * 2^16 = 2^30) stay in registers to the end.
// Bound by the matrix unit at the clock that such operands leave it (14336 x 57344, 32 rows: its products alone 185 us, with
// the remainders 248; the weights 130) once the digits reach LDS fast enough: a step has ten times as many bytes of them as
// of weights per 16 rows, so the more output rows share them the better, and the compute units are filled by splitting the
// contraction over workgroups, not the output (64 output rows and the whole contraction per workgroup 302 us, 128 and half
// of it 265, 256 and a quarter 248; the fp64 form 458 on the outlier columns of a decode step).
// Codes and digits move through an LDS ring filled by asynchronous copies, NSLOT - 1 steps ahead, the weights go straight to
// registers, PW steps ahead; while step s is multiplied, the fragments of step s + 1 are read into the registers they
// replace and its remainders are worked out.
// Tiles are 16 rows x 64 columns, see LinearW; lane l takes row l % 16 of panel (or token tile) (l / 16) % 2 and column
// group l / 32 + 2 h for instruction h of a step.
// Of the PS_DIGIT_SPLITS waves that share a pair of panels, the one that gets there last adds the sums, always in the same
// order, and goes through the linear's tail.  (While this form and the tails were launches of their own, a call that does not come
// here paid 2 us for either: dense of a 14336-wide block with few outlier columns, 24 rows, 47.6 us in the fp64 form alone, 49.7
// with them, 48.3 with all in one launch; with a third outlier columns 89.3 and 91.1 at 32 rows, 157 and 156 at 64.)  The sums
// pass between compute units, most of them on other XCDs, by relaxed agent-scope atomics, which are written through and read
// past the L2s, and every store has been acknowledged before the count goes up.  Plain stores with a release and an acquire
// would do as well, for 10 us more per linear: each has its L2 written back or dropped as a whole.
__host__ __device__ inline int digit_grid_x(int N, int M) {
    const int wgs = (N / 32 + DIGIT_PAIRS - 1) / DIGIT_PAIRS;
    return M > 32 ? (wgs + 7) / 8 * 16 : wgs;
}
__device__ __forceinline__ void digit_linear(const LinearW &w, const int8_t *__restrict__ xq_tiled, const uint32_t *__restrict__ mask,
                                             const __half *__restrict__ X, const float *__restrict__ sx, int M, const OutDesc &o,
                                             const SessTable *__restrict__ sess, const DigitCall &dc, unsigned char *lds) {
    constexpr int NSLOT = DIGIT_SLOTS, PAIRS = DIGIT_PAIRS, TOK = 10, PD = NSLOT - 1, PW = 3, MORE = TOK - PAIRS;
    const int lane = threadIdx.x & 63;
    const int KT = w.K >> 6, pairs = w.N >> 5, MTT = (M + 15) >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    // 33 rows and more: the two halves of the tokens in workgroups 8 apart, that is on one XCD, whose L2 then gives the
    // weights to the second one
    const int share = (int)blockIdx.x / digit_grid_x(w.N, M);
    int bx = (int)blockIdx.x - share * digit_grid_x(w.N, M), half = 0;
    if (M > 32) {
        half = (bx >> 3) & 1;
        bx = (bx >> 4) * 8 + (bx & 7);
    }
    if (share >= PS_DIGIT_SPLITS || bx * PAIRS >= pairs) return;
    const int pair = min(bx * PAIRS + wave, pairs - 1);
    const int k_first = KT * share / PS_DIGIT_SPLITS, NS = KT * (share + 1) / PS_DIGIT_SPLITS - k_first;

    // Buffer form of the requests: descriptor = the run of tiles, bounds-checked by the hardware, and no address arithmetic in
    // the vector unit; with the flat form of the copies the compiler waits for ALL requests wherever it waits for weights.
    const __amdgpu_buffer_rsrc_t src_w = __builtin_amdgcn_make_buffer_rsrc((void *)(w.wt + ((size_t)pair * 2 * KT + k_first) * 1024), 0,
                                                                            (KT + NS) * 1024, 0x00020000);
    const int lane_tile = ((lane & 15) + 16 * (lane >> 5)) * 16, second = (lane >> 4) & 1;
    const int lane_w = second * KT * 1024 + lane_tile, lane_t = second * 5 * 1024 + lane_tile;
    // this wave's part of the ten tiles (per token tile: codes, four digit planes): tile `wave`, waves 0 and 1 also tile 8 + wave
    __amdgpu_buffer_rsrc_t src_t[2];
    int step_t[2];
    const bool more = wave < MORE;
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const int s = min(wave + PAIRS * i, TOK - 1), mt = min(half * 2 + s / 5, MTT - 1), j = s % 5;
        const int8_t *p = j == 0 ? xq_tiled + ((size_t)mt * KT + k_first) * 1024 : dc.xd + (((size_t)mt * KT + k_first) * 4 + (j - 1)) * 1024;
        step_t[i] = j == 0 ? 1024 : 4096;
        src_t[i] = __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, (NS - 1) * step_t[i] + 1024, 0x00020000);
    }
    auto request_w = [&](int s, v4i *wt) {           // steps beyond the last read it again: every wait counts the same
        const int at = min(s, NS - 1) * 1024;
        wt[0] = buffer_load16(src_w, lane_w, at);
        wt[1] = buffer_load16(src_w, lane_w, at + 512);
    };
    auto request_t = [&](int s) {
        const int at = min(s, NS - 1);
        unsigned char *slot = lds + ((s % NSLOT) * TOK + wave) * 1024;
        buffer_copy16(src_t[0], slot, lane * 16, at * step_t[0]);
        if (more) buffer_copy16(src_t[1], slot + PAIRS * 1024, lane * 16, at * step_t[1]);
    };
    auto wait = [&](auto steps) {                    // all but the requests of the last `steps` steps have landed
        constexpr int n = decltype(steps)::value;
        if (more) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(n * 4) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(n * 3) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    auto read_t = [&](int s, int h, int i) {
        return *(const v4i *)(lds + ((s % NSLOT) * TOK + i) * 1024 + lane_t + h * 512);
    };

    float a;
    int E, m;
    digit_scale(w.sw[pair * 32 + (lane & 31)], a, E, m);
    const _Float16 mu = (_Float16)a, magic = (_Float16)ldexpf(1.5f, E);     // 1536 u = 1.5 * 2^E
    v16i acc, ac[4], ar[4];
#pragma unroll
    for (int r = 0; r < 16; r++) {
        acc[r] = 0;
#pragma unroll
        for (int d = 0; d < 4; d++) ac[d][r] = ar[d][r] = 0;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // from here on only the requests below are counted
    v4i wq[PW][2], x[2][5], rem0[2], rem1[2];              // weights of step i in wq[i % PW]
#pragma unroll
    for (int s = 0; s < PD - PW; s++) request_t(s);
#pragma unroll
    for (int s = 0; s < PW; s++) {
        request_t(PD - PW + s);
        request_w(s, wq[s]);
    }
    wait(std::integral_constant<int, 0>());
#pragma unroll
    for (int h = 0; h < 2; h++) {
#pragma unroll
        for (int i = 0; i < 5; i++) x[h][i] = read_t(0, h, i);
        rem0[h] = digit_remainders(wq[0][h], a, mu, magic);
    }
    // the products of a step; next >= 0: every fragment is replaced by that of step `next` after its use
    auto multiply = [&](const v4i *wt, const v4i *rem, int next) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(wt[h], x[h][0], acc, 0, 0, 0);
            if (next >= 0) x[h][0] = read_t(next, h, 0);
#pragma unroll
            for (int d = 0; d < 4; d++) {
                ac[d] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wt[h], x[h][1 + d], ac[d], 0, 0, 0);
                ar[d] = __builtin_amdgcn_mfma_i32_32x32x32_i8(rem[h], x[h][1 + d], ar[d], 0, 0, 0);
                if (next >= 0) x[h][1 + d] = read_t(next, h, 1 + d);
            }
        }
    };
    // step s from (wt, rem); the remainders of step s + 1 from nwt into nrem; wt then takes step s + PW
    auto step = [&](int s, v4i *wt, const v4i *rem, const v4i *nwt, v4i *nrem) {
        wait(std::integral_constant<int, (PD - 2 < 5 ? PD - 2 : 5)>());   // step s + 1 has landed, and everybody has read step s - 1
        request_t(s + PD);
        multiply(wt, rem, s + 1);
#pragma unroll
        for (int h = 0; h < 2; h++) {
            nrem[h] = digit_remainders(nwt[h], a, mu, magic);
            asm volatile("" : "+v"(nrem[h][0]), "+v"(nrem[h][1]), "+v"(nrem[h][2]), "+v"(nrem[h][3]));   // here, not in front of their use
        }
#pragma unroll
        for (int i = 0; i < 18; i++) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                    // one matrix instruction,
            if (i != 1 && i != 3 && i != 5 && i != 7 && i != 10 && i != 12 && i != 14 && i != 16)
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                // a read of local memory behind the last use,
            __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);                    // seven vector instructions
        }
        __builtin_amdgcn_sched_barrier(0);
        request_w(s + PW, wt);           // into the registers it replaces (requested any earlier they are copied, and waited for)
        __builtin_amdgcn_sched_barrier(0);
    };
    int s = 0;
    for (; s + 6 < NS; s += 6) {
        step(s, wq[0], rem0, wq[1], rem1);
        step(s + 1, wq[1], rem1, wq[2], rem0);
        step(s + 2, wq[2], rem0, wq[0], rem1);
        step(s + 3, wq[0], rem1, wq[1], rem0);
        step(s + 4, wq[1], rem0, wq[2], rem1);
        step(s + 5, wq[2], rem1, wq[0], rem0);
    }
    // the last 1 to 6 steps, one at a time: the weights and remainders of the current one in wq[0] and rem0
    for (; s + 1 < NS; s++) {
        step(s, wq[0], rem0, wq[1], rem1);
        const v4i t[2] = {wq[0][0], wq[0][1]};
#pragma unroll
        for (int h = 0; h < 2; h++) { wq[0][h] = wq[1][h]; wq[1][h] = wq[2][h]; wq[2][h] = t[h]; rem0[h] = rem1[h]; }
    }
    multiply(wq[0], rem0, -1);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the copies beyond the end have landed, too

    // m sum_j 256^j A_code[j] + sum_j 256^j A_rem[j] in fp64 from the top digit down: exact below 2^53, i.e. up to the last
    // step.  Register 4 q + r of lane l is output row 8 q + 4 (l / 32) + r of the pair, token l % 32.
    if (bx * PAIRS + wave >= pairs) return;
    const size_t at = ((size_t)half * pairs + pair) * 16 * 64 + lane, split = (size_t)2 * pairs * 16 * 64;
    double own[16];
#pragma unroll
    for (int r = 0; r < 16; r++) {
        const int m1 = __shfl(m, 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3));      // lane n holds the scale of row n
        double tc = 0.0, tr = 0.0;
#pragma unroll
        for (int d = 3; d >= 0; d--) { tc = tc * 256.0 + (double)ac[d][r]; tr = tr * 256.0 + (double)ar[d][r]; }
        own[r] = fma((double)m1, tc, tr);
        __hip_atomic_store(dc.part + share * split + at + r * 64, own[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(dc.part_acc + share * split + at + r * 64, acc[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // they are where everybody sees them
    int before = 0;
    if (lane == 0) before = __hip_atomic_fetch_add(dc.done + half * (PS_DIGIT_DONE / 2) + pair, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane(before) != PS_DIGIT_SPLITS - 1) return;
    asm volatile("" ::: "memory");                         // no load in front of the count
    const int t = half * 32 + (lane & 31);
    const float sw = w.sw[pair * 32 + (lane & 31)];
    digit_scale(sw, a, E, m);
    const bool overflow = __any(!(sw <= 65504.0f));        // some |Wd| of such a row may overflow fp16
    int e[16];
#pragma unroll
    for (int r = 0; r < 16; r++) e[r] = __shfl(E, 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) - 34;    // u = 2^(E-10), activations in units of 2^-24
    if (t >= M) return;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const int n0 = pair * 32 + 8 * q + 4 * (lane >> 5);
        v4i sum;
        v4d od;
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const size_t i = at + (4 * q + r) * 64;
            const auto other = [&](int j) { return (j + (j >= share)) * split + i; };
            const auto part = [&](int j) { return __hip_atomic_load(dc.part + other(j), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
            const auto part_acc = [&](int j) { return __hip_atomic_load(dc.part_acc + other(j), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
            static_assert(PS_DIGIT_SPLITS == 4, "");
            const double p0 = part(0), p1 = part(1), p2 = part(2), p = own[4 * q + r];
            sum[r] = acc[4 * q + r] + part_acc(0) + part_acc(1) + part_acc(2);
            od[r] = share == 0 ? p : p0;               // in the order of the shares, its own in its place
            od[r] += share == 0 ? p0 : share == 1 ? p : p1;
            od[r] += share <= 1 ? p1 : share == 2 ? p : p2;
            od[r] += share == 3 ? p : p2;
        }
#pragma unroll
        for (int r = 0; r < 4; r++) od[r] = __builtin_amdgcn_ldexp(od[r], e[4 * q + r]);
        if (overflow) {                                    // column by column, infinities and all
            for (int r = 0; r < 4; r++) {
                const int n = n0 + r;
                if (w.sw[n] <= 65504.0f) continue;
                double v = 0.0;
                for (int kw = 0; kw < w.K >> 5; kw++)
                    for (uint32_t b = mask[kw]; b; b &= b - 1) {
                        const int k = kw * 32 + __ffs(b) - 1;
                        const int code = w.wt[((size_t)(n >> 4) * KT + (k >> 6)) * 1024 + (((k & 63) >> 4) * 16 + (n & 15)) * 16 + (k & 15)];
                        v += (double)__half2float(X[(size_t)t * w.K + k]) * (double)dequant_w16(code, w.sw[n] / 127.0f);
                    }
#pragma unroll
                for (int i = 0; i < 4; i++) od[i] = i == r ? v : od[i];
            }
        }
        emit_output4(o, sess, w.N, t, n0, sum, od, sx[t] / 127.0f, w.sw, w.bias);
    }
}

}  // namespace

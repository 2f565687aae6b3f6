// One token of ONE session through all blocks of a narrow span in a single launch.
//
// As separate launches (five per block: QKV, attention, dense, up, down) such a step is bound by the launches themselves: 2.6 us
// each from a stream whatever they do, and behind that the latency of the row, of weights that nobody asked for before, of the
// operands of the tail, 5 us a launch for some 0.5 us of arithmetic.  Here workgroups take work items (a few 16-row panels of a
// linear, or one head's attention over a range of keys) from a counter, request the item's weights or cached keys, and wait for
// the item's input row.  24 blocks of 1024 columns, 128 keys: 618 -> 382 us a step; 8 blocks of 2048 columns 271 -> 175, 8 of
// 1024 with 1000 keys 257 -> 188.  What is left of a stage, 3 us: 0.7 until its row is seen, 1.1 for LayerNorm and codes, 0.4 for
// the products, 0.5 for the reduction and the tail.
//
// One workgroup per compute unit, 256 in all: a stage has 16 (attention of 16 heads) to 256 items (QKV, dense, up and down of 4096
// columns), so those of the next stages are waited for, with their weights on the way, by the workgroups that have none of
// this one.  (Two per unit: 41 spilled registers; and with 512 workgroups polling the words' few memory channels the stores to
// them starved, 42 ms a step.  The next item's number taken while an item is worked on: workgroups end up with two items of a
// stage, 567 us.)
//
// Rows go from workgroup to workgroup as 32-bit words in device memory: the fp16 value in the low half, the number of the
// block (counted from 1) in the high half, written and read by relaxed atomics of agent scope, which every XCD sees.  A reader
// polls the words themselves, so waiting for a row and loading it are one.
//
// No deadlock, whatever part of the grid is resident and whatever else the GPU runs: items are numbered in the order of the
// data flow, an item only waits for items of smaller numbers, and numbers are handed out in order to workgroups that are
// running and done with their last.  The item with the smallest number among the unfinished ones is always being worked on
// and has nothing left to wait for.
//
// One set of words serves all blocks: a word is overwritten only behind everything that reads it.  E.g. the words of x1 of
// block b + 1 need all of the contexts of b + 1, these all of x of b + 1, these all panels of down of b, each of which has
// read the residual from x1 of b before it published anything, and all of the GeLU outputs of b, whose panels have read x1 of b.
#include "attn_state.h"
#include "common.h"
#include "epilogue.h"

namespace {

constexpr int THREADS = 512, WAVES = 8;
// Every wait ends (see above); so that a defect cannot hang the GPU all the same, a reader gives up after s.patience polls and
// tells the others; the values that it did not get count as NaN, which the layers carry into the output.  (Polls, not time: a
// call that something else keeps off the GPU for long doesn't poll meanwhile.)  Counted here, as nothing else outlives the call.
static __device__ int d_given_up;
__global__ void k_given_up(int *out) { *out = __hip_atomic_load(&d_given_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

static __device__ const CodeTable d_code_table = ps_make_code_table();

__device__ __forceinline__ uint64_t load_words2(const uint32_t *p) {
    return __hip_atomic_load((const uint64_t *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish(uint32_t *p, uint32_t tag, __half v) {
    __hip_atomic_store(p, tag << 16 | __half_as_ushort(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// N pairs of words into packed halves, once all of them carry the tag.  STEP > 1: every STEP-th pair is polled before all of them
// are (a thread's consecutive words were stored together): the polling of wide rows keeps the words' memory channels busy.
template <int N, int STEP = 1>
__device__ __forceinline__ void await_words(const uint32_t *const (&p)[N], uint32_t tag, int (&out)[N], const StepArgs &s) {
    const uint64_t want = (uint64_t)(tag << 16) << 32 | tag << 16;
    int *gave_up = s.ticket + 1;
    for (uint32_t spins = 0;; spins++) {
        uint64_t w[N], off = 0;
        if constexpr (STEP > 1) {
#pragma unroll
            for (int i = 0; i < N; i += STEP) w[i] = load_words2(p[i]);
#pragma unroll
            for (int i = 0; i < N; i += STEP) off |= w[i] ^ want;
        }
        if (!(off & 0xffff0000ffff0000ull)) {
#pragma unroll
            for (int i = 0; i < N; i++) w[i] = load_words2(p[i]);
#pragma unroll
            for (int i = 0; i < N; i++) {
                off |= w[i] ^ want;
                out[i] = (int)__builtin_amdgcn_perm((uint32_t)(w[i] >> 32), (uint32_t)w[i], 0x05040100);
            }
            if (!(off & 0xffff0000ffff0000ull)) return;
        }
        __builtin_amdgcn_s_sleep(1);
        if ((spins & 1023) == 1023 && __hip_atomic_load(gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
        if (spins >= s.patience) {
            if (!__hip_atomic_exchange(gave_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicAdd(&d_given_up, 1);
            break;
        }
    }
#pragma unroll
    for (int i = 0; i < N; i++) out[i] = 0x7e007e00;
}

// Waits, with one lane and pauses, until the stage before an item's own has something to work on: the rows are polled only by
// the workgroups whose turn is next, not by all that wait (with everybody polling, the words' few memory channels are so
// busy that the stores to them starve).  p may be null.
__device__ __forceinline__ void await_turn(const uint32_t *p, uint32_t tag, int tid, const StepArgs &s) {
    if (!p) return;
    if (tid == 0) {
        for (uint32_t spins = 0; __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> 16 != tag && spins < s.patience; spins++) {
            __builtin_amdgcn_s_sleep(8);
            if ((spins & 1023) == 1023 && __hip_atomic_load(s.ticket + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
        }
    }
    lds_barrier();
}

// What the workgroups pass on: words in device memory
struct Words {
    uint32_t *x, *qkv, *ctx, *x1, *g;
};

template <int CW, int D>
struct Lds {
    static constexpr int KMAX = 2048 * CW;           // widest row
    __align__(16) int8_t codes[KMAX];
    union {
        __align__(16) __half row[KMAX];              // the values that were quantized, for outlier columns
        double ao[WAVES][D];                         // attention: the waves' sums
    };
    uint16_t mask[KMAX / 16];                        // outlier columns of each 16
    double sum[WAVES], sq[WAVES], red_f[WAVES][64], am[WAVES], al[WAVES];
    int mx[WAVES], red_i[WAVES][64];
    int next, last;
};

__device__ __forceinline__ float low_half(int w) { return __half2float(__ushort_as_half((unsigned short)(w & 0xffff))); }
__device__ __forceinline__ float high_half(int w) { return __half2float(__ushort_as_half((unsigned short)((uint32_t)w >> 16))); }

// The row of a linear into codes, values and outlier masks in LDS, every thread CT consecutive columns NCH times; returns
// the largest regular magnitude.  The arithmetic is that of the one-row kernel (LayerNorm in fp64, row scale and codes in
// fp32).
template <bool LN, int CT, int NCH, int CW, int D>
__device__ __forceinline__ float prepare_row(Lds<CW, D> &l, int tid, int K, const StepArgs &s, const __half *plain, bool coded, const uint32_t *words,
                                             uint32_t tag, const __half *gain, const __half *bias) {
    constexpr int NP = CT / 2;                       // pairs of columns of a chunk
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    int v[NCH][NP], gr[LN ? NP : 1], br[LN ? NP : 1];
    static_assert(!LN || NCH == 1, "a LayerNorm's row is one chunk per thread");
    const bool mine0 = (int)tid * CT < K;
    if constexpr (LN) {
        const int c = mine0 ? tid * CT : 0;
#pragma unroll
        for (int e = 0; e < NP; e++) { gr[e] = *(const int *)(gain + c + 2 * e); br[e] = *(const int *)(bias + c + 2 * e); }
    }
    if (words) {
        const uint32_t *p[NCH * NP];
#pragma unroll
        for (int i = 0; i < NCH; i++) {
            const int c = (tid + THREADS * i) * CT;
#pragma unroll
            for (int e = 0; e < NP; e++) p[i * NP + e] = words + (c < K ? c : 0) + 2 * e;
        }
        if (mine0) await_words<NCH * NP, (CW == 8 ? NP : 1)>(p, tag, *(int(*)[NCH * NP])v, s);
    }
#pragma unroll
    for (int i = 0; i < NCH; i++) {
        const int c = (tid + THREADS * i) * CT;
        if (c >= K) {
#pragma unroll
            for (int e = 0; e < NP; e++) v[i][e] = 0;
        } else if (!words) {
            if (coded) {                      // the columns of a thread share a codec block
                const float am = s.q8_absmax[c / s.q8_block];
#pragma unroll
                for (int e = 0; e < NP; e++) {
                    const uint32_t q = *(const uint16_t *)(s.q8 + c + 2 * e);
                    v[i][e] = (int)((uint32_t)__half_as_ushort(decode_q8(d_code_table.code, q & 255u, am)) |
                                    (uint32_t)__half_as_ushort(decode_q8(d_code_table.code, q >> 8, am)) << 16);
                }
            } else {
#pragma unroll
                for (int e = 0; e < NP; e++) v[i][e] = *(const int *)(plain + c + 2 * e);
            }
        }
    }
    if constexpr (LN) {
        double sm = 0.0, sq = 0.0;
#pragma unroll
        for (int e = 0; e < NP; e++) {
            const double a = (double)low_half(v[0][e]), b = (double)high_half(v[0][e]);
            sm += a; sq = fma(a, a, sq);
            sm += b; sq = fma(b, b, sq);
        }
        sm = wave_sum(sm);
        sq = wave_sum(sq);
        if (lane == 0) { l.sum[wave] = sm; l.sq[wave] = sq; }
        lds_barrier();
        sm = sq = 0.0;
#pragma unroll
        for (int i = 0; i < WAVES; i++) { sm += l.sum[i]; sq += l.sq[i]; }
        // (quotients by the row's length from its reciprocal and the exact remainder: three instructions)
        auto over_k = [&](double x) { const double q = x * s.inv_h; return fma(fma(-q, (double)K, x), s.inv_h, q); };
        const double mean = over_k(sm), inv = rsqrt_f64(fmax(over_k(sq) - mean * mean, 0.0) + (double)s.eps);
#pragma unroll
        for (int e = 0; e < NP; e++) {
            const __half a = d2h_rn(((double)low_half(v[0][e]) - mean) * inv * (double)low_half(gr[e]) + (double)low_half(br[e]));
            const __half b = d2h_rn(((double)high_half(v[0][e]) - mean) * inv * (double)high_half(gr[e]) + (double)high_half(br[e]));
            v[0][e] = mine0 ? (int)((uint32_t)__half_as_ushort(a) | (uint32_t)__half_as_ushort(b) << 16) : 0;
        }
    }
    uint32_t mreg = 0, obits[NCH];
#pragma unroll
    for (int i = 0; i < NCH; i++) {
        const int c = (tid + THREADS * i) * CT;
        uint32_t bits = 0;
#pragma unroll
        for (int e = 0; e < NP; e++) {
            const uint32_t a = (uint32_t)v[i][e] & 0x7fffu, b = ((uint32_t)v[i][e] >> 16) & 0x7fffu;
            if (a >= s.theta_bits) bits |= 1u << (2 * e); else mreg = max(mreg, a);
            if (b >= s.theta_bits) bits |= 2u << (2 * e); else mreg = max(mreg, b);
        }
        if (c >= K) bits = 0;                        // (a threshold of 0 flags the zeros there as well)
        obits[i] = bits;
        // the bits of 16 columns meet in the first of their 16 / CT threads
        const uint32_t m16 = group_reduce<16 / CT>(bits << (c & 15), [](uint32_t a, uint32_t b) { return a | b; });
        if ((c & 15) == 0 && c < K) l.mask[c >> 4] = (uint16_t)m16;
#pragma unroll
        for (int e = 0; e < NP; e++)
            if (c < K) *(int *)(l.row + c + 2 * e) = v[i][e];
    }
    mreg = wave_max(mreg);
    if (lane == 0) l.mx[wave] = (int)mreg;
    lds_barrier();
#pragma unroll
    for (int i = 0; i < WAVES; i++) mreg = max(mreg, (uint32_t)l.mx[i]);
    const float s_x = __half2float(__ushort_as_half((unsigned short)mreg));
    const float r = s_x > 0.0f ? 127.0f / s_x : 0.0f;
    float neg0 = -0.0f;
    asm("" : "+v"(neg0));
#pragma unroll
    for (int i = 0; i < NCH; i++) {
        const int c = (tid + THREADS * i) * CT;
        // (|x r| <= 127.00002 for regular columns: the addition leaves the rounded integer in the low byte)
        uint32_t t[CT], o2[(CT + 3) / 4];
#pragma unroll
        for (int e = 0; e < CT; e++)
            t[e] = __float_as_uint(fmaf(e & 1 ? high_half(v[i][e >> 1]) : low_half(v[i][e >> 1]), r, neg0) + 12582912.0f);
#pragma unroll
        for (int e = 0; e < CT; e += 4) {
            const uint32_t lo = __builtin_amdgcn_perm(t[e + 1], t[e], 0x0c0c0400);
            if constexpr (CT == 2) o2[0] = lo;
            else o2[e >> 2] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(t[(e + 3) % CT], t[(e + 2) % CT], 0x0c0c0400), lo, 0x05040100);
        }
        if (obits[i]) {
#pragma unroll
            for (int e = 0; e < CT; e++) o2[e >> 2] &= ~(((obits[i] >> e) & 1u) * (0xffu << (8 * (e & 3))));
        }
        if (c < K) {
            if constexpr (CT == 8) *(uint2 *)(l.codes + c) = make_uint2(o2[0], o2[1]);
            else if constexpr (CT == 4) *(uint32_t *)(l.codes + c) = o2[0];
            else *(uint16_t *)(l.codes + c) = (uint16_t)o2[0];
        }
    }
    lds_barrier();
    return s_x;
}

// 16 bytes of a matrix that is read once; zeros from `bytes` on (no branch around the loads: registers that are written on one
// side of a branch only cost the kernel 32 spilled ones)
__device__ __forceinline__ v4i load_tile(const int8_t *base, int bytes, uint32_t offset) {
    const auto x = __builtin_amdgcn_raw_buffer_load_b128(__builtin_amdgcn_make_buffer_rsrc((void *)base, 0, bytes, 0x00020000), offset, 0, 2 /* non-temporal */);
    return (v4i){(int)x[0], (int)x[1], (int)x[2], (int)x[3]};
}

__device__ __forceinline__ int byte_of(const v4i &w, int j) {
    const int word = (j < 8) ? ((j < 4) ? w[0] : w[1]) : ((j < 12) ? w[2] : w[3]);
    return (int)(int8_t)((word >> ((j & 3) * 8)) & 0xff);
}

// PN 16-row panels of a linear, the K / 64 tiles shared out over the waves (wave w takes tiles w, w + 8, ...; WT of
// them at most, all requested before the row is there).  Returns in the first 16 PN lanes of wave 0 the sums before GeLU and
// residual.  ready: what row the codes in LDS are of (tag and linear); a second item of a stage finds its row prepared.
template <bool LN, int CT, int NCH, int WT, int PN, int CW, int D, typename AFTER>
__device__ __forceinline__ double panels(Lds<CW, D> &l, int tid, const StepArgs &s, const LinearW &w, size_t offset, int p0, int which, int &ready, float &s_x, const __half *plain, bool coded,
                                         const uint32_t *turn, uint32_t turn_tag, const uint32_t *words, uint32_t tag,
                                         const __half *gain, const __half *bias, AFTER after) {
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, kg = lane >> 4, K = w.K, KT = K >> 6, last = w.N / 16 - 1;
    v4i wv[PN][WT];
#pragma unroll
    for (int p = 0; p < PN; p++)
#pragma unroll
        for (int u = 0; u < WT; u++) {
            const int kt = wave + WAVES * u;
            wv[p][u] = load_tile(w.wt + offset + (size_t)p0 * KT * 1024, min(PN, last + 1 - p0) * KT * 1024, kt < KT ? (uint32_t)((p * KT + kt) * 1024 + lane * 16) : ~0u);
        }
    float swd[PN];
#pragma unroll
    for (int p = 0; p < PN; p++) swd[p] = ((const float *)((const uint8_t *)w.sw + offset))[min(p0 + p, last) * 16 + (lane & 15)] / 127.0f;
    const int n = min(p0 * 16 + min(lane, PN * 16 - 1), w.N - 1);            // the output that this lane finishes, if it does
    const float sn = ((const float *)((const uint8_t *)w.sw + offset))[n] / 127.0f;
    const float bn = __half2float(((const __half *)((const uint8_t *)w.bias + offset))[n]);
    const int row = (int)tag * 4 + which;
    if (row != ready) {                              // the same in all threads
        await_turn(turn, turn_tag, tid, s);
        s_x = prepare_row<LN, CT, NCH, CW, D>(l, tid, K, s, plain, coded, words, tag, gain, bias);
        ready = row;
    }
    after();                                         // requests whose data the tail needs
    int acc[PN];
    double outl[PN];
#pragma unroll
    for (int p = 0; p < PN; p++) { acc[p] = 0; outl[p] = 0.0; }
#pragma unroll
    for (int u = 0; u < WT; u++) {
        const int kt = wave + WAVES * u;
        if (kt < KT) {                               // wave-uniform
            const v4i xv = *(const v4i *)(l.codes + kt * 64 + kg * 16);
#pragma unroll
            for (int p = 0; p < PN; p++)
#pragma unroll
                for (int i = 0; i < 4; i++) acc[p] = __builtin_amdgcn_sdot4(wv[p][u][i], xv[i], acc[p], false);
            uint32_t bits = l.mask[kt * 4 + kg];
            while (bits) {                           // outlier columns: rare
                const int j = __ffs(bits) - 1;
                bits &= bits - 1;
                const double x = (double)__half2float(l.row[kt * 64 + kg * 16 + j]);
#pragma unroll
                for (int p = 0; p < PN; p++)
                    outl[p] += x * (double)dequant_w16(byte_of(wv[p][u], j), swd[p]);
            }
        }
    }
#pragma unroll
    for (int p = 0; p < PN; p++) {
        acc[p] = swap_sum<32>(swap_sum<16>(acc[p]));
        outl[p] = swap_reduce<32>(swap_reduce<16>(outl[p], add_f64), add_f64);
        if (lane < 16) { l.red_i[wave][p * 16 + lane] = acc[p]; l.red_f[wave][p * 16 + lane] = outl[p]; }
    }
    lds_barrier();
    double v = 0.0;
    if (wave == 0) {
        int a = 0;
        double f = 0.0;
        const int at = min(lane, PN * 16 - 1);
#pragma unroll
        for (int i = 0; i < WAVES; i++) { a += l.red_i[i][at]; f += l.red_f[i][at]; }
        v = (double)a * (double)(s_x / 127.0f) * (double)sn + f + (double)bn;
    }
    return v;
}

// One head's attention over keys [k_begin, k_end): as k_attn_decode, the keys in equal shares over the waves.  The new key
// and value come from the words of the QKV linear and go into the cache here.
template <int D, int CW>
__device__ __forceinline__ void attention(Lds<CW, D> &l, int tid, const StepArgs &s, int blk, int h, int range, const uint32_t *turn, uint32_t turn_tag, uint32_t tag,
                                          const Words &words) {
    constexpr int LPK = D / 8, KPI = 64 / LPK, NIT = 8;       // lanes per key, keys per load, loads of a block
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, sub = lane % LPK, kslot = lane / LPK, nh = s.nh;
    const SessTable *sess = s.sess;
    const int i = sess->len[0], cap = sess->cap[0];
    const int CH = ((i + s.ranges) / s.ranges + WAVES * KPI - 1) / (WAVES * KPI) * (WAVES * KPI);
    const int k_begin = min(range * CH, i + 1), k_end = min(i + 1, k_begin + CH);
    // (global memory, said explicitly: a pointer from the table is a generic one, whose loads the LDS barriers would wait for)
    typedef __attribute__((address_space(1))) __half *global_half;
    global_half Kc = (global_half)(sess->kv[0] + ((size_t)blk * 2 * nh + h) * cap * D);
    global_half Vc = Kc + (size_t)nh * cap * D;
    const double slope = sess->slopes[h], inv_rsd = 1.0 / sqrt((double)D);
    const int per = ((k_end - k_begin + WAVES - 1) / WAVES + KPI - 1) / KPI * KPI;
    const int wb = min(k_begin + wave * per, k_end), we = min(k_end, wb + per), newest = max(i - 1, 0);
    // cached keys and values of the first block: in flight while the query is waited for
    v8h kk[NIT], vv[NIT];
    auto load = [&](int base) {
#pragma unroll
        for (int it = 0; it < NIT; it++) {
            if (base + it * KPI >= we) continue;     // wave-uniform
            const size_t at = (size_t)min(min(base + it * KPI + kslot, we - 1), newest) * D + sub * 8;
            kk[it] = *(const __attribute__((address_space(1))) v8h *)(Kc + at);
            vv[it] = *(const __attribute__((address_space(1))) v8h *)(Vc + at);
        }
    };
    load(wb);
    await_turn(turn, turn_tag, tid, s);
    v8h qv, kn, vn;
    {
        const uint32_t *p[12];
        int w[12];
        const uint32_t *from = words.qkv + h * 3 * D + sub * 8;
#pragma unroll
        for (int e = 0; e < 12; e++) p[e] = from + (e >> 2) * D + (e & 3) * 2;
        await_words<12>(p, tag, w, s);
        qv = *(const v8h *)w;
        kn = *(const v8h *)(w + 4);
        vn = *(const v8h *)(w + 8);
    }
    if (wave == 0 && kslot == 0 && range == s.ranges - 1) {
        *(__attribute__((address_space(1))) v8h *)(Kc + (size_t)i * D + sub * 8) = kn;
        *(__attribute__((address_space(1))) v8h *)(Vc + (size_t)i * D + sub * 8) = vn;
    }
    double qf[8];
#pragma unroll
    for (int e = 0; e < 8; e++) qf[e] = (double)(float)qv[e] * inv_rsd;
    double m_run = -INFINITY, l_run = 0.0, o[8];
#pragma unroll
    for (int e = 0; e < 8; e++) o[e] = 0.0;
    for (int base = wb; base < we; base += NIT * KPI) {
        if (base > wb) load(base);
        double sc_mine = -INFINITY, mb = -INFINITY;
#pragma unroll
        for (int it = 0; it < NIT; it++) {
            if (base + it * KPI >= we) continue;     // wave-uniform
            const int j = base + it * KPI + kslot;
            const v8h k8 = min(j, we - 1) == i ? kn : kk[it];
            double dot = 0.0;
#pragma unroll
            for (int e = 0; e < 8; e++) dot += qf[e] * (double)(float)k8[e];
            dot = group_reduce<LPK>(dot, add_f64);
            const double sc = (j < we) ? dot - slope * (double)(i - j) : -INFINITY;
            mb = fmax(mb, sc);
            if (sub == it) sc_mine = sc;
        }
        const double m_new = fmax(m_run, mb);
        const double alpha = (m_run == -INFINITY) ? 0.0 : exp_f64(m_run - m_new);
        const double p_mine = (sc_mine == -INFINITY) ? 0.0 : exp_f64(sc_mine - m_new);      // (NaN stays NaN)
        l_run = l_run * alpha + group_reduce<LPK>(p_mine, add_f64);
        m_run = m_new;
#pragma unroll
        for (int e = 0; e < 8; e++) o[e] *= alpha;
        auto add_value = [&](auto itc) {
            constexpr int it = decltype(itc)::value;
            if (base + it * KPI >= we) return;
            const double p = group_bcast<LPK, it>(p_mine);
            const v8h v8 = min(base + it * KPI + kslot, we - 1) == i ? vn : vv[it];
#pragma unroll
            for (int e = 0; e < 8; e++) o[e] += p * (double)(float)v8[e];
        };
        for_constants(add_value, std::make_integer_sequence<int, NIT>());
    }
    merge_wave<LPK>(m_run, l_run, o);
    if (lane == 0) { l.am[wave] = m_run; l.al[wave] = l_run; }
#pragma unroll
    for (int e = 0; e < LPK / 8; e++) l.ao[wave][merged_dim<LPK>(lane) + e] = o[e];
    lds_barrier();
    double m = 0.0, sl = 0.0, ov = 0.0;
    if (wave < D / 64) ov = merge_waves<WAVES, D>(l.am, l.al, l.ao, lane, tid, m, sl);
    if (s.ranges > 1) {
        // the range whose sums get there last merges them all, in the order of the ranges
        double *mine = s.partials + (size_t)h * s.ranges * (D + 2);
        if (tid < D) {
            double *to = mine + (size_t)range * (D + 2);
            if (tid == 0) {
                __hip_atomic_store(to, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(to + 1, sl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __hip_atomic_store(to + 2 + tid, ov, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // this wave's sums are where every XCD sees them
        lds_barrier();
        if (tid == 0)
            l.last = __hip_atomic_fetch_add(s.done + h, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (blk + 1) * s.ranges - 1;
        lds_barrier();
        if (!l.last) return;                                        // the whole workgroup
        if (tid < D) {
            m = -INFINITY;
            sl = ov = 0.0;
            for (int c = 0; c < s.ranges; c++) m = fmax(m, __hip_atomic_load(mine + (size_t)c * (D + 2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            for (int c = 0; c < s.ranges; c++) {
                const double *pc = mine + (size_t)c * (D + 2);
                const double mc = __hip_atomic_load(pc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const double f = (mc == -INFINITY) ? 0.0 : exp_f64(mc - m);
                sl += f * __hip_atomic_load(pc + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ov += f * __hip_atomic_load(pc + 2 + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    if (tid < D) publish(words.ctx + h * D + tid, tag, d2h_rn(ov / sl));
}

// Panels per item: with one per workgroup QKV and up of 1024 columns would be 192 and 256 items, each of which prepares the row
// and polls it (and waits longer for it: the words' memory channels are busy); with two 96 and 128.  WT: tiles of a panel per
// wave, of down four times as many.
template <int CW, int WT, int D>
__global__ void __launch_bounds__(THREADS, 2) k_decode_row(StepArgs s) {
    __shared__ Lds<CW, D> l;
    constexpr int PQ = CW == 8 ? 3 : CW, PU = CW == 8 ? 4 : CW, NCH = WT / 2;
    const int H = s.H, F = s.F;
    const int nq = (3 * H / 16 + PQ - 1) / PQ, na = s.nh * s.ranges, nd = H / 16, nu = (F / 16 + PU - 1) / PU;
    const int per_block = nq + na + 2 * nd + nu, total = per_block * s.n_blocks;
    Words words;
    words.x = s.words;
    words.qkv = words.x + H;
    words.ctx = words.qkv + 3 * H;
    words.x1 = words.ctx + H;
    words.g = words.x1 + H;
    if (threadIdx.x == 0) l.next = __hip_atomic_fetch_add(s.ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    lds_barrier();
    int t = l.next, ready = -1;
    float s_x = 0.0f;
    while (t < total) {
        int tid = threadIdx.x;                       // opaque: what depends on it is worked out again for every item, not kept over all
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63;
        const int b = t / per_block;
        const size_t off = (size_t)b * s.stride;
        const uint32_t tag = (uint32_t)b + 1;
        int i = t - b * per_block;
        const bool first = b == 0;
        const int spread = (int)(blockIdx.x * 32u) % H, spread_g = (int)(blockIdx.x * 32u) % F;  // the word whose arrival this workgroup takes as its turn
        auto at = [&](const __half *p) { return (const __half *)((const uint8_t *)p + off); };
        auto none = [] {};
        if (i < nq) {
            const double v = panels<true, CW, 1, WT, PQ, CW, D>(l, tid, s, s.lin[0], off, i * PQ, 0, ready, s_x, s.x, s.q8 != nullptr, first ? nullptr : words.g + spread_g,
                                                             (uint32_t)b, first ? nullptr : words.x, (uint32_t)b, at(s.ln1g), at(s.ln1b), none);
            const int n = i * PQ * 16 + lane;
            if (tid < PQ * 16 && n < 3 * H) publish(words.qkv + n, tag, d2h_rn(v));
        } else if ((i -= nq) < na) {
            ready = -1;                              // (the attention's sums lie where the row was)
            attention<D, CW>(l, tid, s, b, i / s.ranges, i % s.ranges, first ? nullptr : words.x + spread, (uint32_t)b, tag, words);
        } else if ((i -= na) < nd) {
            uint32_t res = 0;
            const int n = i * 16 + (lane & 15);
            const double v = panels<false, CW, 1, WT, 1, CW, D>(l, tid, s, s.lin[1], off, i, 1, ready, s_x, nullptr, false, words.qkv + spread, tag, words.ctx, tag, nullptr, nullptr, [&] {
                if (tid >= 16) return;
                if (!first) res = __hip_atomic_load(words.x + n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                else if (s.q8) res = __half_as_ushort(decode_q8(d_code_table.code, s.q8[n], s.q8_absmax[n / s.q8_block]));
                else res = __half_as_ushort(s.x[n]);
            });
            if (tid < 16) publish(words.x1 + n, tag, d2h_rn(v + (double)low_half((int)res)));
        } else if ((i -= nd) < nu) {
            const double v = panels<true, CW, 1, WT, PU, CW, D>(l, tid, s, s.lin[2], off, i * PU, 2, ready, s_x, nullptr, false, words.ctx + spread, tag, words.x1, tag,
                                                             at(s.ln2g), at(s.ln2b), none);
            const int n = i * PU * 16 + lane;
            if (tid < PU * 16 && n < F) publish(words.g + n, tag, d2h_rn(gelu_tanh(v)));
        } else {
            i -= nu;
            uint32_t res = 0;
            const int n = i * 16 + (lane & 15);
            const double v = panels<false, 8, NCH, 4 * WT, 1, CW, D>(l, tid, s, s.lin[3], off, i, 3, ready, s_x, nullptr, false, words.x1 + spread, tag, words.g, tag, nullptr, nullptr, [&] {
                if (tid < 16) res = __hip_atomic_load(words.x1 + n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            });
            if (tid < 16) {
                const __half hv = d2h_rn(v + (double)low_half((int)res));
                if (b == s.n_blocks - 1) s.out[n] = hv;
                else publish(words.x + n, tag, hv);
            }
        }
        // (not earlier: a workgroup that held two numbers would have two items of one stage now and then)
        if (tid == 0) l.next = __hip_atomic_fetch_add(s.ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        lds_barrier();                               // ... and everybody is done with the item's LDS
        t = l.next;
        lds_barrier();
    }
}

}  // namespace

// The line: a stage of 4096 columns is as many items as there are workgroups, none of which then waits with weights on the way for
// the next one (64 keys, per block: 4096 columns 55.1 us as five launches, 53.7 in one; 3840 62.8 and 48.8; 3072 45.2 and 35.8;
// 2560 41.7 and 30.7; with 5 % of the columns outliers 4096 96 and 70, with 2048 keys 70 and 67).
// The price: with more than 128 registers a workgroup has its unit for itself, so the steps of several spans on several streams run
// one after the other instead of into each other.  Three blocks, 256 keys, one, two, three spans at a time, us a step of all: 2048 columns 71, 124,
// 165 (as separate launches 107, 146, 185); 3072 112, 211, 268 (145, 196, 265); 3840 150, 293, 424 (193, 270, 361); 4096 163, 321, 461
// (176, 262, 349).
bool ps_decode_row_applies(int H, int F, int d, int n_blocks) {
    return H <= 4096 && F <= 16384 && (d == 64 || d == 128) && n_blocks < 65535;
}

hipError_t ps_steps_given_up(int *dev_count, hipStream_t st) {
    k_given_up<<<1, 1, 0, st>>>(dev_count);
    return hipGetLastError();
}

hipError_t ps_decode_row(const StepArgs &s0, int d, int max_keys, hipStream_t st) {
    StepArgs s = s0;
    s.inv_h = 1.0 / s.H;
    // One workgroup per head up to 64 KB of keys; more ranges than that cost more in their merge (4 to 5 us a block) than they save
    // (8 blocks of 1024 columns, 16 heads of 64, 2048 keys: 4 ranges 188 us, 8 ranges 202, 16 ranges 252; 8 heads of 128, 1000
    // keys: 1 range 205, 3 ranges 189), and together no more than half of the workgroups (4 blocks of 2048 columns, 32 heads,
    // 2000 keys: 8 ranges 126 us, 4 ranges 115) - three quarters once half would leave each 192 KB of keys and as many values:
    // from there on it is the units that read the cache that count (us a block at 128, 192, 256 ranges in all, and as five launches:
    // 48 heads of 64, 16384 keys: 103, 78, 75, 87; 32 heads of 128, 32768 keys: 187, 154, 152, 159; below that line 16 heads of 128,
    // 4096 keys: 36, 38, 41, 47; 16 heads of 64, 8192 keys: 32, 33, 36, 42).  All of them leave no unit to what comes behind (32 heads
    // of 128, 4096 keys: 71 at 192, 72 at 256).
    const int half = max(128 / s.nh, 1);
    const int most = (long long)max_keys * d >= 98304ll * half ? 192 / s.nh : half;
    s.ranges = max(1, min(min((long long)max_keys * d / 32768, (long long)most), (long long)PS_ATTN_MAX_SPLITS));
    // columns of a LayerNorm row per thread, tiles of a panel per wave: the smallest form that takes the span (fewer registers,
    // fewer loads beyond the panels' ends)
    auto fits = [&](int h) { return s.H <= h && s.F <= 4 * h; };
    auto kern = fits(1024)   ? (d == 64 ? k_decode_row<2, 2, 64> : k_decode_row<2, 2, 128>)
                : fits(2048) ? (d == 64 ? k_decode_row<4, 4, 64> : k_decode_row<4, 4, 128>)
                : fits(3072) ? (d == 64 ? k_decode_row<8, 6, 64> : k_decode_row<8, 6, 128>)
                             : (d == 64 ? k_decode_row<8, 8, 64> : k_decode_row<8, 8, 128>);
    kern<<<256, THREADS, 0, st>>>(s);
    return hipGetLastError();
}

// ALiBi causal attention of query rows against the per-session key/value caches, fp64 throughout
// (products of fp16 values are exact; the fp16 context equals the exactly rounded one).
// Decode (one query per session): k_attn_decode, one workgroup per (key range, head, query row),
// wave-local online softmax, k_attn_combine merges the key ranges.  Prefill (several queries per
// session): k_attn_prefill on the fp64 matrix instruction; for the backward pass it can also store the
// log of the softmax denominators and the context before its fp16 rounding.
#include <mutex>
#include <utility>

#include "attn_state.h"
#include "common.h"
#include "digits.h"

namespace {

constexpr int ATTN_SPLIT_BELOW = 256;
// Where the running maximum of k_attn_prefill starts: below every score but finite, so that a masked score (-infinity)
// minus the maximum is -infinity, whose exponential is 0, also before the first visible key - no test per key.
constexpr double ATTN_LOWEST = -1e300;

// Start of a call: workgroup 0 copies the table word by word, all of them clear the outlier masks and the records of the LayerNorms (or a row's words) (one launch: a launch
// of its own costs 2 to 4.5 us whatever it does).
__global__ void __launch_bounds__(256) k_call_setup(SessTable t, SessTable *dst, uint32_t *masks, size_t n_masks, uint32_t *more,
                                                    size_t n_more) {
    if (blockIdx.x == 0) {
        const uint32_t *s = (const uint32_t *)&t;
        uint32_t *d = (uint32_t *)dst;
        for (int i = threadIdx.x; i < (int)(sizeof(SessTable) / 4); i += 256) d[i] = s[i];
    }
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n_masks; i += (size_t)gridDim.x * 256) masks[i] = 0u;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n_more; i += (size_t)gridDim.x * 256) more[i] = 0u;
}

// N consecutive halves at an address aligned to min(16, 2 N) bytes
template <int N>
__device__ __forceinline__ void load_halves(const __half *p, __half (&dst)[N]) {
    if constexpr (N >= 8) {
#pragma unroll
        for (int i = 0; i < N / 8; i++) *(v8h *)(dst + 8 * i) = *(const v8h *)(p + 8 * i);
    } else if constexpr (N == 4) {
        *(v4h *)dst = *(const v4h *)p;
    } else if constexpr (N == 2) {
        *(__half2 *)dst = *(const __half2 *)p;
    } else {
        dst[0] = *p;
    }
}

// Scores of one tile of 16 keys x 16 queries as exact int8 digit products (D = 64 or 128): ka holds the keys' digit
// planes as A operands, qa the queries' as B operands ([plane][64 dims]); lane (g, c), register r of the result is key
// 4r + g of query c, as the fp64 instruction returns it, scaled by inv_rsd.  The pairs with the same i + j share an
// accumulator (at most 4 * 2^14 * 128 = 2^23); the two lowest and the fifth and sixth meet in int32 (2^30 at most).
// The int8 instruction returns row 4g + r: the tile's keys are handed in permuted, see digit_key_slot.
template <int HALVES>
__device__ __forceinline__ v4d digit_scores(const v4i (&ka)[4][HALVES], const v4i (&qa)[4][HALVES], double scale) {
    v4i acc[7];
#pragma unroll
    for (int s = 0; s < 7; s++) acc[s] = (v4i){0, 0, 0, 0};
#pragma unroll
    for (int h = 0; h < HALVES; h++)
#pragma unroll
        for (int d = 0; d < 4; d++)               // diagonals of the pair table: consecutive products are independent
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int j = (i + d) & 3;
                acc[i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ka[i][h], qa[j][h], acc[i + j], 0, 0, 0);
            }
    v4d S;
    const double sc = scale * 0x1p-48;
#pragma unroll
    for (int r = 0; r < 4; r++) {
        double t = (double)acc[6][r];
        t = t * 65536.0 + (double)((acc[5][r] << 8) + acc[4][r]);
        t = t * 256.0 + (double)acc[3][r];
        t = t * 256.0 + (double)acc[2][r];
        t = t * 65536.0 + (double)((acc[1][r] << 8) + acc[0][r]);
        S[r] = t * sc;
    }
    return S;
}
// slot (row of the A operand) of key k of a tile: row 4g + r of the result belongs to key 4r + g
__device__ __forceinline__ constexpr int digit_key_slot(int k) { return 4 * (k & 3) + (k >> 2); }

// Prefill (T > 1 new tokens per session): exact attention on the matrix cores.
// A workgroup of four waves owns 64 consecutive query rows of one (session, head), 16 per wave, and
// walks the key tiles (16 keys each) up to the causal limit with an online softmax per wave.
//   S^T = K Q^T: head_dim 64 and 128 as exact int8 digit products (32 instructions of 16 clocks and some 30 vector
//   instructions per tile and 128 dims, where the fp64 instruction takes 32 of 64 clocks); smaller head_dims, and tiles
//   in which a key or query value of 127.5 or more does not fit four digits, on
//   v_mfma_f64_16x16x4_f64, A = keys (row = key), B = queries (column = query);
//                   lane l feeds row/column l%16 and the dims [l/16 * D/4, +D/4) - any pairing of
//                   the contraction index works as long as both operands use the same one.
//   the result registers hold S^T[key 4r + l/16][query l%16], which is exactly the B operand of
//   O^T += V^T P^T on the fp64 instruction (A = values with row i = output dims i*D/16 + blk), so the probabilities
//   never change lanes.  Products of fp16 inputs are exact in fp64; the fp16 context equals the exactly
//   rounded one (a different summation order moves the fp64 sum by ~1e-16 relative).
// The conversions of a key / value tile (fp16 to digits, to fp64) cost about as much vector-ALU time as its
// matrix instructions take, so they are done once per workgroup: the four waves convert the next
// tile together into LDS, already in A-operand order,
// while the current one is multiplied.  Queries are converted once per wave and stay in registers.
// 8 x 512 tokens, 32 heads of 128: 445 us with fp64 scores, 375 us with digits.
template <int D>
__global__ void __launch_bounds__(256, 2) k_attn_prefill(const __half *__restrict__ q, const SessTable *__restrict__ sess,
                                                         int blk, int B, int T, int nh, __half *__restrict__ ctx,
                                                         uint32_t *__restrict__ mask, float theta,
                                                         float *__restrict__ lse, float *__restrict__ ctx32) {
    constexpr int DS = D / 4, NB = D / 16;           // dims per lane group; output blocks of 16 dims
    constexpr bool DIGITS = D >= 64;
    constexpr int HALVES = DIGITS ? D / 64 : 1;
    constexpr int VT = 16 * D * 8;                   // bytes of a value tile (fp64)
    constexpr int KTB = DIGITS ? 4 * HALVES * 1024 : 16 * D * 8;     // bytes of a key tile (digit planes or fp64)
    extern __shared__ __align__(16) unsigned char kvl[];             // [2 buffers][keys | values]
    __shared__ int kbig[2];                          // DIGITS: tile + 1 of a buffer's tile that needs the fp64 form
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
    // One-dimensional grid.  Consecutive workgroup ids land on different XCDs (8, each with its own L2): the id
    // is decoded so that all query blocks of one (session, head) run on the same XCD and share its keys/values.
    // A workgroup takes TWO query blocks of its (session, head), number i and number nbx - 1 - i, one after the
    // other: with the causal limit a block walks 4 i + 4 key tiles (plus the cached ones), so every workgroup of
    // the launch does the same amount of work and none is left running alone at the end.
    const int nbx = (T + 63) / 64, nbh = (nbx + 1) / 2, grp = blockIdx.x / (8 * nbh), rem = blockIdx.x - grp * 8 * nbh;
    const int pair = grp * 8 + (rem & 7);
    if (pair >= B * nh) return;                       // the whole workgroup
    const int qb0 = rem >> 3, s = pair / nh, h = pair - s * nh;
    if (threadIdx.x < 2) kbig[threadIdx.x] = 0;
    if constexpr (DIGITS) __syncthreads();
    for (int pass = 0; pass < 2; pass++) {
    const int qb = pass ? nbx - 1 - qb0 : qb0;
    if (pass && qb == qb0) break;                     // odd count: the middle block stands alone
    if (pass) __syncthreads();                        // the tile buffers are reused
    const int qt = qb * 4 + wave;
    const int L = sess->len[s], cap = sess->cap[s], H = nh * D;
    const __half *Kc = sess->kv[s] + ((size_t)blk * 2 * nh + h) * cap * D;
    const __half *Vc = Kc + (size_t)nh * cap * D;
    const double slope = sess->slopes[h], inv_rsd = 1.0 / sqrt((double)D);
    const int last_key = L + T - 1;                   // newest key in the cache (already appended)
    const int tq = qt * 16 + c;                       // this lane's query row inside the session
    const int qpos = L + tq;                          // its absolute position
    const size_t qrow = (size_t)s * T + min(tq, T - 1);

    const __half *qp = q + qrow * H + h * D;
    double qd[DIGITS ? 1 : DS];
    v4i qa[4][HALVES];
    bool q_big = false;
    if constexpr (DIGITS) {
#pragma unroll
        for (int hf = 0; hf < HALVES; hf++) {
            __half x[16];
            load_halves<16>(qp + hf * 64 + g * 16, x);
#pragma unroll
            for (int w = 0; w < 4; w++) {
                const __half x4[4] = {x[4 * w], x[4 * w + 1], x[4 * w + 2], x[4 * w + 3]};
                int pl[4];
                digit_planes4(x4, pl);
#pragma unroll
                for (int i = 0; i < 4; i++) qa[i][hf][w] = pl[i];
            }
#pragma unroll
            for (int e = 0; e < 16; e++) q_big |= (__half_as_ushort(x[e]) & 0x7fffu) >= DIGITS_BIG;
        }
        q_big = __any(q_big);
    } else {
#pragma unroll
        for (int e = 0; e < DS; e++) qd[e] = (double)__half2float(qp[g * DS + e]) * inv_rsd;   // 1/sqrt(d) folded into the query
    }
    v4d O[NB];
#pragma unroll
    for (int b = 0; b < NB; b++) O[b] = (v4d){0.0, 0.0, 0.0, 0.0};
    double m_run = ATTN_LOWEST, l_run = 0.0;

    // key tiles this wave needs (none if its queries lie beyond T) and the workgroup's last wave needs
    const int nkt_w = qt * 16 < T ? min(L + qt * 16 + 15, last_key) / 16 + 1 : 0;
    const int nkt = min(L + (qb * 4 + 3) * 16 + 15, last_key) / 16 + 1;

    // conversion duty of this thread: NB consecutive dims of one key of the tile, keys and values alike
    const int fk = threadIdx.x >> 4, fd = (threadIdx.x & 15) * NB;
    __half kraw[NB], vraw[NB];
    auto fetch = [&](int kt) {
        const size_t off = (size_t)min(kt * 16 + fk, last_key) * D + fd;
        load_halves<NB>(Kc + off, kraw);
        load_halves<NB>(Vc + off, vraw);
    };
    auto stash = [&](int kt) {
        const int buf = kt & 1;
        double *vd = (double *)(kvl + (size_t)buf * (KTB + VT) + KTB);
        if constexpr (DIGITS) {
            unsigned char *kb = kvl + (size_t)buf * (KTB + VT);
            // dims fd .. fd + NB: half fd / 64, lane group fd % 64 / 16; the 16 keys of a (half, group) are rotated by 4 per
            // group so that the writes of a wave spread over the banks (a read takes all 16)
            const int hf = fd >> 6, gg = (fd & 63) >> 4, slot = gg * 16 + ((digit_key_slot(fk) + 4 * gg) & 15);
            int pl[NB / 4][4];
            bool big = false;
#pragma unroll
            for (int w = 0; w < NB / 4; w++) {
                const __half x4[4] = {kraw[4 * w], kraw[4 * w + 1], kraw[4 * w + 2], kraw[4 * w + 3]};
                digit_planes4(x4, pl[w]);
            }
#pragma unroll
            for (int i = 0; i < NB; i++) big |= (__half_as_ushort(kraw[i]) & 0x7fffu) >= DIGITS_BIG;
#pragma unroll
            for (int i = 0; i < 4; i++) {
                unsigned char *dst = kb + ((size_t)(i * HALVES + hf) * 64 + slot) * 16 + (fd & 15);
                if constexpr (NB == 8) *(v2i *)dst = (v2i){pl[0][i], pl[1][i]};
                else *(int *)dst = pl[0][i];
            }
            if (__any(big) && lane == 0) kbig[buf] = kt + 1;
        }
#pragma unroll
        for (int i = 0; i < NB; i++) {
            if constexpr (!DIGITS) {
                double *kd = (double *)(kvl + (size_t)buf * (KTB + VT));
                const int d = fd + i;
                // keys: A operand of step e is K[key][g * DS + e] at lane (g, key); the 64 values of a step are
                // rotated by 4 * (e / 8) positions so that the 64 threads of a wave, which write 4 steps, 4 lane
                // groups and 4 keys at a time, spread over all LDS banks (reads stay 64 consecutive values)
                const int e = d % DS;
                kd[e * 64 + (((d / DS) * 16 + fk + 4 * (e >> 3)) & 63)] = (double)__half2float(kraw[i]);
            }
            // values: A operand of step (r, b) is V[key 4r + g][c * NB + b] at lane (g, c)
            vd[((fk >> 2) * NB + i) * 64 + (fk & 3) * 16 + (threadIdx.x & 15)] = (double)__half2float(vraw[i]);
        }
    };
    // Newest tile first: the running maximum is then found early (the ALiBi bias falls with the distance), and the
    // rescaling of sums and outputs is skipped while no query of the wave has a new one.
    fetch(nkt - 1);
    stash(nkt - 1);
    __syncthreads();
    double dist = (double)(qpos - (nkt - 1) * 16 - g);               // distance to this lane's first key of the tile
    for (int kt = nkt - 1; kt >= 0; kt--, dist += 16.0) {
        if (kt > 0) fetch(kt - 1);                    // in flight during the multiplications below
        if (kt < nkt_w) {
            const unsigned char *kb = kvl + (size_t)(kt & 1) * (KTB + VT);
            const double *kd0 = (const double *)kb, *vd = (const double *)(kb + KTB) + lane;
            v4d S;
            if (DIGITS && !q_big && kbig[kt & 1] != kt + 1) {
                v4i ka[4][HALVES];
#pragma unroll
                for (int i = 0; i < 4; i++)
#pragma unroll
                    for (int hf = 0; hf < HALVES; hf++)
                        ka[i][hf] = *(const v4i *)(kb + ((size_t)(i * HALVES + hf) * 64 + g * 16 + ((c + 4 * g) & 15)) * 16);
                S = digit_scores<HALVES>(ka, qa, inv_rsd);
            } else {
                // scores of 16 keys x 16 queries in fp64
                // (a dependent fp64 matrix instruction issues at about half the rate of independent ones:
                // up to four partial sums run side by side)
                constexpr int NCH = DS >= 16 ? 4 : (DS >= 8 ? 2 : 1);
                v4d Sp[NCH];
#pragma unroll
                for (int i = 0; i < NCH; i++) Sp[i] = (v4d){0.0, 0.0, 0.0, 0.0};
                if constexpr (DIGITS) {               // rare: straight from the cache
                    const __half *kr = Kc + (size_t)min(kt * 16 + c, last_key) * D + g * DS;
#pragma unroll 4
                    for (int e = 0; e < DS; e++)
                        Sp[0] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)__half2float(kr[e]), (double)__half2float(qp[g * DS + e]) * inv_rsd, Sp[0], 0, 0, 0);
                } else {
#pragma unroll
                    for (int e = 0; e < DS; e++)
                        Sp[e % NCH] = __builtin_amdgcn_mfma_f64_16x16x4f64(kd0[e * 64 + ((lane + 4 * (e >> 3)) & 63)], qd[e], Sp[e % NCH], 0, 0, 0);
                }
                S = Sp[0];
#pragma unroll
                for (int i = 1; i < NCH; i++) S += Sp[i];
            }
            double sc[4], mt = -INFINITY;
#pragma unroll
            for (int r = 0; r < 4; r++) sc[r] = fma(-slope, dist - 4.0 * r, S[r]);
            if (kt * 16 + 15 > L + qt * 16) {         // wave-uniform: keys some query of the wave does not see
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const int kpos = kt * 16 + 4 * r + g;
                    if (kpos > qpos || kpos > last_key) sc[r] = -INFINITY;
                }
            }
#pragma unroll
            for (int r = 0; r < 4; r++) mt = fmax(mt, sc[r]);
            mt = swap_reduce<32>(swap_reduce<16>(mt, max_f64), max_f64);
            const double m_new = fmax(m_run, mt);
            if (__any(m_new > m_run)) {
                const double alpha = exp_f64(m_run - m_new);
                l_run *= alpha;
#pragma unroll
                for (int b = 0; b < NB; b++) O[b] *= alpha;
                m_run = m_new;
            }
            double p[4];
#pragma unroll
            for (int r = 0; r < 4; r++) {
                p[r] = exp_f64(sc[r] - m_run);
                l_run += p[r];                        // per lane group; the groups are added at the end
            }
#pragma unroll
            for (int r = 0; r < 4; r++)
#pragma unroll
                for (int b = 0; b < NB; b++)
                    O[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(vd[(r * NB + b) * 64], p[r], O[b], 0, 0, 0);
        }
        if (kt > 0) stash(kt - 1);                    // that buffer was last read before the previous barrier
        __syncthreads();
    }
    l_run = swap_reduce<32>(swap_reduce<16>(l_run, add_f64), add_f64);
    // log of the softmax denominator, kept for the backward pass: [head][row of the call]
    if (lse && tq < T && g == 0) lse[(size_t)h * B * T + qrow] = (float)(m_run + log(l_run));
    if (tq < T) {
        // O[b][r] = output dim (4r + g) * NB + b of query c: NB consecutive dims per (r, g)
        __half *dst = ctx + qrow * H + h * D;
#pragma unroll
        for (int r = 0; r < 4; r++) {
            __half out[NB];
#pragma unroll
            for (int b = 0; b < NB; b++) out[b] = d2h_rn(O[b][r] / l_run);
#pragma unroll
            for (int b = 0; b < NB; b++) {
                dst[(4 * r + g) * NB + b] = out[b];
                flag_outlier(mask, theta, h * D + (4 * r + g) * NB + b, out[b]);
            }
            if (ctx32) {   // the context before its fp16 rounding, for the backward pass
#pragma unroll
                for (int b = 0; b < NB; b++) ctx32[qrow * H + h * D + (4 * r + g) * NB + b] = (float)(O[b][r] / l_run);
            }
        }
    }
    }   // pass
}

// The same attention for launches of few workgroups (short prompts, few sessions and heads: 128 tokens x 16 heads
// made 16 workgroups of k_attn_prefill, and 33 us of a 120 us block).  A workgroup owns ONE tile of 16 queries; its
// NWK waves share out the KEY tiles (wave w takes tiles w, w + NWK, ...), each with its own online softmax, and the
// states meet in LDS at the end, added in wave order.  No operand is shared between waves, so every lane loads its
// fragments of the next key tile straight into registers (both products' A operands are consecutive halves of a key
// or value row) and converts them itself: twice the conversions of the other form per matrix instruction, but 8 times
// as many workgroups with a quarter of the chain.  Operand layouts and arithmetic as in k_attn_prefill.
template <int D, int NWK>
__global__ void __launch_bounds__(64 * NWK, 2) k_attn_prefill_split(const __half *__restrict__ q, const SessTable *__restrict__ sess,
                                                                 int blk, int B, int T, int nh, __half *__restrict__ ctx,
                                                                 uint32_t *__restrict__ mask, float theta,
                                                                 float *__restrict__ lse, float *__restrict__ ctx32) {
    constexpr int DS = D / 4, NB = D / 16;
    extern __shared__ __align__(16) double part[];   // [NWK][4 r][NB b][64 lanes] outputs, then [NWK][16] m, [NWK][16] l
    double *pm = part + NWK * 4 * NB * 64, *pl = pm + NWK * 16;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, c = lane & 15, g = lane >> 4;
    // all query tiles of one (session, head) on one XCD, those with the most keys first
    const int nqt = (T + 15) / 16, grp = blockIdx.x / (8 * nqt), rem = blockIdx.x - grp * 8 * nqt;
    const int pair = grp * 8 + (rem & 7), qt = nqt - 1 - (rem >> 3);
    if (pair >= B * nh) return;                       // the whole workgroup
    const int s = pair / nh, h = pair - s * nh;
    const int L = sess->len[s], cap = sess->cap[s], H = nh * D;
    const __half *Kc = sess->kv[s] + ((size_t)blk * 2 * nh + h) * cap * D;
    const __half *Vc = Kc + (size_t)nh * cap * D;
    const double slope = sess->slopes[h], inv_rsd = 1.0 / sqrt((double)D);
    const int last_key = L + T - 1, tq = qt * 16 + c, qpos = L + tq;
    const size_t qrow = (size_t)s * T + min(tq, T - 1);
    const int nkt = min(L + qt * 16 + 15, last_key) / 16 + 1;

    __half kn[DS], vn[4][NB];
    auto fetch = [&](int kt) {                        // this lane's fragments of a key tile (rows clamped to the newest key)
        load_halves<DS>(Kc + (size_t)min(kt * 16 + c, last_key) * D + g * DS, kn);
#pragma unroll
        for (int r = 0; r < 4; r++) load_halves<NB>(Vc + (size_t)min(kt * 16 + 4 * r + g, last_key) * D + c * NB, vn[r]);
    };
    fetch(min(wave, nkt - 1));
    double qd[DS];
    {
        __half qh[DS];
        load_halves<DS>(q + qrow * H + h * D + g * DS, qh);
#pragma unroll
        for (int e = 0; e < DS; e++) qd[e] = (double)__half2float(qh[e]) * inv_rsd;
    }
    v4d O[NB];
#pragma unroll
    for (int b = 0; b < NB; b++) O[b] = (v4d){0.0, 0.0, 0.0, 0.0};
    double m_run = -INFINITY, l_run = 0.0;
    for (int kt = wave; kt < nkt; kt += NWK) {
        __half kc[DS], vc[4][NB];
#pragma unroll
        for (int e = 0; e < DS; e++) kc[e] = kn[e];
#pragma unroll
        for (int r = 0; r < 4; r++)
#pragma unroll
            for (int b = 0; b < NB; b++) vc[r][b] = vn[r][b];
        fetch(min(kt + NWK, nkt - 1));
        constexpr int NCH = DS >= 16 ? 4 : (DS >= 8 ? 2 : 1);
        v4d Sp[NCH];
#pragma unroll
        for (int i = 0; i < NCH; i++) Sp[i] = (v4d){0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < DS; e++)
            Sp[e % NCH] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)__half2float(kc[e]), qd[e], Sp[e % NCH], 0, 0, 0);
        v4d S = Sp[0];
#pragma unroll
        for (int i = 1; i < NCH; i++) S += Sp[i];
        double sc[4], mt = -INFINITY;
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int kpos = kt * 16 + 4 * r + g;
            sc[r] = (kpos <= qpos && kpos <= last_key) ? S[r] - slope * (double)(qpos - kpos) : -INFINITY;
            mt = fmax(mt, sc[r]);
        }
        mt = swap_reduce<32>(swap_reduce<16>(mt, max_f64), max_f64);
        const double m_new = fmax(m_run, mt);         // -infinity while this wave has seen no key of this query
        const double alpha = (m_run == -INFINITY) ? 0.0 : exp_f64(m_run - m_new);
        double p[4], psum = 0.0;
#pragma unroll
        for (int r = 0; r < 4; r++) {
            p[r] = (sc[r] == -INFINITY) ? 0.0 : exp_f64(sc[r] - m_new);
            psum += p[r];
        }
        l_run = l_run * alpha + psum;
        m_run = m_new;
#pragma unroll
        for (int b = 0; b < NB; b++) O[b] *= alpha;
#pragma unroll
        for (int r = 0; r < 4; r++)
#pragma unroll
            for (int b = 0; b < NB; b++)
                O[b] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)__half2float(vc[r][b]), p[r], O[b], 0, 0, 0);
    }
    l_run = swap_reduce<32>(swap_reduce<16>(l_run, add_f64), add_f64);
    // states of the waves -> LDS; wave r < 4 finishes register r of every output block
#pragma unroll
    for (int r = 0; r < 4; r++)
#pragma unroll
        for (int b = 0; b < NB; b++) part[((wave * 4 + r) * NB + b) * 64 + lane] = O[b][r];
    if (g == 0) { pm[wave * 16 + c] = m_run; pl[wave * 16 + c] = l_run; }
    __syncthreads();
    if (wave >= 4 || tq >= T) return;
    double m = pm[c], l = 0.0, o[NB], f[NWK];
#pragma unroll
    for (int w = 1; w < NWK; w++) m = fmax(m, pm[w * 16 + c]);     // key 0 is visible to every query: finite
#pragma unroll
    for (int w = 0; w < NWK; w++) {
        f[w] = exp_f64(pm[w * 16 + c] - m);
        l += f[w] * pl[w * 16 + c];
    }
#pragma unroll
    for (int b = 0; b < NB; b++) {
        o[b] = 0.0;
#pragma unroll
        for (int w = 0; w < NWK; w++) o[b] += f[w] * part[((w * 4 + wave) * NB + b) * 64 + lane];
    }
    if (lse && g == 0 && wave == 0) lse[(size_t)h * B * T + qrow] = (float)(m + log(l));
    const int d0 = (4 * wave + g) * NB;               // NB consecutive dims
    __half *dst = ctx + qrow * H + h * D + d0;
#pragma unroll
    for (int b = 0; b < NB; b++) {
        const double v = o[b] / l;
        const __half hv = d2h_rn(v);
        dst[b] = hv;
        flag_outlier(mask, theta, h * D + d0 + b, hv);
        if (ctx32) ctx32[qrow * H + h * D + d0 + b] = (float)v;
    }
}

template <int D, int NWK>
hipError_t launch_prefill_split(const __half *q, const SessTable *sess, int blk, int B, int T, int nh, __half *ctx, uint32_t *mask,
                                float theta, float *lse, float *ctx32, hipStream_t st) {
    const size_t lds = ((size_t)NWK * 4 * (D / 16) * 64 + 2 * NWK * 16) * 8;
    auto kern = k_attn_prefill_split<D, NWK>;
    if (lds > 64 * 1024) {
        static std::mutex attr_lock;
        static bool attr_set = false;
        std::lock_guard<std::mutex> hold(attr_lock);
        if (!attr_set) {
            hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            attr_set = true;
        }
    }
    kern<<<(B * nh + 7) / 8 * 8 * ((T + 15) / 16), 64 * NWK, lds, st>>>(q, sess, blk, B, T, nh, ctx, mask, theta, lse, ctx32);
    return hipGetLastError();
}

// Decode (one query per session): every wave owns a contiguous slice of the key range and runs
// its own online softmax over 64-key blocks with no workgroup barrier in the loop.  Inside a
// wave, head_dim/8 neighbouring lanes share a key (16 bytes of it each), so one load
// instruction reads 1 KB of consecutive cache bytes; each lane group keeps its own softmax
// state, the groups, then the 4 waves, then the key ranges are merged at the end.  fp64
// throughout: the kernel waits on HBM anyway, and the fp16 context then equals the exactly
// rounded one.
// NW waves per workgroup: 8 instead of 4 where that lets one workgroup take the whole key range of a (row, head),
// so that no partial results go through memory.
template <int D, int NW>
__global__ void __launch_bounds__(64 * NW) k_attn_decode(const __half *__restrict__ q, const SessTable *__restrict__ sess,
                                                     int blk, int nh, int CH, int nsplit,
                                                     double *__restrict__ partials, __half *__restrict__ ctx,
                                                     uint32_t *__restrict__ mask, float theta) {
    constexpr int LPK = D / 8, KPI = 64 / LPK, NIT = LPK;
    __shared__ double red_m[NW], red_l[NW], red_o[NW][D];
    const int c = blockIdx.x, h = blockIdx.y, s = blockIdx.z;
    const int i = sess->len[s];                                // position of the query; keys 0..i
    const int k_begin = c * CH, k_end = min(i + 1, k_begin + CH);
    if (k_begin >= k_end) return;                              // whole workgroup leaves together
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, sub = lane % LPK, kslot = lane / LPK;
    const int cap = sess->cap[s], H = nh * D;
    const __half *Kc = sess->kv[s] + ((size_t)blk * 2 * nh + h) * cap * D;
    const __half *Vc = Kc + (size_t)nh * cap * D;
    // (q . k) / sqrt(d) is computed as (q / sqrt(d)) . k: one division per query element instead of one per key;
    // the fp64 result moves by a few 1e-16 relative, far below the final fp16 rounding
    const double slope = sess->slopes[h], inv_rsd = 1.0 / sqrt((double)D);
    const int per = (((k_end - k_begin + NW - 1) / NW) + 63) & ~63;
    const int wb = k_begin + wave * per, we = min(k_end, wb + per);
    double qf[8];
    {
        v8h qv = *(const v8h *)(q + (size_t)s * H + h * D + sub * 8);
#pragma unroll
        for (int e = 0; e < 8; e++) qf[e] = (double)(float)qv[e] * inv_rsd;   // 1/sqrt(d) folded into the query
    }
    double m_run = -INFINITY, l_run = 0.0, o[8];
#pragma unroll
    for (int e = 0; e < 8; e++) o[e] = 0.0;

    for (int base = wb; base < we; base += 64) {
        // all loads of the block are issued unconditionally (index clamped into the slice) so they
        // go out back to back; out-of-range keys are masked by their score
        v8h kv[NIT];
#pragma unroll
        for (int it = 0; it < NIT; it++)
            kv[it] = *(const v8h *)(Kc + (size_t)min(base + it * KPI + kslot, we - 1) * D + sub * 8);
        double sc_mine = -INFINITY, mb = -INFINITY;
#pragma unroll
        for (int it = 0; it < NIT; it++) {
            const int j = base + it * KPI + kslot;
            double dot = 0.0;
#pragma unroll
            for (int e = 0; e < 8; e++) dot += qf[e] * (double)(float)kv[it][e];
            dot = group_reduce<LPK>(dot, add_f64);
            const double sc = (j < we) ? dot - slope * (double)(i - j) : -INFINITY;
            mb = fmax(mb, sc);
            if (sub == it) sc_mine = sc;                       // lane `sub` of a group exponentiates key `it`
        }
        // values of the same keys: in flight while the exponentials are computed
#pragma unroll
        for (int it = 0; it < NIT; it++)
            kv[it] = *(const v8h *)(Vc + (size_t)min(base + it * KPI + kslot, we - 1) * D + sub * 8);
        const double m_new = fmax(m_run, mb);                  // mb = -inf: no key of this lane group in the block

        const double alpha = (m_run == -INFINITY) ? 0.0 : exp_f64(m_run - m_new);
        // keys past the end: 0 (also where m_new is still -infinity).  Not decided on mb, which skips NaN scores: a NaN
        // has to reach the sums
        const double p_mine = (sc_mine == -INFINITY) ? 0.0 : exp_f64(sc_mine - m_new);
        l_run = l_run * alpha + group_reduce<LPK>(p_mine, add_f64);     // per lane group; no other cross-lane traffic inside
        m_run = m_new;
#pragma unroll
        for (int e = 0; e < 8; e++) o[e] *= alpha;
        // the probability of key `it` is lane `it`'s of the group (0 for keys past the end)
        auto add_value = [&](auto itc) {
            constexpr int it = decltype(itc)::value;
            double p;
            if constexpr (LPK >= 8) p = group_bcast<LPK, it>(p_mine);
            else p = __shfl(p_mine, kslot * LPK + it);
#pragma unroll
            for (int e = 0; e < 8; e++) o[e] += p * (double)(float)kv[it][e];
        };
        for_constants(add_value, std::make_integer_sequence<int, NIT>());
    }
    merge_wave<LPK>(m_run, l_run, o);
    if (lane == 0) { red_m[wave] = m_run; red_l[wave] = l_run; }
#pragma unroll
    for (int e = 0; e < (LPK + 7) / 8; e++) red_o[wave][merged_dim<LPK>(lane) + e] = o[e];
    __syncthreads();
    // (with all lanes of the waves that hold a dim: the scales of the waves are exchanged between lanes)
    if (wave * 64 < D) {
        double m, l;
        const double ov = merge_waves<NW, D>(red_m, red_l, red_o, lane, min((int)threadIdx.x, D - 1), m, l);
        if (threadIdx.x >= D) return;
        if (nsplit == 1) {
            const __half hv = d2h_rn(ov / l);
            ctx[(size_t)s * H + h * D + threadIdx.x] = hv;
            flag_outlier(mask, theta, h * D + threadIdx.x, hv);
        } else {
            double *pp = partials + ((size_t)(s * nh + h) * nsplit + c) * (D + 2);
            if (threadIdx.x == 0) { pp[0] = m; pp[1] = l; }
            pp[2 + threadIdx.x] = ov;
        }
    }
}

// merges the per-range partial results of one (row, head) in a fixed order
template <int D>
__global__ void k_attn_combine(const SessTable *__restrict__ sess, int T, int nh, int CH, int nsplit,
                               const double *__restrict__ partials, __half *__restrict__ ctx,
                               uint32_t *__restrict__ mask, float theta) {
    const int h = blockIdx.x, t = blockIdx.y;
    const int s = t / T, i = sess->len[s] + (t - s * T);
    const int nvalid = min(nsplit, (i + 1 + CH - 1) / CH);
    const double *pp = partials + (size_t)(t * nh + h) * nsplit * (D + 2);
    double m = -INFINITY;
    for (int c = 0; c < nvalid; c++) m = fmax(m, pp[c * (D + 2)]);
    double l = 0.0, o = 0.0;
    for (int c = 0; c < nvalid; c++) {
        const double wgt = exp_f64(pp[c * (D + 2)] - m);
        l += wgt * pp[c * (D + 2) + 1];
        o += wgt * pp[c * (D + 2) + 2 + threadIdx.x];
    }
    const __half hv = d2h_rn(o / l);
    ctx[(size_t)t * nh * D + h * D + threadIdx.x] = hv;
    flag_outlier(mask, theta, h * D + threadIdx.x, hv);
}

template <int D>
hipError_t attn_launch(const __half *q, const SessTable *sess, int blk, int M, int T, int nh, int max_keys,
                       double *partials, __half *ctx, uint32_t *mask, float theta, float *lse, float *ctx32, hipStream_t st) {
    // Split the key range only as far as rows*heads alone leave the GPU short of about two workgroups per
    // compute unit (the kernel is bound by its fp64 arithmetic and by latency, not by the number of workgroups:
    // measured on 112 heads and 2048 keys, 4 ranges beat 9 and 16), at least 128 keys per range.
    int nsplit = max(1, 512 / (M * nh));
    nsplit = min(nsplit, max(1, max_keys / 128));
    nsplit = min(nsplit, PS_ATTN_MAX_SPLITS);
    if ((size_t)M * nh * nsplit > PS_ATTN_PARTIAL_SLOTS) nsplit = 1;
    int CH = ((max_keys + nsplit - 1) / nsplit + 63) / 64 * 64;
    if (nsplit == 1) CH = 1 << 30;
    if (T > 1 || lse) {   // the matrix-core kernel also covers T = 1; it is the one that can report the denominators
        const int B = M / T;
        // Few workgroups of the shared-tile form (64 to 128 queries each): 16-query workgroups that split the keys.
        // The line: one workgroup of the shared form per compute unit.  Below it the split wins (128 tokens, 16 heads of 64:
        // 33 -> 8 us; 3 x 117 tokens, 32 heads of 128, mean of a first and a second call: 73 -> 34 us), from it on the
        // shared conversions do (one block's prefill call of 512-token prompts, 32 heads: 2 prompts 446 us shared, 466
        // split; 4 prompts 730 and 799).
        if (B * nh * (((T + 63) / 64 + 1) / 2) < ATTN_SPLIT_BELOW) {
            if (max_keys > 512 && B * nh * ((T + 15) / 16) <= 256)
                return launch_prefill_split<D, 8>(q, sess, blk, B, T, nh, ctx, mask, theta, lse, ctx32, st);
            return launch_prefill_split<D, 4>(q, sess, blk, B, T, nh, ctx, mask, theta, lse, ctx32, st);
        }
        k_attn_prefill<D><<<(B * nh + 7) / 8 * 8 * (((T + 63) / 64 + 1) / 2), 256, D >= 64 ? (size_t)2 * (D * 64 + 16 * D * 8) : (size_t)2 * 2 * 16 * D * 8, st>>>(q, sess, blk, B, T, nh, ctx, mask, theta, lse, ctx32);
        return hipGetLastError();
    }
    if (nsplit == 2) {   // twice the waves per workgroup instead of two key ranges: nothing to merge afterwards
        k_attn_decode<D, 8><<<dim3(1, nh, M), 512, 0, st>>>(q, sess, blk, nh, 1 << 30, 1, partials, ctx, mask, theta);
        return hipGetLastError();
    }
    k_attn_decode<D, 4><<<dim3(nsplit, nh, M), 256, 0, st>>>(q, sess, blk, nh, CH, nsplit, partials, ctx, mask, theta);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || nsplit == 1) return e;
    k_attn_combine<D><<<dim3(nh, M), D, 0, st>>>(sess, T, nh, CH, nsplit, partials, ctx, mask, theta);
    return hipGetLastError();
}

}  // namespace

hipError_t ps_call_setup(const SessTable &host_table, SessTable *dev_table, uint32_t *masks, size_t n_masks, uint32_t *more, size_t n_more, hipStream_t st) {
    const size_t want = ((n_masks > n_more ? n_masks : n_more) + 255) / 256;
    k_call_setup<<<(unsigned)(want < 1 ? 1 : want > 256 ? 256 : want), 256, 0, st>>>(host_table, dev_table, masks, n_masks, more, n_more);
    return hipGetLastError();
}

hipError_t ps_attention(const __half *q, const SessTable *sess, int blk, int M, int T, int nh, int d, int max_keys,
                        double *partials, __half *ctx, uint32_t *mask, float theta, float *lse, float *ctx32,
                        hipStream_t st) {
    switch (d) {
        case 16: return attn_launch<16>(q, sess, blk, M, T, nh, max_keys, partials, ctx, mask, theta, lse, ctx32, st);
        case 32: return attn_launch<32>(q, sess, blk, M, T, nh, max_keys, partials, ctx, mask, theta, lse, ctx32, st);
        case 64: return attn_launch<64>(q, sess, blk, M, T, nh, max_keys, partials, ctx, mask, theta, lse, ctx32, st);
        case 128: return attn_launch<128>(q, sess, blk, M, T, nh, max_keys, partials, ctx, mask, theta, lse, ctx32, st);
    }
    return hipErrorInvalidValue;
}

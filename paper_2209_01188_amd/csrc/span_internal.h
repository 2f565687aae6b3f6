// Host-side state of a span, shared by the two files that implement the C ABI (forward calls; backward pass).
#pragma once
#include <vector>

#include "../../include/petals_span.h"
#include "common.h"
#include "host_util.h"

inline size_t ps_align_up(size_t v) { return (v + 255) & ~(size_t)255; }

struct BlockW {
    LinearW lin[4];
    __half *ln1g, *ln1b, *ln2g, *ln2b;
    bool loaded;
};

struct Workspace {
    SessTable *table;
    __half *a, *q, *ctx, *x1, *xa, *xb, *g;
    int8_t *xq;
    int8_t *xo;         // outlier values per (token, 16-column group) of calls of at most 64 rows
    float *sx;
    uint32_t *masks;    // [n_blocks][4][mask_words]
    uint8_t *flags;     // [n_blocks][2][hidden], right behind masks: outlier columns of the LayerNorms' outputs, one byte each (spans that take more than 64 rows)
    double *partials;
    int *ocount;
    double *wd64, *x64;
    ManyOutliers many;     // only carved when max_rows_per_call > 64
    int8_t *xd;            // wide spans: digits of the outlier columns of calls of 17 to 64 rows, see gemm_digits.h
    DigitCall digits;
    uint64_t *records;     // outlier columns that the rows of a LayerNorm tell each other, see k_layernorm_codes; null: one row
    uint32_t *record_masks;
    uint32_t *step;        // narrow spans: rows on their way between workgroups in a one-row step, see decode_row.hip
    size_t mask_words;
    size_t total;
};

// Optional per-launch timing with HIP events recorded on the caller's stream.
struct Profiler {
    bool on = false;
    std::vector<hipEvent_t> ev;        // pairs (start, stop)
    std::vector<int> cls, kind;        // kernel class of pair i; which linear it was (-1: none)
    size_t used = 0;
    bool begin(int kernel_class, int which, hipStream_t st) {
        if (!on || (used + 1) * 2 > ev.size()) return false;
        cls[used] = kernel_class;
        kind[used] = which;
        return hipEventRecord(ev[used * 2], st) == hipSuccess;
    }
    void end(bool started, hipStream_t st) {
        if (!started) return;
        (void)hipEventRecord(ev[used * 2 + 1], st);
        used++;
    }
};

struct petals_span {
    petals_span_config cfg;
    Profiler prof;
    uint8_t *wmem;
    Workspace ws;
    std::vector<BlockW> blocks;
    double slopes[PS_MAX_HEADS];
    int open_sessions;
    // optional cache of the transposed dequantized weights for the backward pass: [block][linear]
    __half *bwd_cache = nullptr;
    uint32_t step_patience = 1u << 24;   // polls for a row of a one-launch step, of half a microsecond and more each
    uint32_t norm_patience = 10000;      // 100 us: what a row of a LayerNorm waits for the others' outlier columns
    std::vector<uint8_t> bwd_cached;     // 1: the tiles of (block, linear) are in the cache
};

struct petals_session {
    petals_span *span;
    __half *kv;
    int cap, len;
};

// What a forward pass keeps for the backward pass, per block: the block's input x[b] (x[n_blocks] is the
// span's output), queries, the attention context before its fp16 rounding, x1 = x + attention branch, the sum
// fed to GeLU, and the log of the softmax denominators.  Keys and values stay in the (internal) caches.
struct SaveSet {
    std::vector<__half *> x, q, x1, pre;
    std::vector<float *> lse, ctx32;
};

// what a call of M rows clears first: nothing, the masks, or the masks and the flags behind them
inline size_t ps_mask_clear_words(const petals_span_config &c, const Workspace &ws, int M) {
    return M <= 1 ? 0 : (size_t)c.n_blocks * 4 * ws.mask_words + (M > 64 ? (size_t)c.n_blocks * 2 * c.hidden / 4 : 0);
}
// ... and in 32-bit words the records of its LayerNorms
inline size_t ps_record_words(const Workspace &ws, int M) {
    return M <= 1 || !ws.records || M > PS_NORM_ROWS_MAX ? 0 : (size_t)M * PS_NORM_RECORD_WORDS;
}
// N and K of linear `which` (0 qkv, 1 dense, 2 up, 3 down)
void ps_linear_dims(const petals_span_config &c, int which, int *N, int *K);
int ps_check_config(const petals_span_config *c);
// The blocks of the span on M = B*T rows whose session table already sits in the workspace.
// save == nullptr: intermediates live in the workspace.  Otherwise they are written where save says and
// the up linear also stores the sum it feeds to GeLU; then hidden_out may be null, and the down linear of the
// last block (whose result only hidden_out would receive) is skipped.
int ps_forward_blocks(petals_span *sp, int M, int T, int max_keys, const __half *hidden_in, __half *hidden_out,
                      const SaveSet *save, hipStream_t st);

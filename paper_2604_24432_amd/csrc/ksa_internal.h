// Internal declarations shared by the host-side translation units of libksa.
#ifndef KSA_INTERNAL_H_
#define KSA_INTERNAL_H_

#include <algorithm>
#include <numeric>
#include <vector>

#include "ksa.h"
#include "ksa_schedule.h"

struct ksa_layout {
    ksa_params p;
    int64_t aug_len;      // L
    int32_t n_chunks;     // J
    std::vector<KsaWorkItem> items;   // one per query tile, heaviest first
    std::vector<KsaWgEntry> entries;  // one per workgroup
    bool ragged = false;              // some run's last key tile reaches past the end of its index space
    int32_t running_text = INT32_MAX, running_sum = INT32_MAX;   // first row of the first text / summary item with running_max
    int32_t head_stack = 1;           // query heads per workgroup (1, 2 or 4)
    bool dq_direct = false;           // ... and dQ
    bool dkv_direct = false;          // dK and dV take the kernel of ksa_prefill_bwd_dkv.hip where tiles are split
    bool dkv_unsplit_direct = false;  // ... and where none is
    bool direct = false;              // the forward pass takes the kernel for short key runs (see takes_direct)
    int32_t q_tile_rows = KSA_Q_TILE; // rows of a query tile = KSA_Q_TILE / head_stack
    std::vector<KsaDkvEntry> dkv_entries;   // backward dK / dV, per (batch, KV head), longest first
    std::vector<KsaDkvSplit> dkv_splits;    // the tiles whose work is dealt to several workgroups
    int32_t dkv_slots = 0;                  // scratch slots per (batch, KV head)
    // device copies (owned), valid on `device` once uploaded
    int device = -1;
    void *d_items = nullptr;          // the allocation: items, entries, dkv_entries, dkv_splits
    void *d_entries = nullptr;
    void *d_dkv = nullptr;            // dkv_entries, then dkv_splits
};

// Validates the problem statement; returns KSA_OK or the error.
int ksa_validate_params(const ksa_params *p);

// Launchers implemented in the .hip files.  All pointers device, strides in elements.
// Bytes from the first to behind the last element of a [batch, rows, heads, d] bf16 tensor with these {batch, row, head}
// strides, and whether two ranges of memory share no byte.
inline int64_t ksa_extent(const int64_t strides[3], int64_t batch, int64_t rows, int64_t heads, int64_t d) {
    return 2 * ((batch - 1) * strides[0] + (rows - 1) * strides[1] + (heads - 1) * strides[2] + d);
}
inline bool ksa_apart(const void *x, int64_t x_bytes, const void *y, int64_t y_bytes) {
    const char *p = static_cast<const char *>(x), *r = static_cast<const char *>(y);
    return p + x_bytes <= r || p >= r + y_bytes;
}

struct KsaPrefillLaunch {
    const void *q, *k, *v;
    void *o;
    float *lse;
    int64_t q_strides[3], kv_strides[3], o_strides[3];
    const KsaWorkItem *items;
    const KsaWgEntry *entries;
    int32_t n_entries;
    bool ragged;              // some run's last key tile reaches past the end of its index space
    int32_t running_text, running_sum;   // first row of the first text / summary work item with KsaWorkItem::running_max
    int32_t head_stack;                           // query heads per workgroup
    ksa_params p;
    int64_t aug_len;
    void *workspace;          // key-major copy of V, written by the launch itself
    bool direct;              // run the kernel for short key runs instead (ksa_prefill_direct.hip)
    int32_t phases;           // bit 0: write the key-major copy of V; bit 1: run the attention kernels
    size_t workspace_bytes;
};
size_t ksa_prefill_workspace_size(const ksa_params &p);
int ksa_launch_prefill(const KsaPrefillLaunch &a, void *stream);
// The kernel for short key runs and chunk shapes that are no powers of two (ksa_prefill_direct.hip).  knorm_parts, knorm:
// the row norms in the workspace, of parts of the rows (room for one per 64 rows) and of the whole (batch, KV head).
int ksa_launch_prefill_direct(const KsaPrefillLaunch &a, float *knorm_parts, float *knorm, void *stream);
// How many rows of the augmented sequence the rows of one key tile of that kernel may span where the tile holds the last
// summaries and the first text rows of a query tile's key list (at most 63 of each; q_rows rows per query tile).  A text
// tile's summaries end, and its text begins, C chunks before chunks that lie at most ceil((q_rows - 1) / c) apart.  A summary
// tile's text begins in the chunk of its first row while its last summaries lie in the chunk of its last row, up to
// ceil((q_rows - 1) / m) chunks later, whatever the number of summaries in the key tile.
inline int64_t ksa_mixed_tile_rows(int64_t c, int64_t m, int64_t q_rows) {
    if (m <= 0) return 0;   // no summaries, no such tile
    auto chunks = [&](int64_t rows, int64_t per) { return (rows + per - 1) / per; };
    const int64_t text = chunks(63, m) + chunks(63, c) + chunks(q_rows, c), sums = chunks(q_rows, m) + chunks(63, c);
    return ((text > sums ? text : sums) + 1) * (c + m);
}

// About how many keys the longest list of one of its query tiles holds, none less.  A text tile's text begins C chunks before the chunk of
// its first row, whose place in that chunk is a multiple of gcd(c, q_rows); a summary tile sees the chunks of its rows and their summaries.
inline int64_t ksa_longest_list(int64_t c, int64_t m, int64_t C, int64_t n_text, int64_t n_sum, int64_t q_rows) {
    const int64_t chunks = (n_text - 1) / c;
    const int64_t text = (chunks > C ? (chunks - C) * m : 0) + std::min(n_text, C * c + q_rows + c - std::gcd(c, q_rows));
    if (m <= 0) return text;
    const int64_t rows = std::min(n_sum, q_rows + m - std::gcd(m, q_rows));
    return std::max(text, std::min((rows + m - 1) / m * c, n_text) + rows);
}
// Whether a launch of that kernel (grad: of the one for dQ) takes eight waves per workgroup, the second four every other key tile.  With no
// more workgroups than compute units that halves the chain of tiles.  us, four waves / eight, forward (backward): head_dim 64 12/4 heads,
// 2000 tokens, c 48, m 6 30.5 / 23.4 (78.7 / 69.2), 2 x 1024, c 64, m 8 25.3 / 21.2 (58.2 / 51.0), 1 head, 512 tokens 12.1 / 11.6 (29.9 /
// 28.3); head_dim 128 16/16 heads, 1024 tokens 31.1 / 26.7 (67.8 / 61.7), 1 head, 3000 tokens 17.7 / 16.8 (61.1 / 60.0), but with few tiles
// in a list (1 head, window of 255) 13.8 / 14.3, and with four heads per workgroup, whose waves all read the same keys, 512 tokens 15.9 /
// 16.6 (58.2 / 59.0), 700 in the paper's form 22.6 / 22.0 (81.2 / 81.4).  Lists of one key tile leave nothing to the second four (head_dim 64,
// 32/8 heads, 48 tokens, c 48 5.56 / 6.52 (23.6 / 24.0), c 8, window of 128 6.11 / 7.12 (19.8 / 20.3)), a few keys more hardly anything forward
// (70 keys 6.38 / 6.77 (28.4 / 28.0), but 80 keys, 700 tokens, 12/4 heads, c 16, window of 32 8.80 / 8.27 (28.1 / 27.1)).
inline bool ksa_two_teams(int head_dim, int64_t n_wg, int head_stack, int64_t longest_list, bool grad) {
    if (n_wg > 256) return false;
    return head_dim == 64 ? longest_list > (grad ? 64 : 72) : head_stack == 1 && longest_list > 8 * 64;
}

struct KsaPrefillBwdLaunch {
    const void *q, *k, *v, *o, *d_o;
    const float *lse;
    void *dq, *dk, *dv;
    int64_t q_strides[3], kv_strides[3], o_strides[3], dq_strides[3], dkv_strides[3];
    const KsaWorkItem *items;
    const KsaWgEntry *entries;
    int32_t n_entries;
    int32_t head_stack;       // query heads per workgroup of the schedule
    const KsaDkvEntry *dkv_entries;   // NULL: every key tile is one workgroup
    const KsaDkvSplit *dkv_splits;
    int32_t n_dkv_entries, n_dkv_splits;
    bool dkv_direct, dkv_unsplit_direct;   // dK and dV by the kernel of ksa_prefill_bwd_dkv.hip: with split tiles, without
    bool dq_direct;                   // dQ by the kernel for short key runs (ksa_prefill_direct.hip)
    ksa_params p;
    int64_t aug_len;
    void *workspace;          // delta_i = dO_i . O_i per (batch, query head, row), fp32
    size_t workspace_bytes;
};
size_t ksa_prefill_bwd_workspace_size(const ksa_params &p, int64_t aug_len);
int ksa_launch_prefill_bwd(const KsaPrefillBwdLaunch &a, void *stream);
// dQ by the kernel for short key runs and odd chunk shapes (ksa_prefill_direct.hip); stats: the row statistics.
int ksa_launch_dq_direct(const KsaPrefillBwdLaunch &a, const float *stats, void *stream);
// dK and dV (ksa_prefill_bwd_dkv.hip); scratch: where the partial sums of split key tiles go, NULL: no tile is split; entries:
// workgroups per (batch, KV head), whose number the caller has checked to be a grid's.
void ksa_launch_dkv_direct(const KsaPrefillBwdLaunch &a, const float *stats, float *scratch, int entries, void *stream);
// Second step of the split dK / dV tiles (ksa_prefill_bwd_sum.hip).
struct KsaDkvSumArgs {
    const float *scratch;
    const KsaDkvSplit *splits;
    void *dk, *dv;
    int64_t strides[3];       // of dk and dv, {batch, row, head}
    int32_t n_splits, sum_tiles, n_text, n_sum, c, m, n_kv_heads, n_bh, head_dim;
    float scale;
};
void ksa_launch_dkv_sum(const KsaDkvSumArgs &a, void *stream);

struct KsaDecodeLaunch {
    const void *q, *k_cache, *v_cache;
    const int32_t *pos;
    void *o;
    float *lse;
    int64_t cache_strides[3];
    float *workspace;
    int32_t n_splits;         // spans per sequence; 0: dealt by the sequences' lengths (batch <= 64)
    int32_t n_spans;          // spans per KV head: batch * n_splits, or those to deal (at least two per sequence)
    bool wide;                // workgroups of 1024 threads (512 with eight query heads per KV head) instead of 256
    int32_t summary_capacity;
    int32_t kind;             // KSA_ROW_TEXT: pos is a text index; KSA_ROW_SUMMARY: pos is a summary ordinal
    ksa_params p;
};
int ksa_launch_decode(const KsaDecodeLaunch &a, void *stream);
// Device address (current device) of the library's static scratch array of KSA_DECODE_STATIC_SCRATCH_BYTES bytes.
int ksa_decode_static_scratch(float **ptr);

struct KsaCacheFillLaunch {
    const void *k, *v;
    void *k_cache, *v_cache;
    int64_t kv_strides[3], cache_strides[3];
    int64_t n_prefill;
    int32_t summary_capacity;
    ksa_params p;
};
int ksa_launch_cache_fill(const KsaCacheFillLaunch &a, void *stream);

struct KsaCacheAppendLaunch {
    const void *k_new, *v_new;
    const int32_t *pos;
    void *k_cache, *v_cache;
    int64_t cache_strides[3];
    int32_t kind;
    int32_t summary_capacity;
    ksa_params p;
};
int ksa_launch_cache_append(const KsaCacheAppendLaunch &a, void *stream);
int ksa_decode_default_splits(const ksa_params *p);

#endif

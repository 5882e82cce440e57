// C-ABI entry points that touch the GPU: schedule upload, prefill and decode launches.
// Every argument check happens before the first HIP call.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>

#include "ksa_internal.h"

namespace {

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

void default_strides(int64_t out[3], const int64_t *given, int64_t d0, int64_t d1, int64_t d2) {
    // contiguous [x, d0-dim, d1-dim, d2] -> strides of the three leading dims
    if (given) {
        out[0] = given[0], out[1] = given[1], out[2] = given[2];
    } else {
        out[2] = d2;
        out[1] = d1 * d2;
        out[0] = d0 * d1 * d2;
    }
}

bool strides_ok(const int64_t s[3]) {
    // rows must keep 16-byte alignment of the head vectors (bf16: multiples of 8 elements)
    return s[0] >= 0 && s[1] > 0 && s[2] > 0 && s[0] % 8 == 0 && s[1] % 8 == 0 && s[2] % 8 == 0;
}

}  // namespace

extern "C" {

void ksa_layout_destroy(ksa_layout *lay) {
    if (!lay) return;
    if (lay->d_items) (void)hipFree(lay->d_items);
    delete lay;
}

int ksa_layout_upload(ksa_layout *lay) {
    if (!lay) return KSA_ERR_INVALID_ARG;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return KSA_ERR_HIP;
    if (lay->d_items && lay->device == dev) return KSA_OK;
    if (lay->d_items) {
        (void)hipFree(lay->d_items);
        lay->d_items = lay->d_entries = lay->d_dkv = nullptr;
    }
    // the parts follow each other in one allocation (all records are multiples of 16 bytes)
    static_assert(sizeof(KsaWorkItem) % 16 == 0 && sizeof(KsaWgEntry) % 16 == 0 && sizeof(KsaDkvEntry) % 16 == 0, "alignment of the parts");
    const size_t ib = lay->items.size() * sizeof(KsaWorkItem), eb = lay->entries.size() * sizeof(KsaWgEntry);
    const size_t kb = lay->dkv_entries.size() * sizeof(KsaDkvEntry), sb = lay->dkv_splits.size() * sizeof(KsaDkvSplit);
    std::vector<unsigned char> all;
    try {
        all.resize(ib + eb + kb + sb);
    } catch (...) {
        return KSA_ERR_OUT_OF_MEMORY;
    }
    std::memcpy(all.data(), lay->items.data(), ib);
    std::memcpy(all.data() + ib, lay->entries.data(), eb);
    std::memcpy(all.data() + ib + eb, lay->dkv_entries.data(), kb);
    if (sb > 0) std::memcpy(all.data() + ib + eb + kb, lay->dkv_splits.data(), sb);
    void *dst = nullptr;
    if (hipMalloc(&dst, all.size()) != hipSuccess) return KSA_ERR_HIP;
    if (hipMemcpy(dst, all.data(), all.size(), hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipFree(dst);
        return KSA_ERR_HIP;
    }
    lay->d_items = dst;
    lay->d_entries = static_cast<char *>(dst) + ib;
    lay->d_dkv = static_cast<char *>(dst) + ib + eb;
    lay->device = dev;
    return KSA_OK;
}

size_t ksa_prefill_workspace_bytes(const ksa_layout *lay) { return lay ? ksa_prefill_workspace_size(lay->p) : 0; }

namespace {

int prefill_call(ksa_layout *lay, const void *q, const void *k, const void *v, void *o, float *lse,
                 const int64_t q_strides[3], const int64_t kv_strides[3], const int64_t o_strides[3], void *workspace,
                 size_t workspace_bytes, void *stream, int32_t phases) {
    if (!lay || !q || !k || !v || !o || !workspace) return KSA_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o)) return KSA_ERR_INVALID_ARG;
    if (lse && (reinterpret_cast<uintptr_t>(lse) & 3u)) return KSA_ERR_INVALID_ARG;
    if (!aligned16(workspace)) return KSA_ERR_INVALID_ARG;
    if (workspace_bytes < ksa_prefill_workspace_size(lay->p)) return KSA_ERR_WORKSPACE_TOO_SMALL;
    const ksa_params &p = lay->p;
    KsaPrefillLaunch a;
    default_strides(a.q_strides, q_strides, lay->aug_len, p.n_q_heads, p.head_dim);
    default_strides(a.kv_strides, kv_strides, lay->aug_len, p.n_kv_heads, p.head_dim);
    default_strides(a.o_strides, o_strides, lay->aug_len, p.n_q_heads, p.head_dim);
    if (!strides_ok(a.q_strides) || !strides_ok(a.kv_strides) || !strides_ok(a.o_strides)) return KSA_ERR_INVALID_ARG;
    const int rc = ksa_layout_upload(lay);
    if (rc != KSA_OK) return rc;
    a.q = q, a.k = k, a.v = v, a.o = o, a.lse = lse;
    a.items = static_cast<const KsaWorkItem *>(lay->d_items);
    a.entries = static_cast<const KsaWgEntry *>(lay->d_entries);
    a.n_entries = (int32_t)lay->entries.size();
    a.ragged = lay->ragged;
    a.running_text = lay->running_text, a.running_sum = lay->running_sum;
    a.head_stack = lay->head_stack;
    a.p = p;
    a.aug_len = lay->aug_len;
    a.workspace = workspace;
    a.workspace_bytes = workspace_bytes;
    a.direct = lay->direct;
    a.phases = phases;
    return ksa_launch_prefill(a, stream);
}

}  // namespace

int ksa_prefill_fwd(ksa_layout *lay, const void *q, const void *k, const void *v, void *o, float *lse,
                    const int64_t q_strides[3], const int64_t kv_strides[3], const int64_t o_strides[3],
                    void *workspace, size_t workspace_bytes, void *stream) {
    return prefill_call(lay, q, k, v, o, lse, q_strides, kv_strides, o_strides, workspace, workspace_bytes, stream, 3);
}

int ksa_prefill_relayout_v(ksa_layout *lay, const void *v, const int64_t kv_strides[3], void *workspace,
                           size_t workspace_bytes, void *stream) {
    // the attention tensors are not touched in this phase; v stands in for them in the shared argument checks
    return prefill_call(lay, v, v, v, workspace, nullptr, nullptr, kv_strides, nullptr, workspace, workspace_bytes, stream, 1);
}

size_t ksa_prefill_bwd_workspace_bytes(const ksa_layout *lay) {
    return lay ? ksa_prefill_bwd_workspace_size(lay->p, lay->aug_len) : 0;
}

int ksa_prefill_bwd(ksa_layout *lay, const void *q, const void *k, const void *v, const void *o, const float *lse,
                    const void *d_o, void *dq, void *dk, void *dv, const int64_t q_strides[3],
                    const int64_t kv_strides[3], const int64_t o_strides[3], const int64_t dq_strides[3],
                    const int64_t dkv_strides[3], void *workspace, size_t workspace_bytes, void *stream) {
    if (!lay || !q || !k || !v || !o || !lse || !d_o || !dq || !dk || !dv || !workspace) return KSA_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k) || !aligned16(v) || !aligned16(o) || !aligned16(d_o) || !aligned16(dq) ||
        !aligned16(dk) || !aligned16(dv) || !aligned16(workspace))
        return KSA_ERR_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(lse) & 3u) return KSA_ERR_INVALID_ARG;
    if (workspace_bytes < ksa_prefill_bwd_workspace_size(lay->p, lay->aug_len)) return KSA_ERR_WORKSPACE_TOO_SMALL;
    const ksa_params &p = lay->p;
    KsaPrefillBwdLaunch a;
    default_strides(a.q_strides, q_strides, lay->aug_len, p.n_q_heads, p.head_dim);
    default_strides(a.kv_strides, kv_strides, lay->aug_len, p.n_kv_heads, p.head_dim);
    default_strides(a.o_strides, o_strides, lay->aug_len, p.n_q_heads, p.head_dim);
    default_strides(a.dq_strides, dq_strides, lay->aug_len, p.n_q_heads, p.head_dim);
    default_strides(a.dkv_strides, dkv_strides, lay->aug_len, p.n_kv_heads, p.head_dim);
    if (!strides_ok(a.q_strides) || !strides_ok(a.kv_strides) || !strides_ok(a.o_strides) ||
        !strides_ok(a.dq_strides) || !strides_ok(a.dkv_strides))
        return KSA_ERR_INVALID_ARG;
    const int rc = ksa_layout_upload(lay);
    if (rc != KSA_OK) return rc;
    a.q = q, a.k = k, a.v = v, a.o = o, a.d_o = d_o, a.lse = lse;
    a.dq = dq, a.dk = dk, a.dv = dv;
    a.items = static_cast<const KsaWorkItem *>(lay->d_items);
    a.entries = static_cast<const KsaWgEntry *>(lay->d_entries);
    a.n_entries = (int32_t)lay->entries.size();
    a.head_stack = lay->head_stack;
    a.dkv_entries = static_cast<const KsaDkvEntry *>(lay->d_dkv);
    a.n_dkv_entries = (int32_t)lay->dkv_entries.size();
    a.dkv_splits = reinterpret_cast<const KsaDkvSplit *>(a.dkv_entries + a.n_dkv_entries);
    a.n_dkv_splits = (int32_t)lay->dkv_splits.size();
    a.dq_direct = lay->dq_direct;
    a.dkv_direct = lay->dkv_direct, a.dkv_unsplit_direct = lay->dkv_unsplit_direct;
    a.p = p;
    a.aug_len = lay->aug_len;
    a.workspace = workspace;
    a.workspace_bytes = workspace_bytes;
    return ksa_launch_prefill_bwd(a, stream);
}

namespace {

// a span's record per query head: head_dim partial outputs + running max + running sum, fp32
size_t record_bytes(const ksa_params *p) { return (size_t)p->n_q_heads * (p->head_dim + 2) * sizeof(float); }

// Spans of a call that leaves their number to the library.
struct DecodePlan {
    int32_t n_splits;   // spans per sequence; 0: n_spans per KV head dealt by the sequences' lengths
    int32_t n_spans;    // per KV head, all sequences together
    bool wide;          // workgroups of 1024 threads (512 with eight query heads per KV head) instead of 256
};

/*
 * rows: the most that a sequence can read.  All times below in us, per call, the same number of spans for every sequence unless they
 * are called dealt; w: rows in units of 256 bytes of K, "n wide" / "n": n workgroups of 1024 / 256 threads.
 *
 * One span per sequence has no merge kernel.  It is ahead up to w = 256 (16/16 heads, 384 rows: batch 1 6.5, 128 workgroups 5.8;
 * 32/8 heads: batch 1 9.3, 128 7.5), with 64 and more (sequence, KV head) pairs up to 384 (32/8, 384 rows, batch 16: 10.4, 512 11.2),
 * and where it fills the chip once (256 pairs, wide: 16/16 heads, 1128 rows 19.7, 768 22.4; 8/4 heads 21.5, 24.2) or more
 * (512 pairs, 640 rows: 24.8, 1024 31.2).
 *
 * Workgroups go to the compute units evenly, so a launch of a multiple of 256 ends together (32K, batch 4, 32/8 heads: 192 23.2, 256
 * 20.9, 320 22.8, 384 21.3, 512 19.7): the number of spans is taken near `want` where the last round is best filled.
 * `want`: short launches want a workgroup per unit (12/12 heads, d 64, 2000 rows: 256 7.6, 512 8.9); with more rows the loads in flight count:
 * two on each unit with four heads per KV head (batch 4, 3808 rows: 256 18.0, 512 15.4, 768 16.3), three with one or two (8/4 heads, batch
 * 8, 2176 rows: 256 wide 11.2, 512 11.1, 768 10.7), five with one and enough pairs (8/8 heads, batch 16, 3120 rows: 768 27.2, 1280 26.4; batch 1,
 * 118744 rows: 768 77.8, 1280 79.1), a wide one with eight (batch 64, 1128 rows: 256 wide 12.9, 512 14.0) up to 250 000 rows (64/8 heads, batch 1,
 * 230 000: 256 27.7, 512 29.5; batch 4 26.6, 25.9; 280 000: 30.8, 29.4).  The other lines, both sides: 30 000 rows, 8/8 heads, batch 1,
 * 24 000 256 8.5, 512 8.8, 4/1, batch 3 13.6, 14.6, 32/8, batch 4, 36 000 12.5, 11.5; 65 000, 8/8, batch 4, 55 000 512 9.5, 768 10.0, 75 000
 * 11.1, 10.8; 130 000, the same, 110 000 768 12.6, 1280 13.5, 150 000 15.9, 15.2.  One sequence takes no more than that however long it is (850 000
 * rows: 64/8 heads 512 74.9, 1536 88.6; 32/8 72.0, 78.7).  Spans of
 * about 24 rows at least (16 where that fills a round better), and up to 64 per sequence, which the merge kernel takes at once (8/1 heads,
 * batch 1, 3808 rows: 64 10.4, 192 13.3); more have 768 rows or, within one round, 512 (2/1 heads, batch 3, 50000 rows: 255 19.4, 291 22.4).
 *
 * Spans dealt by the sequences' lengths cost 1 - 1.5 to work out.  Lengths 1 : 4, batch 64 at 128K 511 -> 457, batch 16 133 -> 118, batch 8 in
 * the paper's form 74.5 -> 68.7; all alike 658 -> 652, 173 -> 169, 97 -> 92 (before: about 1536 workgroups, none below 768 rows).  Batch 64:
 * 512 workgroups 537, 768 507, 1536 457.  They pay from 800 000 rows on (batch 16, 16/8 heads, 850 000 rows, lengths 1 : 4 / alike: 768 the same
 * for all 57.6 / 73.5, dealt 50.5 / 70.8), with up to 128 pairs and four or eight heads per KV head from 500 000 (batch 33, 8/2, 760 000 rows 59.3 / 68.1, 512
 * dealt 48.2 / 69.1; batch 12, 4/1 55.3 / 64.2, 46.4 / 64.9), with two to four sequences from a million (batch 4, 32/8, 700 000 rows 47.2 / 61.0, 48.1 /
 * 61.7); more than 64 sequences are never dealt and take 1536 workgroups from 800 000 rows on (batch 96, 16/4, 3 million rows 208, 768 224).
 * Two and more per sequence, or there is nothing to deal: with one and two heads
 * per KV head three where it would be less than two and a half (lengths 1 : 4 / alike, batch 60, 32/16, 1600 rows, 1.3 99.9 / 126, three 88.0 /
 * 127; batch 33, 32/16, 9000 rows, 2.4 249 / 411, three 246 / 374; but batch 64, 16/8, 6400 rows, 2.5 170 / 248, three 190 / 262), with more
 * heads two (batch 28, 128/32, 3500 rows, 1.7 177 / 271, two 178 / 250, three 178 / 263).  From 1024 pairs on the workgroups balance each
 * other and nothing is dealt (dealt one by one / the same number each: batch 64, 64/32 heads, 2100 rows 237 / 341, 231 / 335; batch 33,
 * 64/32 heads, 4000 rows 252 / 366, two each 229 / 345), with two each up to 1500 pairs (batch 44, 128/32, 3500 rows 271 / 391, one 283 / 401).
 *
 * fit: for how many spans of a KV head there is room, one per sequence at least.
 */
DecodePlan plan_decode(const ksa_params *p, int64_t rows, int64_t fit) {
    const int64_t groups = (int64_t)p->batch * p->n_kv_heads, total = groups * rows;
    const int64_t w = rows * p->head_dim / 128;
    const int32_t heads = p->n_q_heads / p->n_kv_heads;
    auto wide = [&](int64_t splits) {
        if (splits * groups > 256) return false;
        const int64_t per = w / splits;
        return per >= (heads == 8 ? 64 : heads == 4 ? (splits == 1 ? 900 : 280) : 300);
    };
    if (w <= (groups < 64 ? 256 : 384) || (groups >= 192 && groups <= 256 && rows < 1536) ||
        (groups > 256 && rows < (groups >= 512 ? 1536 : 768)))
        return {1, p->batch, groups <= 256 && (wide(1) || (w >= 384 && groups >= 192))};
    int64_t want = total < 30000 ? 256 : heads <= 2 ? (total < 65000 ? 512 : heads == 2 || groups < 16 || total < 130000 ? 768 : 1280)
                                                    : heads == 4 || total > 250000 ? 512 : 256;
    const int64_t enough = heads <= 2 ? 5 * p->batch / 2 : 2 * p->batch;   // dealt spans per KV head
    const int64_t large = p->batch <= 4 ? 1000000 : heads >= 4 && groups <= 128 ? 500000 : 800000;
    const bool deal = total >= large && p->batch > 1 && p->batch <= 64 && groups < 1024 && fit >= enough;
    if (deal)
        want = heads == 1 ? 1536 : heads == 2 ? (groups <= 256 ? 768 : 1280) : groups <= 64 || total < 1000000 ? 512 : groups <= 128 ? 768 : 1536;
    else if (total >= 800000 && p->batch > 4)
        want = groups >= 1024 ? 2048 : 1536;
    want = std::max<int64_t>(std::min(want, total / 24), 1);
    if (deal) {
        const int64_t spans = want / p->n_kv_heads;
        return {0, (int32_t)std::min<int64_t>(spans >= enough ? spans : (heads <= 2 ? 3 : 2) * p->batch, fit), false};
    }
    const int64_t most = std::max({(int64_t)64, rows / 768, std::min(rows / 512, 256 / groups)});
    const int64_t hi = std::max<int64_t>(1, std::min({3 * want / (2 * groups), most, fit / p->batch}));
    const int64_t lo = std::max<int64_t>(1, std::min({want / (2 * groups), hi, std::max<int64_t>(64, hi / 2)}));
    int64_t best = 1;
    double best_score = -1e30;
    auto look_at = [&](int64_t s) {
        const int64_t n = s * groups, places = (n + 255) / 256 * 256;
        const double score = (double)n / places - 0.25 * std::fabs(std::log((double)n / want));
        if (score > best_score) best = s, best_score = score;
    };
    // (from 64 workgroups on the score rises up to the last number of a round; below, up to `want`)
    for (const int64_t s : {want / groups, want / groups + 1}) look_at(std::min(std::max(s, lo), hi));
    for (int64_t round = (lo * groups + 255) / 256; round <= (hi * groups + 255) / 256; ++round) look_at(std::min(std::max(256 * round / groups, lo), hi));
    return {(int32_t)best, (int32_t)(p->batch * best), wide(best)};
}

// records no larger than the static array of ksa_decode_fwd_static, unless those of the least number are
int64_t most_spans(const ksa_params *p) {
    const int64_t most = KSA_DECODE_STATIC_SCRATCH_BYTES / (p->batch * record_bytes(p));
    return p->batch * std::max<int64_t>(most, ksa_decode_default_splits(p));
}

int64_t most_rows(const ksa_params *p, int32_t kind) {
    if (kind == KSA_ROW_SUMMARY) return (int64_t)p->chunk_len + p->n_summary;
    return (int64_t)(p->n_text / p->chunk_len) * p->n_summary + (int64_t)(p->window_chunks + 1) * p->chunk_len;
}

}  // namespace

size_t ksa_decode_workspace_bytes(const ksa_params *p, int32_t n_splits) {
    if (ksa_validate_params(p) != KSA_OK || n_splits < 0) return 0;
    int64_t spans = (int64_t)p->batch * n_splits;
    if (n_splits == 0) {   // (no less than the least that a call accepts)
        spans = (int64_t)p->batch * ksa_decode_default_splits(p);
        for (const int32_t kind : {KSA_ROW_TEXT, KSA_ROW_SUMMARY}) spans = std::max<int64_t>(spans, plan_decode(p, most_rows(p, kind), most_spans(p)).n_spans);
    }
    return (size_t)spans * record_bytes(p);
}

namespace {

int decode_call(const ksa_params *p, int32_t kind, const void *q, const void *k_cache, const void *v_cache,
                const int32_t *pos, void *o, float *lse, const int64_t cache_strides[3], void *workspace,
                size_t workspace_bytes, int32_t n_splits, void *stream) {
    int32_t s_cap = 0, rows = 0;
    const int rc = ksa_cache_geometry(p, &s_cap, &rows);
    if (rc != KSA_OK) return rc;
    if (!q || !k_cache || !v_cache || !pos || !o || !workspace) return KSA_ERR_INVALID_ARG;
    if (!aligned16(q) || !aligned16(k_cache) || !aligned16(v_cache) || !aligned16(o) || !aligned16(workspace))
        return KSA_ERR_INVALID_ARG;
    if (n_splits < 0 || n_splits > 1024) return KSA_ERR_INVALID_ARG;
    if (kind == KSA_ROW_SUMMARY && p->n_summary == 0) return KSA_ERR_INVALID_ARG;
    if (p->n_q_heads / p->n_kv_heads > 8) return KSA_ERR_UNSUPPORTED;
    const int64_t spans = (int64_t)p->batch * (n_splits != 0 ? n_splits : ksa_decode_default_splits(p));
    if (workspace_bytes < (size_t)spans * record_bytes(p)) return KSA_ERR_WORKSPACE_TOO_SMALL;
    DecodePlan plan = {n_splits, (int32_t)spans, n_splits > 1 && spans * p->n_kv_heads <= 256};
    if (n_splits == 0)
        plan = plan_decode(p, most_rows(p, kind), std::min<int64_t>(most_spans(p), workspace_bytes / record_bytes(p)));
    KsaDecodeLaunch a;
    default_strides(a.cache_strides, cache_strides, p->n_kv_heads, rows, p->head_dim);
    if (!strides_ok(a.cache_strides)) return KSA_ERR_INVALID_ARG;
    a.q = q, a.k_cache = k_cache, a.v_cache = v_cache, a.pos = pos, a.o = o, a.lse = lse;
    a.workspace = static_cast<float *>(workspace);
    a.n_splits = plan.n_splits, a.n_spans = plan.n_spans, a.wide = plan.wide;
    a.summary_capacity = s_cap;
    a.kind = kind;
    a.p = *p;
    if (a.p.softmax_scale <= 0.f) a.p.softmax_scale = 1.0f / __builtin_sqrtf((float)p->head_dim);
    return ksa_launch_decode(a, stream);
}

}  // namespace

int ksa_decode_fwd(const ksa_params *p, const void *q, const void *k_cache, const void *v_cache,
                   const int32_t *pos, void *o, float *lse, const int64_t cache_strides[3], void *workspace,
                   size_t workspace_bytes, int32_t n_splits, void *stream) {
    return decode_call(p, KSA_ROW_TEXT, q, k_cache, v_cache, pos, o, lse, cache_strides, workspace, workspace_bytes,
                       n_splits, stream);
}

int ksa_decode_fwd_static(const ksa_params *p, const void *q, const void *k_cache, const void *v_cache,
                          const int32_t *pos, void *o, float *lse, const int64_t cache_strides[3], int32_t n_splits,
                          void *stream) {
    // size check first (host arithmetic only), so that an oversized problem is refused even without a GPU
    const int rc = ksa_validate_params(p);
    if (rc != KSA_OK) return rc;
    if (n_splits < 0 || n_splits > 1024) return KSA_ERR_INVALID_ARG;
    const int32_t splits = n_splits == 0 ? ksa_decode_default_splits(p) : n_splits;
    const size_t need = ksa_decode_workspace_bytes(p, splits);
    if (need > KSA_DECODE_STATIC_SCRATCH_BYTES) return KSA_ERR_SCRATCH_LIMIT;
    if (!q || !k_cache || !v_cache || !pos || !o) return KSA_ERR_INVALID_ARG;
    float *buf = nullptr;
    const int rs = ksa_decode_static_scratch(&buf);
    if (rs != KSA_OK) return rs;
    return decode_call(p, KSA_ROW_TEXT, q, k_cache, v_cache, pos, o, lse, cache_strides, buf, KSA_DECODE_STATIC_SCRATCH_BYTES,
                       n_splits, stream);
}

int ksa_decode_summary_fwd(const ksa_params *p, const void *q, const void *k_cache, const void *v_cache,
                           const int32_t *ordinal, void *o, float *lse, const int64_t cache_strides[3],
                           void *workspace, size_t workspace_bytes, int32_t n_splits, void *stream) {
    return decode_call(p, KSA_ROW_SUMMARY, q, k_cache, v_cache, ordinal, o, lse, cache_strides, workspace,
                       workspace_bytes, n_splits, stream);
}

int ksa_cache_from_prefill(const ksa_params *p, int64_t n_prefill, const void *k, const void *v,
                           const int64_t kv_strides[3], void *k_cache, void *v_cache,
                           const int64_t cache_strides[3], void *stream) {
    int32_t s_cap = 0, rows = 0;
    const int rc = ksa_cache_geometry(p, &s_cap, &rows);
    if (rc != KSA_OK) return rc;
    if (n_prefill < 0) return KSA_ERR_INVALID_ARG;
    if (n_prefill > p->n_text) return KSA_ERR_OUT_OF_RANGE;
    if (!k_cache || !v_cache || !aligned16(k_cache) || !aligned16(v_cache)) return KSA_ERR_INVALID_ARG;
    if (n_prefill == 0) return KSA_OK;   // nothing to hand over (k and v may be NULL then)
    if (!k || !v || !aligned16(k) || !aligned16(v)) return KSA_ERR_INVALID_ARG;
    KsaCacheFillLaunch a;
    const int64_t L = n_prefill / p->chunk_len * (int64_t)(p->chunk_len + p->n_summary) + n_prefill % p->chunk_len;
    if (kv_strides) {
        for (int x = 0; x < 3; ++x) a.kv_strides[x] = kv_strides[x];
    } else {   // contiguous [B, L, Hkv, d]: {batch, row, head}
        a.kv_strides[2] = p->head_dim;
        a.kv_strides[1] = (int64_t)p->n_kv_heads * p->head_dim;
        a.kv_strides[0] = L * a.kv_strides[1];
    }
    default_strides(a.cache_strides, cache_strides, p->n_kv_heads, rows, p->head_dim);
    if (!strides_ok(a.kv_strides) || !strides_ok(a.cache_strides)) return KSA_ERR_INVALID_ARG;
    a.k = k, a.v = v, a.k_cache = k_cache, a.v_cache = v_cache;
    a.n_prefill = n_prefill;
    a.summary_capacity = s_cap;
    a.p = *p;
    return ksa_launch_cache_fill(a, stream);
}

int ksa_cache_append(const ksa_params *p, int32_t kind, const void *k_new, const void *v_new, const int32_t *pos,
                     void *k_cache, void *v_cache, const int64_t cache_strides[3], void *stream) {
    int32_t s_cap = 0, rows = 0;
    const int rc = ksa_cache_geometry(p, &s_cap, &rows);
    if (rc != KSA_OK) return rc;
    if (kind != KSA_ROW_TEXT && kind != KSA_ROW_SUMMARY) return KSA_ERR_INVALID_ARG;
    if (kind == KSA_ROW_SUMMARY && p->n_summary == 0) return KSA_ERR_INVALID_ARG;
    if (!k_new || !v_new || !pos || !k_cache || !v_cache) return KSA_ERR_INVALID_ARG;
    if (!aligned16(k_new) || !aligned16(v_new) || !aligned16(k_cache) || !aligned16(v_cache)) return KSA_ERR_INVALID_ARG;
    KsaCacheAppendLaunch a;
    default_strides(a.cache_strides, cache_strides, p->n_kv_heads, rows, p->head_dim);
    if (!strides_ok(a.cache_strides)) return KSA_ERR_INVALID_ARG;
    a.k_new = k_new, a.v_new = v_new, a.pos = pos, a.k_cache = k_cache, a.v_cache = v_cache;
    a.kind = kind;
    a.summary_capacity = s_cap;
    a.p = *p;
    return ksa_launch_cache_append(a, stream);
}

const char *ksa_build_info(void) {
    static char info[320];
    // the compiler is part of the description: the kernels place MFMA wait states by hand in inline assembly, and
    // those were validated with this one
#ifdef __clang_version__
    const char *compiler = "clang " __clang_version__;
#else
    const char *compiler = "not hipcc (host-only test build)";
#endif
    std::snprintf(info, sizeof(info), "libksa gfx950 q_tile=%d k_tile=%d max_segments=%d compiler=%s", KSA_Q_TILE,
                  KSA_K_TILE, KSA_MAX_SEGMENTS, compiler);
    return info;
}

}  // extern "C"

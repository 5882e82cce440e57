// Prints what a decode call that leaves the number of spans to the library launches, for each line of standard input (entry: 0 text, 1
// summary, 2 text with the static workspace; workspace: 0 what the library asks for, 1 the least it accepts; batch, heads, KV heads,
// head_dim, tokens, chunk length, summaries, window chunks): status, spans per sequence (0: dealt by length), spans per KV head, whether
// the workgroups are large ones, and the bytes of the workspace.  Launches end here: nothing reaches a GPU.
#include <algorithm>
#include <cstdio>

#include "ksa.h"
#include "ksa_internal.h"

static KsaDecodeLaunch seen;
static float *const somewhere = reinterpret_cast<float *>(4096);   // (aligned, never read)

size_t ksa_prefill_workspace_size(const ksa_params &) { return 0; }
size_t ksa_prefill_bwd_workspace_size(const ksa_params &, int64_t) { return 0; }
int ksa_launch_prefill(const KsaPrefillLaunch &, void *) { return KSA_ERR_HIP; }
int ksa_launch_prefill_bwd(const KsaPrefillBwdLaunch &, void *) { return KSA_ERR_HIP; }
int ksa_launch_cache_fill(const KsaCacheFillLaunch &, void *) { return KSA_ERR_HIP; }
int ksa_launch_cache_append(const KsaCacheAppendLaunch &, void *) { return KSA_ERR_HIP; }
int ksa_launch_decode(const KsaDecodeLaunch &L, void *) {
    seen = L;
    return KSA_OK;
}
int ksa_decode_static_scratch(float **buf) {
    *buf = somewhere;
    return KSA_OK;
}
// as in ksa_decode.hip: what the least workspace holds records for
int ksa_decode_default_splits(const ksa_params *p) {
    const int64_t groups = (int64_t)p->batch * p->n_kv_heads;
    const int64_t rows = (int64_t)(p->n_text / p->chunk_len) * p->n_summary + (int64_t)(p->window_chunks + 1) * p->chunk_len;
    return (int)std::max<int64_t>(1, std::min<int64_t>({(1536 + groups - 1) / groups, std::max<int64_t>(1, rows / 768), 64}));
}

int main() {
    int entry, least, B, Hq, Hkv, d, n, c, m, C;
    while (std::scanf("%d %d %d %d %d %d %d %d %d %d", &entry, &least, &B, &Hq, &Hkv, &d, &n, &c, &m, &C) == 10) {
        ksa_params p{};
        p.batch = B, p.n_q_heads = Hq, p.n_kv_heads = Hkv, p.head_dim = d, p.n_text = n, p.chunk_len = c, p.n_summary = m, p.window_chunks = C;
        p.compress_ratio = m ? c / m : 0;
        seen = KsaDecodeLaunch{};
        const size_t bytes = ksa_decode_workspace_bytes(&p, least ? ksa_decode_default_splits(&p) : 0);
        float *x = somewhere;
        int rc;
        if (entry == 2)
            rc = ksa_decode_fwd_static(&p, x, x, x, (const int32_t *)x, x, nullptr, nullptr, 0, nullptr);
        else
            rc = (entry ? ksa_decode_summary_fwd : ksa_decode_fwd)(&p, x, x, x, (const int32_t *)x, x, nullptr, nullptr, x, bytes, 0, nullptr);
        std::printf("%d %d %d %d %zu\n", rc, seen.n_splits, seen.n_spans, (int)seen.wide, bytes);
    }
    return 0;
}

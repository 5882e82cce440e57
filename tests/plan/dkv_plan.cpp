// Prints the dK / dV plan of one layout per line of standard input (batch, heads, KV heads, head_dim, tokens, chunk length,
// summaries, window chunks, flags): kernel with split tiles, kernel without (1: 32-row query tiles, 0: 64-row blocks), number of
// pieces, of split tiles, of partial sums per (batch, KV head), and the steps of every tile as its pieces add them up.  Ends with
// status 1 if pieces of a tile overlap or leave steps out.
#include <cstdio>
#include <map>
#include <set>

#include "ksa_internal.h"

int main() {
    int B, Hq, Hkv, d, n, c, m, C, flags;
    while (std::scanf("%d %d %d %d %d %d %d %d %d", &B, &Hq, &Hkv, &d, &n, &c, &m, &C, &flags) == 9) {
        ksa_params p{};
        p.batch = B, p.n_q_heads = Hq, p.n_kv_heads = Hkv, p.head_dim = d, p.n_text = n, p.chunk_len = c, p.n_summary = m, p.window_chunks = C;
        p.compress_ratio = m ? c / m : 0, p.flags = flags;
        ksa_layout *lay = nullptr;
        if (ksa_build_layout(&p, &lay) != KSA_OK) return 1;
        std::map<int, std::map<int, int>> pieces;   // tile -> begin -> end
        std::set<int> slots;
        for (const KsaDkvEntry &e : lay->dkv_entries) {
            if (e.step_end <= e.step_begin || !pieces[e.tile].insert({e.step_begin, e.step_end}).second) return 1;
            if (e.slot >= 0 && !slots.insert(e.slot).second) return 1;
        }
        std::map<int, int> split;
        for (const KsaDkvSplit &s : lay->dkv_splits) split[s.tile] = s.n_slots;
        std::printf("%d %d %zu %zu %zu", (int)lay->dkv_direct, (int)lay->dkv_unsplit_direct, lay->dkv_entries.size(), lay->dkv_splits.size(), slots.size());
        for (const auto &t : pieces) {
            int at = 0;
            for (const auto &x : t.second) {
                if (x.first != at) return 1;
                at = x.second;
            }
            if ((split.count(t.first) ? split[t.first] : 1) != (int)t.second.size()) return 1;
            std::printf(" %d", at);
        }
        std::printf("\n");
        delete lay;
    }
}

// Host side of libksa: the integer work of Eq. 1 / Eq. 3 (index maps, per-row visible ranges), the
// block-sparse tile scheduler of section 2.3, and the geometry of the decode cache (section 2.3.1).
// No GPU call in this file.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <functional>
#include <new>
#include <numeric>
#include <queue>

#include "ksa_internal.h"

namespace {

inline int32_t pos_part(int64_t x) { return x > 0 ? (int32_t)x : 0; }

// Visible ranges of a text row (chunk j, text index i): summaries of chunks 0..j-C-1 and text of chunks
// max(0,j-C)..j up to i (Eq. 3).
inline void text_row_ranges(const ksa_params &p, int64_t i, int32_t out[4]) {
    const int64_t j = i / p.chunk_len;
    out[0] = 0;
    out[1] = pos_part(j - p.window_chunks) * p.n_summary;
    out[2] = pos_part(j - p.window_chunks) * p.chunk_len;
    out[3] = (int32_t)i + 1;
}

// Visible ranges of a summary row (ordinal u = j*m + slot): its chunk's text, itself, and (unless the
// self-only flag is set) the earlier summaries of its chunk.
inline void summary_row_ranges(const ksa_params &p, int64_t u, int32_t out[4]) {
    const int64_t j = u / p.n_summary;
    out[0] = (p.flags & KSA_FLAG_SUMMARY_SELF_ONLY) ? (int32_t)u : (int32_t)(j * p.n_summary);
    out[1] = (int32_t)u + 1;
    out[2] = (int32_t)(j * p.chunk_len);
    out[3] = (int32_t)((j + 1) * p.chunk_len);
}

inline int32_t tiles_in(const KsaSegment &s) { return (s.end - s.begin + KSA_K_TILE - 1) / KSA_K_TILE; }

// The run starts at the multiple of 16 at or below its first visible key, or of 64 if its tiles would otherwise end behind
// the next multiple of 64 of its index space (of n_space keys): the pipelined forward kernel reads V from a key-major copy
// whose keys are permuted in groups of 16 and which ends there.  The extra keys in front lie outside every row's visible
// range, so the first tile stays live and its mask clips them.
void push_segment(KsaWorkItem &it, int32_t space, int64_t begin, int64_t end, int64_t full_lo, int64_t full_hi, int64_t n_space) {
    if (end <= begin) return;
    auto tiles_end = [&](int64_t b) { return b + (end - b + KSA_K_TILE - 1) / KSA_K_TILE * KSA_K_TILE; };
    begin -= begin % 16;
    it.running_max |= tiles_end(begin) > n_space;
    if (tiles_end(begin) > (n_space + KSA_K_TILE - 1) / KSA_K_TILE * KSA_K_TILE) begin -= begin % KSA_K_TILE;
    KsaSegment &s = it.seg[it.n_seg++];
    s.space = space;
    s.begin = (int32_t)begin;
    s.end = (int32_t)end;
    s.full_lo = (int32_t)full_lo;
    s.full_hi = (int32_t)full_hi;
    s.pad = 0;
    it.n_tiles += tiles_in(s);
}

// Does tile t of the run need no mask?
inline bool tile_is_full(const KsaSegment &s, int32_t t) {
    const int64_t k0 = (int64_t)s.begin + (int64_t)t * KSA_K_TILE;
    return k0 >= s.full_lo && k0 + KSA_K_TILE <= s.full_hi;
}

// Query tile of text rows [t0, t0+cnt).
KsaWorkItem text_item(const ksa_params &p, int64_t t0, int32_t cnt) {
    KsaWorkItem it;
    std::memset(&it, 0, sizeof(it));
    it.q_space = KSA_SPACE_TEXT;
    it.q_begin = (int32_t)t0;
    it.q_count = cnt;
    const int64_t c = p.chunk_len, m = p.n_summary, C = p.window_chunks, n_sum = (int64_t)(p.n_text / p.chunk_len) * m;
    const int32_t j0 = (int32_t)t0 / p.chunk_len, j1 = (int32_t)(t0 + cnt - 1) / p.chunk_len;
    // distant summaries: the first row's chunk sees the fewest (those every row sees), the last row's chunk the most
    if (m > 0) push_segment(it, KSA_SPACE_SUMMARY, 0, pos_part(j1 - C) * m, 0, pos_part(j0 - C) * m, n_sum);
    // sliding-chunk text: [lo_first, ...) is seen by the first row's chunk, [lo_last, t0) by every row
    const int64_t lo_first = pos_part(j0 - C) * c, lo_last = pos_part(j1 - C) * c;
    push_segment(it, KSA_SPACE_TEXT, lo_first, t0 + cnt, lo_last, t0, p.n_text);
    return it;
}

// Query tile of summary rows [u0, u0+cnt): block-diagonal against their chunks' text and summaries.
KsaWorkItem summary_item(const ksa_params &p, int64_t u0, int32_t cnt) {
    KsaWorkItem it;
    std::memset(&it, 0, sizeof(it));
    it.q_space = KSA_SPACE_SUMMARY;
    it.q_begin = (int32_t)u0;
    it.q_count = cnt;
    const int64_t c = p.chunk_len, m = p.n_summary, n_sum = (int64_t)(p.n_text / p.chunk_len) * m;
    const int64_t j0 = (int32_t)u0 / p.n_summary, j1 = (int32_t)(u0 + cnt - 1) / p.n_summary;
    push_segment(it, KSA_SPACE_TEXT, j0 * c, (j1 + 1) * c, 0, 0, p.n_text);
    push_segment(it, KSA_SPACE_SUMMARY, j0 * m, u0 + cnt, 0, 0, n_sum);
    return it;
}

// Items in the order of their key tiles, most first, equal ones as they were.  (A counting sort: an item has at most four key
// tiles per item of the layout, and a few.)
void heaviest_first(std::vector<KsaWorkItem> &items) {
    int32_t most = 0;
    for (const KsaWorkItem &it : items) most = std::max(most, it.n_tiles);
    std::vector<int32_t> at(most + 2, 0);   // at[most - n]: where the next item of n tiles goes
    for (const KsaWorkItem &it : items) ++at[most - it.n_tiles + 1];
    for (int32_t x = 0; x < most; ++x) at[x + 1] += at[x];
    std::vector<int32_t> to(items.size());
    for (size_t x = 0; x < items.size(); ++x) to[x] = at[most - items[x].n_tiles]++;
    for (int32_t x = 0; x < (int32_t)items.size(); ++x)
        while (to[x] != x) {
            const int32_t y = to[x];
            std::swap(items[x], items[y]), std::swap(to[x], to[y]);
        }
}

// Which of the two forward kernels a layout takes: true = ksa_prefill_direct.hip.
//   - Chunk shapes that are no powers of two always (c 48, m 6, 16K tokens, 32/8 heads, d 128: 0.63 -> 0.36 ms; 6K tokens,
//     12/4 heads, d 64: 124 -> 54 us): the other kernel's pipelined loop maps rows with shifts.
//   - Otherwise by the mean number of key tiles per query tile.  Up to the line the pipelined kernel's time goes into what
//     its workgroups, alone on their compute unit, do outside the tile loop; beyond it the direct kernel's doubled operand
//     traffic costs more.  Measured on both sides (pipelined / direct kernel, us, c 64, m 8 unless stated; cards and runs
//     differ by 2 % in the comparison):
//       d 128, 4 heads of a group per workgroup: 4K tokens (7 tiles) 134 / 93, 16K (17) 398 / 356, 24K (24) 710 / 685, 28K
//         (28) 898 / 890, 30K (30) 1015 / 1015, 32K (31) 1112 / 1138, 34K (33) 1257 / 1280, 36K (35) 1378 / 1415; c 128, m 16
//         28K (29) 922 / 937, 32K (33) 1157 / 1189.  With outlier keys (1 % of the K rows eight times larger), where both keep
//         running maxima, 28K 1103 / 948, 32K 1404 / 1195, c 128, m 16, 32K 1448 / 1246.  On ordinary keys the two are level
//         at 30 tiles; the line lies at 34 because between the two the direct kernel loses 2 - 3 % on those and gains 14 % on
//         the others.  No summaries (the line is at 30): window 256 at 128K (5) 1347 / 1081, window 700 (12) 1982 / 1878, window
//         1024 (17) 320 / 307 at 16K, 622 / 613 at 32K, 2456 / 2450 at 128K, window 1500 (25) 430 / 406 at 16K, 3318 / 3290 at
//         128K, window 2048 (33) 497 / 515, causal 4K (33) 133 / 148;
//       2 heads: 32K (33) 635 / 611, 40K (41) 926 / 911, 48K (49) 1209 / 1227, 64K (62) 1999 / 2112; no summaries: window
//         1500 (25) 934 / 883, causal 4K (33) 107 / 97, window 2048 (33) 1099 / 1128, window 3000 (49) 1408 / 1483;
//       1 head, 16 heads: 16K (20) 271 / 195, 48K (52) 1382 / 1285, 64K (66) 2219 / 2206, 80K (82) 3305 / 3358; no
//         summaries: window 2048 (36) 1238 / 1214, window 3000 (51) 1576 / 1587, causal 8K (66) 247 / 270;
//       d 64: 16K 268 / 218, 64K (60) 2527 / 2527, 128K (117) 9165 / 9659, 256K (8/2 heads, 231) 8360 / 9137, window 4096
//         (65) 2280 / 2406.
bool takes_direct(const ksa_layout &lay) {
    const ksa_params &p = lay.p;
    auto pow2 = [](int64_t x) { return x > 0 && (x & (x - 1)) == 0; };
    if (!pow2(p.chunk_len) || (p.n_summary > 0 && !pow2(p.n_summary))) return true;
    int64_t tiles = 0;
    for (const KsaWorkItem &it : lay.items) tiles += it.n_tiles;
    const bool sums = p.n_summary > 0;
    const int64_t line = p.head_dim == 64 ? 60 : lay.head_stack == 4 ? (sums ? 34 : 30) : lay.head_stack == 2 ? (sums ? 44 : 34) : 56;
    return tiles <= line * (int64_t)lay.items.size();
}

// Does dQ take the kernel of ksa_prefill_direct.hip?  It does unless every key run is a long stretch of text: with two
// workgroups per compute unit the other kernel's fixed costs are hidden, and its extra operand reads only show on dense causal
// attention.  Whole backward pass, ksa_bwd_dq_kernel / direct, ms: 2 x 4096 tokens 0.449 / 0.336, 16K 1.476 / 1.269, 128K 58.3 /
// 57.0 (c 64, m 8, 32/8 heads, d 128), 20K in the paper's form, 16 heads, 1.646 / 1.401, window 1024 at 16K (17 tiles) 1.227 /
// 1.071, 64K d 64 9.19 / 8.81; causal 4K (33 tiles) 0.539 / 0.528, causal 8K (65) 1.846 / 1.875, causal 32K, 4 heads 3.53 / 3.63,
// causal 32K d 64 4.21 / 4.11.
bool dq_takes_direct(const ksa_layout &lay) {
    int64_t tiles = 0;
    for (const KsaWorkItem &it : lay.items) tiles += it.n_tiles;
    return lay.p.head_dim == 64 || lay.p.n_summary > 0 || tiles <= 48 * (int64_t)lay.items.size();
}

// Launch order.  Workgroups are dealt to the 8 XCDs round-robin by workgroup id, and each XCD has its
// own L2: queue q (workgroup ids congruent to q mod 8) is given whole (batch, KV head) groups so that the
// workgroups running together on one XCD stream the same K/V rows, and items go heaviest first so the
// long tiles start early (longest-processing-time order).  A whole number of rounds of 8.
void build_entries(ksa_layout &lay) {
    const ksa_params &p = lay.p;
    const int32_t n_items = (int32_t)lay.items.size();
    const int32_t n_groups = p.batch * p.n_kv_heads;
    const int32_t gsz = p.n_q_heads / p.n_kv_heads;
    // entry x of queue q is workgroup x * KSA_NUM_XCD + q
    auto fill = [&](int q, int32_t first_item, int32_t item_step, int32_t first_grp, int32_t grp_step) {
        size_t at = q;
        for (int32_t it = first_item; it < n_items; it += item_step)
            for (int32_t grp = first_grp; grp < n_groups; grp += grp_step) {
                const int32_t b = grp / p.n_kv_heads, head = (grp - b * p.n_kv_heads) * gsz;
                for (int32_t x = 0; x < gsz; x += lay.head_stack, at += KSA_NUM_XCD) lay.entries[at] = {it, b, head + x, 0};
            }
    };
    auto chunks = [](int64_t x, int64_t per) { return (x + per - 1) / per; };
    // (the first queue is the longest: it has the most groups, or the fewest to share its own with)
    const int64_t sharers0 = n_groups >= KSA_NUM_XCD ? 1 : chunks(KSA_NUM_XCD, n_groups), last = std::min(n_groups, KSA_NUM_XCD) - 1;
    const int64_t per_queue = n_groups >= KSA_NUM_XCD ? n_items * chunks(n_groups, KSA_NUM_XCD) : chunks(n_items, std::min(sharers0, chunks(KSA_NUM_XCD - last, n_groups)));
    lay.entries.resize((size_t)(per_queue * (gsz / lay.head_stack) * KSA_NUM_XCD), KsaWgEntry{-1, 0, 0, 0});
    for (int q = 0; q < KSA_NUM_XCD; ++q) {
        if (n_groups >= KSA_NUM_XCD) {
            fill(q, 0, 1, q, KSA_NUM_XCD);
        } else {
            // fewer groups than XCDs: the queues congruent to grp mod n_groups share the items of group grp
            const int32_t grp = q % n_groups;
            const int32_t sharers = (KSA_NUM_XCD - grp + n_groups - 1) / n_groups;  // queues serving grp
            fill(q, q / n_groups, sharers, grp, n_groups);
        }
    }
}

// The dK / dV key tiles of one (batch, KV head) for a kernel that walks query rows in aligned blocks, and a launch of them.
struct DkvTiles {
    const int64_t places, start;     // workgroups that the chip holds at once; what starting and ending one costs, in steps
    std::vector<int32_t> steps;      // per tile, the summary-space ones first: blocks times query heads per KV head
    struct Run {
        int64_t steps, count;
        bool operator<(const Run &x) const { return steps > x.steps; }   // longest first
    };
    std::vector<Run> runs;           // tiles of equal length
    int64_t total = 0, longest = 0, n_bh = 1, mean = 0;   // (mean: steps per place of the whole launch)
    DkvTiles(int64_t places_, int64_t start_) : places(places_), start(start_) {}

    static void merge(std::vector<Run> &x) {   // equal lengths in one
        std::sort(x.begin(), x.end());
        size_t n = 0;
        for (const Run &r : x) {
            if (n > 0 && x[n - 1].steps == r.steps) x[n - 1].count += r.count; else x[n++] = r;
        }
        x.resize(n);
    }
    void add(int64_t blocks, int64_t group) {
        const int64_t x = blocks * group;
        steps.push_back((int32_t)x), total += x;
        if (runs.empty() || runs.back().steps != x) runs.push_back({x, 0});
        ++runs.back().count;
    }
    void complete(int64_t n_bh_) {
        merge(runs);
        longest = runs.front().steps, n_bh = n_bh_, mean = total * n_bh / places;
    }
    static int64_t pieces(int64_t x, int64_t most) { return x > most ? ((uint32_t)x - 1) / (uint32_t)most + 1 : 1; }   // (32-bit divisions: this is what the search spends its time on)
    // A launch with pieces of at most so many steps: its workgroups and partial sums per (batch, KV head), its longest piece.
    struct Pieces { int64_t jobs, slots, longest; };
    Pieces cut(int64_t most, bool equal) const {
        Pieces x = {(int64_t)steps.size(), 0, 0};
        for (const Run &r : runs) {
            if (r.steps <= most) {
                x.longest = std::max(x.longest, r.steps);
                break;
            }
            const int64_t n = pieces(r.steps, most);
            x.jobs += (n - 1) * r.count, x.slots += n * r.count, x.longest = std::max(x.longest, equal ? ((uint32_t)r.steps - 1) / (uint32_t)n + 1 : most);
        }
        return x;
    }
    // When its last workgroup ends if they start in the order of their lengths, longest first; INT64_MAX if not before `limit`.
    int64_t makespan(const Pieces &cut, int64_t most, bool equal, int64_t limit) {
        // no launch ends before the mean place or the longest workgroup does, and none that starts one as soon as a place is
        // free after both
        const int64_t busy = ((total + start * cut.jobs) * n_bh + places - 1) / places, most_ = cut.longest + start;
        if (busy >= limit || most_ >= limit) return INT64_MAX;
        lengths.clear();
        size_t split = 0;
        for (; split < runs.size() && runs[split].steps > most; ++split) {
            const Run &r = runs[split];
            const int64_t n = pieces(r.steps, most), len = equal ? (uint32_t)r.steps / (uint32_t)n : r.steps - (n - 1) * most, rest = equal ? r.steps - len * n : n - 1;
            if (rest > 0) lengths.push_back({equal ? len + 1 : most, rest * r.count});   // the longer pieces
            if (n > rest) lengths.push_back({len, (n - rest) * r.count});
        }
        lengths.insert(lengths.end(), runs.begin() + split, runs.end());
        merge(lengths);
        // (in coarser time each of a place's workgroups may end a unit later)
        const int64_t unit = (busy + most_) / MAX_TIMES + 1, late = unit > 1 ? cut.jobs * n_bh / places + 1 : 0;
        const int64_t end_by = std::min((busy + most_) / unit + late, limit / unit) + 1;
        free_at.assign(end_by + 1, 0);   // how many places come free when (the workgroups of all (batch, KV head) pairs are alike)
        free_at[0] = (int32_t)places;
        int64_t t = 0, end = 0;
        for (const Run &r : lengths) {
            const int64_t len = std::max<int64_t>((r.steps + start + unit / 2) / unit, 1);
            for (int64_t left = r.count * n_bh; left > 0;) {
                while (free_at[t] == 0) ++t;
                const int64_t n = std::min<int64_t>(left, free_at[t]), at = t + len;
                if (at * unit >= limit || at > end_by) return INT64_MAX;
                free_at[t] -= (int32_t)n, free_at[at] += (int32_t)n, left -= n, end = at > end ? at : end;
            }
        }
        return end * unit;
    }
    // ... if no tile is split: the longest one, or as long as the mean place is busy
    int64_t unsplit() const { return std::max(longest + start, mean + start * (int64_t)steps.size() * n_bh / places); }

private:
    static constexpr int64_t MAX_TIMES = 1 << 22;   // longer launches (some millions of tokens) are played in coarser time
    std::vector<Run> lengths;
    std::vector<int32_t> free_at;
};

// Fills in the steps of both kernels' launches: per tile of keys [k0, k1) the blocks that overlap the two runs of query rows that
// can see one of them.  The kernels work the same runs out; the one with 64-row blocks counts all summary rows of the keys' chunks
// whatever the self-only flag says.
void dkv_steps(const ksa_params &p, DkvTiles &tiles, DkvTiles &wide) {
    const int64_t c = p.chunk_len, m = p.n_summary, C = p.window_chunks, n_sum = (int64_t)(p.n_text / c) * m, group = p.n_q_heads / p.n_kv_heads;
    const bool self_only = p.flags & KSA_FLAG_SUMMARY_SELF_ONLY;
    auto blocks = [](int64_t b, int64_t e, int shift) { return e > b ? ((e - 1) >> shift) - (b >> shift) + 1 : 0; };
    constexpr int SHIFT = 5, WIDE_SHIFT = 6;
    static_assert(KSA_DKV_ROWS == 1 << SHIFT && KSA_K_TILE == 1 << WIDE_SHIFT, "rows per block");
    for (const int space : {KSA_SPACE_SUMMARY, KSA_SPACE_TEXT}) {
        const int64_t n = space == KSA_SPACE_SUMMARY ? n_sum : p.n_text;
        const uint32_t per = (uint32_t)(space == KSA_SPACE_TEXT ? c : m);
        for (int64_t k0 = 0; k0 < n; k0 += KSA_DKV_KEYS) {
            const int64_t k1 = std::min<int64_t>(k0 + KSA_DKV_KEYS, n), jl = (uint32_t)k0 / per, jh = (uint32_t)(k1 - 1) / per;
            const int64_t b0 = space == KSA_SPACE_TEXT ? k0 : std::min<int64_t>((jl + C + 1) * c, p.n_text);
            const int64_t e0 = space == KSA_SPACE_TEXT ? std::min<int64_t>((jh + C + 1) * c, p.n_text) : p.n_text;
            const int64_t b1 = space == KSA_SPACE_TEXT ? jl * m : k0, e1 = std::min<int64_t>((jh + 1) * m, n_sum);
            tiles.add(blocks(b0, e0, SHIFT) + blocks(b1, space == KSA_SPACE_SUMMARY && self_only ? k1 : e1, SHIFT), group);
            wide.add(blocks(b0, e0, WIDE_SHIFT) + blocks(b1, e1, WIDE_SHIFT), group);
        }
    }
    tiles.complete((int64_t)p.batch * p.n_kv_heads), wide.complete((int64_t)p.batch * p.n_kv_heads);
}

// The backward pass's dK / dV work of one (batch, KV head).  A summary key is seen by every later text row, so the first
// tile of 128 of them is as long as hundreds of text tiles: a few workgroups would run long after the others have finished.
// Long tiles are therefore dealt to several workgroups, whose fp32 partial sums a second kernel adds up in a fixed order.  How
// long a piece may be is found by playing the launch through: workgroups start in the order of the list, longest first, on as
// many places as the chip has (two per compute unit, three at head_dim 64); a step costs 1, the start and the end of a
// workgroup DKV_STEPS_PER_START, the kernel that adds up its launch and 1/16 per partial sum.  Pieces are of equal length, or of
// the full length and what is left, which the greedy order packs better where a launch has few tiles.  Against the best
// of 13 piece lengths tried one by one (12 shapes, 1K to 64K tokens) the choice is within 3 %; pieces of the mean work per
// place, for comparison: 32K tokens 4.44 ms against 3.95, 64K 15.8 / 14.4, 2048 124 us / 87.  Equal pieces only: dense causal
// 16K 3.67 ms against 3.40.  (Whole backward pass, 32/8 heads, d 128.)
// All partial sums have to fit into the memory of dq (see ksa_launch_prefill_bwd), which holds batch * rows * query heads / 512
// of them.  Every layout pays for the search: half of the 0.25 ms that one of 131072 tokens in the paper's form, 8/1 heads takes
// (long tiles, twelve launches played through), a tenth of the 0.2 ms of the same with 32/8 heads, 4 of 7 us at 2 x 4096 tokens.
//
// The kernel that works on blocks of 64 rows (ksa_prefill_bwd.hip) takes the launches whose time is that of their longest
// workgroup: alone on its compute unit a workgroup takes 0.9 us per 32 rows there, 1.1 in ksa_prefill_bwd_dkv.hip (head_dim 64
// 0.6 / 0.75), which is ahead where its two or three workgroups per unit all have work.  Its pieces are of at least 32 steps and
// of the mean work per unit, longer while dq cannot hold them.  Both launches are played through and the 64-row kernel is taken
// where it ends first; likewise for launches in which no tile can be split (few tiles, or a dq that is strided or shares memory).
// Its step counts as 1.75 of the other's (head_dim 64: 1.6), the start of a workgroup as 7 of its steps (6); where c or m is no
// power of two its rows cost divisions (a fifth), and where c neither divides a tile of 32 rows nor is divided by it the other
// kernel works every tile's rows out anew, once for the heads of the group (0.4 of a step).  Dense causal text with no more tiles
// than places, none of them split, is the 64-row kernel's, too: its tiles' lengths run from one block to the whole text, and the
// long ones share their units with others for most of their time (4096 tokens, 16/16 heads 273 / 291).  Whole backward pass, us, 64-row /
// 32-row kernel: window 1024 over 2048 tokens, 16/4 heads, d 64 115 / 141, 8/1 heads, d 128 162 / 186; paper's form 2048 tokens
// 16/4 heads 211 / 226, dense causal 4096 tokens 358 / 379; 8192 tokens in chunks, gradients packed into one tensor, 32/8
// heads 1049 / 1168, d 64 703 / 856; but chunks of 64, 1000 tokens, 16/16 heads 84 / 70, 2 x 4096, 32/8 347 / 292, 20003 in the
// paper's form 1460 / 1318.  Those figures, and the ratios, are from before the 32-row kernel planned its requests in LDS, which takes
// a tenth off its steps: now 114 / 129, 160 / 175, 208 / 213, dense causal 344 / 345, packed 1022 / 1060, 686 / 780, 1000 tokens 79.5 / 62,
// 2 x 4096 322 / 254, 20003 1373 / 1184.  Over 180 layouts (200 - 16K tokens) the choice costs 1.5 % against the better kernel of
// each, all of it where the 64-row kernel is taken, 18 % at most (4/4 heads, d 64, 3 x 231 tokens, c 48, m 6, 29.1 / 24.6).
constexpr int64_t DKV_STEPS_PER_START = 8, DKV_STEPS_OF_SUMS = 12, DKV_MIN_STEPS = 16;
void build_dkv(ksa_layout &lay) {
    const ksa_params &p = lay.p;
    const bool d128 = p.head_dim == 128;
    DkvTiles tiles(d128 ? 512 : 768, DKV_STEPS_PER_START), wide(256, d128 ? 7 : 6);
    dkv_steps(p, tiles, wide);
    const int64_t n_bh = tiles.n_bh, capacity = (int64_t)p.batch * lay.aug_len * p.n_q_heads / 512 / n_bh;
    int64_t most = tiles.longest, best = INT64_MAX, end = INT64_MAX;
    bool equal = true;
    DkvTiles::Pieces chosen = {};
    auto consider = [&](int64_t most_, bool equal_) {   // the launch with pieces of at most so many steps
        const DkvTiles::Pieces cut = tiles.cut(most_, equal_);
        if (cut.slots > capacity) return;
        const int64_t sums = cut.slots > 0 ? DKV_STEPS_OF_SUMS + cut.slots * n_bh / 16 : 0, at = tiles.makespan(cut, most_, equal_, best - sums);
        if (at == INT64_MAX) return;
        best = at + sums, end = at, most = most_, equal = equal_, chosen = cut;
    };
    consider(tiles.longest, true);
    if (tiles.longest > tiles.mean / 8) {
        const int64_t shortest = std::max(DKV_MIN_STEPS, tiles.mean / 8);
        for (int64_t quarters = 2; quarters <= 6; ++quarters)
            if (tiles.mean * quarters / 4 >= DKV_MIN_STEPS && tiles.mean * quarters / 4 < tiles.longest) consider(tiles.mean * quarters / 4, false);
        // (no better than 2 % above the mean is worth looking for)
        for (int64_t quarters = 5; tiles.longest * 4 / quarters >= shortest && best * 50 > (tiles.mean + DKV_STEPS_PER_START) * 51; quarters += quarters / 4)
            consider(tiles.longest * 4 / quarters, true);
    }

    int64_t wide_most = std::max<int64_t>(32, wide.mean);
    DkvTiles::Pieces wide_cut = wide.cut(wide_most, true);
    while (wide_cut.slots > capacity) wide_cut = wide.cut(wide_most *= 2, true);   // (0 once no tile is longer)
    auto divides = [](int64_t x, int64_t y) { return x % y == 0 || y % x == 0; };
    const bool pow2 = (p.chunk_len & (p.chunk_len - 1)) == 0 && (p.n_summary & (p.n_summary - 1)) == 0;
    const double wide_step = (d128 ? 1.75 : 1.6) * (pow2 ? 1. : 1.2);
    const double step = 1. + (divides(p.chunk_len, KSA_DKV_ROWS) ? 0. : 0.4 * p.n_kv_heads / p.n_q_heads);
    const bool dense = p.n_summary == 0 && p.window_chunks >= (p.n_text - 1) / p.chunk_len && (int64_t)tiles.steps.size() * n_bh <= tiles.places;
    lay.dkv_unsplit_direct = !dense && wide.unsplit() * wide_step >= tiles.unsplit() * step;
    lay.dkv_direct = !(dense && chosen.slots == 0) &&
                     wide.makespan(wide_cut, wide_most, true, end) * wide_step >= end * step;   // (its steps are longer: no need to look behind `end` of them)
    if (!lay.dkv_direct) most = wide_most, equal = true, chosen = wide_cut;
    lay.dkv_entries.reserve(chosen.jobs);
    const std::vector<int32_t> &steps = (lay.dkv_direct ? tiles : wide).steps;
    for (size_t t = 0; t < steps.size(); ++t) {
        const int64_t pieces = DkvTiles::pieces(steps[t], most);
        if (pieces > 1) lay.dkv_splits.push_back({(int32_t)t, lay.dkv_slots, (int32_t)pieces, 0});
        int32_t at = 0;
        for (int64_t x = 1; x <= pieces; ++x) {   // equal pieces, or pieces of `most` steps and what is left
            const int32_t end = (int32_t)(equal ? steps[t] * x / pieces : std::min<int64_t>(x * most, steps[t]));
            lay.dkv_entries.push_back({(int32_t)t, at, end, pieces > 1 ? lay.dkv_slots++ : -1});
            at = end;
        }
    }
    std::stable_sort(lay.dkv_entries.begin(), lay.dkv_entries.end(), [](const KsaDkvEntry &a, const KsaDkvEntry &b) {
        return a.step_end - a.step_begin > b.step_end - b.step_begin;
    });
    if (lay.dkv_splits.empty()) lay.dkv_unsplit_direct = lay.dkv_direct;
}

}  // namespace

int ksa_validate_params(const ksa_params *p) {
    if (!p) return KSA_ERR_INVALID_ARG;
    if (p->batch <= 0 || p->n_text <= 0 || p->chunk_len <= 0 || p->n_summary < 0 || p->window_chunks < 0)
        return KSA_ERR_INVALID_ARG;
    if (p->n_q_heads <= 0 || p->n_kv_heads <= 0 || p->n_q_heads % p->n_kv_heads != 0) return KSA_ERR_INVALID_ARG;
    if (p->n_summary > 0 && (int64_t)p->compress_ratio * p->n_summary != p->chunk_len) return KSA_ERR_INVALID_ARG;
    if (p->flags & ~KSA_FLAG_SUMMARY_SELF_ONLY) return KSA_ERR_INVALID_ARG;
    if (!(p->softmax_scale == p->softmax_scale)) return KSA_ERR_INVALID_ARG;  // NaN
    // an incomplete last chunk has text positions only (its summaries do not exist yet)
    const int64_t L = (int64_t)(p->n_text / p->chunk_len) * (p->chunk_len + p->n_summary) + p->n_text % p->chunk_len;
    if (L >= (int64_t)1 << 30) return KSA_ERR_UNSUPPORTED;  // row indices are int32 on the device
    if (p->batch > 65535 || p->n_q_heads > 65535) return KSA_ERR_UNSUPPORTED;
    if (p->head_dim != 64 && p->head_dim != 128) return KSA_ERR_UNSUPPORTED;
    return KSA_OK;
}

extern "C" {

int ksa_build_layout(const ksa_params *params, ksa_layout **out) {
    if (!out) return KSA_ERR_INVALID_ARG;
    *out = nullptr;
    const int rc = ksa_validate_params(params);
    if (rc != KSA_OK) return rc;
    ksa_layout *lay = new (std::nothrow) ksa_layout();
    if (!lay) return KSA_ERR_OUT_OF_MEMORY;
    // the schedule grows std::vectors: no exception may leave through the C boundary
    try {
    lay->p = *params;
    if (lay->p.softmax_scale <= 0.f) lay->p.softmax_scale = 1.0f / std::sqrt((float)params->head_dim);
    if (lay->p.n_summary == 0) lay->p.compress_ratio = 0;
    const ksa_params &p = lay->p;
    lay->n_chunks = p.n_text / p.chunk_len;
    lay->aug_len = (int64_t)lay->n_chunks * (p.chunk_len + p.n_summary) + p.n_text % p.chunk_len;

    // query heads per workgroup: as many heads of one KV group as divide it, up to KSA_MAX_HEAD_STACK
    const int32_t gsz = p.n_q_heads / p.n_kv_heads;
    lay->head_stack = gsz % 4 == 0 ? 4 : gsz % 2 == 0 ? 2 : 1;
    static_assert(KSA_MAX_HEAD_STACK == 4, "head stacks are 1, 2 or 4");
    lay->q_tile_rows = KSA_Q_TILE / lay->head_stack;
    const int64_t qt = lay->q_tile_rows;
    lay->items.reserve((p.n_text + qt - 1) / qt + ((int64_t)lay->n_chunks * p.n_summary + qt - 1) / qt);
    for (int64_t t0 = 0; t0 < p.n_text; t0 += qt)
        lay->items.push_back(text_item(p, t0, (int32_t)std::min<int64_t>(qt, p.n_text - t0)));
    const int64_t n_sum = (int64_t)lay->n_chunks * p.n_summary;
    for (int64_t u0 = 0; u0 < n_sum; u0 += qt)
        lay->items.push_back(summary_item(p, u0, (int32_t)std::min<int64_t>(qt, n_sum - u0)));
    for (const KsaWorkItem &it : lay->items) {
        int32_t &from = it.q_space == KSA_SPACE_TEXT ? lay->running_text : lay->running_sum;
        if (it.running_max) from = std::min(from, it.q_begin);
        for (int32_t s = 0; s < it.n_seg; ++s) {
            const KsaSegment &g = it.seg[s];
            lay->ragged |= g.begin + (int64_t)tiles_in(g) * KSA_K_TILE > (g.space == KSA_SPACE_TEXT ? (int64_t)p.n_text : n_sum);
        }
    }
    heaviest_first(lay->items);
    lay->direct = takes_direct(*lay);
    lay->dq_direct = dq_takes_direct(*lay);
    build_entries(*lay);
    build_dkv(*lay);
    } catch (...) {
        delete lay;
        return KSA_ERR_OUT_OF_MEMORY;
    }
    *out = lay;
    return KSA_OK;
}

int ksa_augmented_rows(const ksa_params *p, int64_t n_text, int64_t *rows) {
    if (!p || !rows || n_text < 0 || p->chunk_len <= 0 || p->n_summary < 0) return KSA_ERR_INVALID_ARG;
    *rows = n_text / p->chunk_len * (int64_t)(p->chunk_len + p->n_summary) + n_text % p->chunk_len;
    return KSA_OK;
}

int ksa_layout_dims(const ksa_layout *lay, int64_t *aug_len, int32_t *n_chunks, int32_t *q_tile_rows,
                    int32_t *k_tile_rows, int32_t *heads_per_workgroup) {
    if (!lay) return KSA_ERR_INVALID_ARG;
    if (aug_len) *aug_len = lay->aug_len;
    if (n_chunks) *n_chunks = lay->n_chunks;
    if (q_tile_rows) *q_tile_rows = lay->q_tile_rows;
    if (k_tile_rows) *k_tile_rows = KSA_K_TILE;
    if (heads_per_workgroup) *heads_per_workgroup = lay->head_stack;
    return KSA_OK;
}

int ksa_layout_index_maps(const ksa_layout *lay, int32_t *aug_chunk, uint8_t *aug_is_summary,
                          int32_t *position_ids, int32_t *text_to_aug, int32_t *summary_to_aug) {
    if (!lay) return KSA_ERR_INVALID_ARG;
    const int64_t c = lay->p.chunk_len, m = lay->p.n_summary, w = c + m;
    for (int64_t a = 0; a < lay->aug_len; ++a) {
        const int64_t j = a / w, r = a % w;
        if (aug_chunk) aug_chunk[a] = (int32_t)j;
        if (aug_is_summary) aug_is_summary[a] = r >= c;
        // a summary token shares the position of its chunk's last text token (section 2.2.1)
        if (position_ids) position_ids[a] = (int32_t)(j * c + std::min<int64_t>(r, c - 1));
    }
    if (text_to_aug)
        for (int64_t i = 0; i < lay->p.n_text; ++i) text_to_aug[i] = (int32_t)(i / c * w + i % c);
    if (summary_to_aug)
        for (int64_t u = 0; u < (int64_t)lay->n_chunks * m; ++u) summary_to_aug[u] = (int32_t)(u / m * w + c + u % m);
    return KSA_OK;
}

int ksa_layout_row_ranges(const ksa_layout *lay, int64_t aq, int32_t out[4]) {
    if (!lay || !out) return KSA_ERR_INVALID_ARG;
    if (aq < 0 || aq >= lay->aug_len) return KSA_ERR_OUT_OF_RANGE;
    const int64_t c = lay->p.chunk_len, w = c + lay->p.n_summary;
    const int64_t j = aq / w, r = aq % w;
    if (r < c)
        text_row_ranges(lay->p, j * c + r, out);
    else
        summary_row_ranges(lay->p, j * lay->p.n_summary + (r - c), out);
    return KSA_OK;
}

int ksa_layout_mask_row(const ksa_layout *lay, int64_t aq, uint8_t *row_out) {
    if (!lay || !row_out) return KSA_ERR_INVALID_ARG;
    int32_t rg[4];
    const int rc = ksa_layout_row_ranges(lay, aq, rg);
    if (rc != KSA_OK) return rc;
    const int64_t c = lay->p.chunk_len, m = lay->p.n_summary, w = c + m;
    std::memset(row_out, 0, (size_t)lay->aug_len);
    for (int64_t u = rg[0]; u < rg[1]; ++u) row_out[u / m * w + c + u % m] = 1;
    for (int64_t i = rg[2]; i < rg[3]; ++i) row_out[i / c * w + i % c] = 1;
    return KSA_OK;
}

int ksa_layout_tile_pairs(const ksa_layout *lay, int64_t *n_pairs, uint8_t *q_space, int32_t *q_begin,
                          int32_t *q_count, uint8_t *k_space, int32_t *k_begin, int32_t *k_count, uint8_t *kind) {
    if (!lay || !n_pairs) return KSA_ERR_INVALID_ARG;
    int64_t x = 0;
    for (const KsaWorkItem &it : lay->items)
        for (int32_t s = 0; s < it.n_seg; ++s)
            for (int32_t kb = it.seg[s].begin; kb < it.seg[s].end; kb += KSA_K_TILE, ++x) {
                if (q_space) q_space[x] = (uint8_t)it.q_space;
                if (q_begin) q_begin[x] = it.q_begin;
                if (q_count) q_count[x] = it.q_count;
                if (k_space) k_space[x] = (uint8_t)it.seg[s].space;
                if (k_begin) k_begin[x] = kb;
                if (k_count) k_count[x] = std::min(KSA_K_TILE, it.seg[s].end - kb);
                if (kind) kind[x] = tile_is_full(it.seg[s], (kb - it.seg[s].begin) / KSA_K_TILE) ? KSA_TILE_FULL : KSA_TILE_MASKED;
            }
    *n_pairs = x;
    return KSA_OK;
}

int ksa_layout_launch_order(const ksa_layout *lay, int64_t *n_entries, uint8_t *q_space, int32_t *q_begin,
                            int32_t *batch, int32_t *q_head) {
    if (!lay || !n_entries) return KSA_ERR_INVALID_ARG;
    *n_entries = (int64_t)lay->entries.size();
    for (size_t x = 0; x < lay->entries.size(); ++x) {
        const KsaWgEntry &e = lay->entries[x];
        if (q_space) q_space[x] = e.item >= 0 ? (uint8_t)lay->items[e.item].q_space : 0;
        if (q_begin) q_begin[x] = e.item >= 0 ? lay->items[e.item].q_begin : -1;
        if (batch) batch[x] = e.batch;
        if (q_head) q_head[x] = e.q_head;
    }
    return KSA_OK;
}

// ---- decode cache geometry ---------------------------------------------------------------------

int ksa_cache_geometry(const ksa_params *p, int32_t *summary_capacity, int32_t *cache_rows) {
    const int rc = ksa_validate_params(p);
    if (rc != KSA_OK) return rc;
    const int64_t s_cap = (int64_t)(p->n_text / p->chunk_len) * p->n_summary;
    const int64_t rows = s_cap + (int64_t)(p->window_chunks + 1) * p->chunk_len;
    if (rows >= (int64_t)1 << 30) return KSA_ERR_UNSUPPORTED;
    if (summary_capacity) *summary_capacity = (int32_t)s_cap;
    if (cache_rows) *cache_rows = (int32_t)rows;
    return KSA_OK;
}

int ksa_cache_text_row(const ksa_params *p, int64_t i, int32_t *row) {
    int32_t s_cap;
    const int rc = ksa_cache_geometry(p, &s_cap, nullptr);
    if (rc != KSA_OK) return rc;
    if (!row) return KSA_ERR_INVALID_ARG;
    if (i < 0 || i >= p->n_text) return KSA_ERR_OUT_OF_RANGE;
    const int64_t j = i / p->chunk_len;
    *row = (int32_t)(s_cap + (j % (p->window_chunks + 1)) * p->chunk_len + i % p->chunk_len);
    return KSA_OK;
}

int ksa_cache_summary_row(const ksa_params *p, int64_t u, int32_t *row) {
    int32_t s_cap;
    const int rc = ksa_cache_geometry(p, &s_cap, nullptr);
    if (rc != KSA_OK) return rc;
    if (!row) return KSA_ERR_INVALID_ARG;
    if (u < 0 || u >= s_cap) return KSA_ERR_OUT_OF_RANGE;
    *row = (int32_t)u;
    return KSA_OK;
}

int ksa_decode_summary_ranges(const ksa_params *p, int64_t u, int32_t out[4]) {
    int32_t s_cap;
    const int rc = ksa_cache_geometry(p, &s_cap, nullptr);
    if (rc != KSA_OK) return rc;
    if (!out) return KSA_ERR_INVALID_ARG;
    if (p->n_summary == 0) return KSA_ERR_INVALID_ARG;
    if (u < 0 || u >= s_cap) return KSA_ERR_OUT_OF_RANGE;
    const int64_t c = p->chunk_len, C = p->window_chunks, m = p->n_summary;
    const int64_t j = u / m, slot = u % m;
    // summaries of the same chunk up to and including itself (Eq. 3, summary rows); only itself with flag bit 0
    const bool self_only = (p->flags & 1u) != 0;
    out[0] = (int32_t)(self_only ? u : j * m);
    out[1] = (int32_t)(self_only ? 1 : slot + 1);
    // the text of its own chunk: one whole ring slot
    out[2] = (int32_t)(s_cap + (j % (C + 1)) * c);
    out[3] = (int32_t)c;
    return KSA_OK;
}

int ksa_decode_ranges(const ksa_params *p, int64_t pos, int32_t out[6]) {
    int32_t s_cap;
    const int rc = ksa_cache_geometry(p, &s_cap, nullptr);
    if (rc != KSA_OK) return rc;
    if (!out) return KSA_ERR_INVALID_ARG;
    if (pos < 0 || pos >= p->n_text) return KSA_ERR_OUT_OF_RANGE;
    const int64_t c = p->chunk_len, C = p->window_chunks;
    const int64_t j = pos / c, r = pos % c;
    const int64_t slot = j % (C + 1);
    // summaries of chunks 0 .. j-C-1 (Eq. 3 left term): a prefix of the summary buffer
    out[0] = 0;
    out[1] = pos_part(j - C) * p->n_summary;
    // ring slots below the current chunk's slot are complete chunks; the current slot is filled up to r
    out[2] = s_cap;
    out[3] = (int32_t)(slot * c + r + 1);
    // slots above the current one hold older in-window chunks once the ring has wrapped (j >= C)
    out[4] = (int32_t)(s_cap + (slot + 1) * c);
    out[5] = j >= C ? (int32_t)((C - slot) * c) : 0;
    return KSA_OK;
}

const char *ksa_status_string(int status) {
    switch (status) {
        case KSA_OK: return "ok";
        case KSA_ERR_INVALID_ARG: return "invalid argument";
        case KSA_ERR_UNSUPPORTED: return "unsupported configuration";
        case KSA_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
        case KSA_ERR_HIP: return "HIP runtime error";
        case KSA_ERR_OUT_OF_RANGE: return "index out of range";
        case KSA_ERR_SCRATCH_LIMIT: return "problem exceeds the static scratch buffer";
        case KSA_ERR_OUT_OF_MEMORY: return "out of host memory";
        default: return "unknown status";
    }
}

}  // extern "C"

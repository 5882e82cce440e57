// KSA prefill for gfx950 with two workgroups per compute unit: the forward kernel for short key runs and for chunk shapes
// that are no powers of two, and the dQ kernel of the backward pass.
//
// The pipelined kernel (ksa_prefill.hip) owns a whole compute unit per workgroup (one wave per SIMD, 512 registers,
// 131 KB of LDS): at long key runs its hand-placed MFMA stream is the fastest, but nothing hides what a workgroup does
// outside that stream, and a 4K prefill spends most of its time there.  Here a workgroup is half as tall (32 query rows
// per wave), needs at most 256 registers per lane and 64 KB of LDS, so two of them share a compute unit (head_dim 64:
// three) and fill each other's start, barriers and end.  It reads K and V as they are: no key-major copy of V has to be
// written first.  What it costs: every operand read from LDS feeds one MFMA instead of two, and V^T comes from
// transposing reads.
// What bounds it: 4K tokens (2 x 4096, 32/8 heads, d 128: 190 MB, 47 GFLOP) take 89 us (before: 135) of which about 40 are
// the start and end of the workgroups (Q rows from HBM, stores; 1 tile per workgroup alone: 48 us) and 50 the tiles: the
// matrix unit is busy 39 % of the time that both waves of a SIMD are there.  At 17 and more tiles per workgroup it is 55 %, at
// 2.0 of 2.4 GHz under the board's power cap (1370 - 1385 of 1400 W), at 15 % more energy per product than the pipelined kernel
// (64K: 1.09 against 1.18 PFLOP/s).  Neither deeper prefetch (5 stages of 32 keys), three workgroups per compute unit, nor the
// scores of the next tile under the exponentials of this one changed the time by more than 3 %; the loads dealt between the
// MFMAs, the row offsets kept from tile to tile and the order of the query tiles did (together 10 - 30 %).  Of a workgroup's 20 us at
// 4K tokens 2.7 pass until its first tile is requested, 2.7 until that tile is there, 13.2 in the loop (6 tiles), 1.6 in its end;
// outside the tile loops a wave issued some 1550 of its 2620 vector instructions: row norms as dot products of pairs, the largest K norm
// by lane moves, output rows as offsets from one address and masks by constants where every row sees a tile's beginning take 2.8 % off
// (91.8 -> 89.2 us, window of 1024 at 16K 314.6 -> 311.2).  Workgroups that take several query tiles and request the next one's rows
// ahead were no faster (the other workgroup of the unit fills those times already).
// The line between the two kernels: takes_direct() in ksa_layout.cpp.  dQ (three products per visible pair instead of two)
// is ahead of ksa_bwd_dq_kernel nearly everywhere (dq_takes_direct()): 103 against 221 us at 2 x 4096 tokens.  It spills 2
// registers (d 64: 7), outside the blocks that hold its MFMAs.
//
// The work of a workgroup follows from its index in closed form (Eq. 3): no schedule is read from memory.  The keys of
// its query tile form one list (summaries, then text) cut into tiles of 64; a team's tiles sit in its two LDS buffers by
// turns, and its next one is requested behind the barrier that publishes the one before (with two teams: the one after the
// other team's).  Layout of scores, weights and operands: as in
// ksa_prefill.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "ksa_device.h"
#include "ksa_internal.h"

namespace {

constexpr int NW = 4;                   // waves per workgroup
constexpr int BN = KSA_K_TILE;          // keys per tile
constexpr int RW = BN / NW;             // rows of a key tile each wave fetches
constexpr int WG_PAIRS = NW * 32;       // (row, head) pairs per workgroup
// Where running maxima are kept, the reference is raised only for a jump above 2^2: the closer it is to the true maximum,
// the more often a row's largest weight is exactly 1 (no rounding).  Relative error of the outputs against fp64 at
// thresholds 0 / 2 / 8: 2.08e-3 / 2.12e-3 / 2.22e-3 (N(0, 1), c 48, m 6), 1.548e-3 / 1.551e-3 / 1.561e-3 (32K, 1 % outlier
// keys); time at 64K, c 48: 4.75 / 4.53 / 4.45 ms.
constexpr float RESCALE_THRESHOLD_LOG2 = 2.0f;

// Parts the K row norms of a (batch, KV head) are kept in.  Every wave of the forward kernel takes the maximum of them all,
// so there are few enough for four loads per lane that are in flight together; kept by 64-key tile
// they were 32 dependent round trips at 128K tokens (32/8 heads, d 128: window 256 1467 -> 1081 us, window 1024 2735 -> 2467;
// 16K tokens, c 64, m 8: 373 -> 356).
constexpr int NORM_PARTS = 256;

struct DirectArgs {
    const __bf16 *q, *k, *v;
    __bf16 *o;
    float *lse;
    int64_t qs[3], ks[3], os[3];        // {batch, row, head} strides in elements
    const float *knorm_parts;           // largest squared K row norm per part of a (batch, KV head)'s rows; NULL: keep running maxima
    float *knorm;                       // ... per (batch, KV head): stored by one workgroup of each
    int32_t own_norms;                  // every workgroup takes the norms of its head's rows itself, nothing is in knorm_parts
    int32_t running_text, running_sum;  // query tiles from these rows on keep running maxima whatever the norms say
    int32_t norm_parts;                 // parts per (batch, KV head), at most NORM_PARTS
    int32_t norm_text_parts;            // the first so many are text
    int32_t norm_run;                   // key tiles per part
    int32_t n_text, n_sum;
    int32_t c, m, C;
    uint32_t small_c, small_m;          // 65536 / c and 65536 / m, rounded up (used where c, m < 64)
    KsaDivisor by_c, by_m, by_bh, by_slices, by_kv_heads;
    int32_t n_q_heads, n_kv_heads, group;
    int32_t n_bh;                       // batch * n_kv_heads
    int32_t stack, stack_shift;         // query heads per workgroup (1, 2 or 4) and its log2
    int32_t slices;                     // workgroups per (batch, KV head, query tile): group / stack
    int32_t q_rows;                     // rows of a query tile: WG_PAIRS / stack
    int32_t text_tiles, sum_tiles;      // query tiles of the two spaces
    int32_t text_before;                // text tiles whose key lists are longer than a summary tile's
    int32_t self_only;
    int32_t longest_list;               // keys in the longest list of a query tile
    int32_t mixed_tiles;                // a key tile may hold the last summaries and the first text rows of a list
    int64_t aug_len;
    float scale_log2e;
    float static_shift;                 // 32 / scale_log2e
    // dQ only: o is dq, the others as in ksa_prefill_bwd.hip
    const __bf16 *g;                    // dLoss/dO
    int64_t gs[3];
    const float *stats;                 // row statistics (ksa_stat_at)
    int32_t nt_pad, ns_pad;
    float scale;
};

__device__ __forceinline__ float other_half(float x) {
    // value held by lane l^32
    const unsigned u = __builtin_bit_cast(unsigned, x);
    auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __builtin_bit_cast(float, (threadIdx.x & 32) ? r[0] : r[1]);
}

__device__ __forceinline__ float other_row(float x) {
    // value held by lane l^16
    const unsigned u = __builtin_bit_cast(unsigned, x);
    auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return __builtin_bit_cast(float, (threadIdx.x & 16) ? r[0] : r[1]);
}
template <int CTRL>
__device__ __forceinline__ float dpp_max(float x) {
    return fmaxf(x, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, false)));
}

#define KSA_FENCE() __builtin_amdgcn_sched_barrier(0)

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

template <int D>
struct Tile {
    static constexpr int CH = D / 8;           // 16-byte pieces per row
    static constexpr int RPI = 64 / CH;        // rows covered by one wavefront load instruction
    static constexpr int NI = RW / RPI;        // load instructions per wave, tile and tensor
    static_assert(RW % RPI == 0 && NI >= 1, "a wave's share of a tile is a whole number of load instructions");
    static constexpr int KS = D / 16;          // k steps of the score MFMA
    static constexpr int DB = D / 32;          // 32-column blocks of the output
    static constexpr int BYTES = BN * D * 2;   // one tensor's tile; a buffer holds K, then V
    static constexpr int STAGE_ROW = D * 2 + 16;
};

// squared norm of a row whose 16-byte pieces lie in CH neighbouring lanes, in all of them
template <int CH>
__device__ __forceinline__ float row_norm2(const bf16x8 &x) {
    float s2 = 0.f;
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        const bf16x2 y = {x[e], x[e + 1]};
        s2 = __builtin_amdgcn_fdot2_f32_bf16(y, y, s2, false);
    }
    return row_allreduce<CH>(s2);
}
// the largest value of a wave whose groups of CH lanes hold one each
template <int CH>
__device__ __forceinline__ float rows_max(float x) {
    if (CH == 8) x = dpp_max<0x140>(x);   // row_mirror
    x = fmaxf(x, other_row(x));
    return fmaxf(x, other_half(x));
}

// LDS tile: row-major [64][D] bf16, the 16-byte piece index XORed with a function of the row: for K all rows of a
// 16-lane phase of the plain read differ, for V the four rows of a transposing read do.  At head_dim 64 two rows share the 256
// bytes that all banks hold, so the rows of one parity have to differ (here and in the other kernels; with all rows treated
// alike, as before: 16K tokens, 32/8 heads 196.6 us, now 194.1, 64K 2457 / 2423).
template <int D>
__device__ __forceinline__ int k_swz(int row) { return D == 64 ? (row >> 1) & 7 : row & (D / 8 - 1); }
template <int D>
__device__ __forceinline__ int v_swz(int row) { return D == 64 ? (row & 2) << 1 : ((row & 3) << 2) & (D / 8 - 1); }

// augmented row (Eq. 1) of compact index idx
__device__ __forceinline__ int row_of(const DirectArgs &a, int space, int idx) {
    return space == KSA_SPACE_TEXT ? idx + ksa_div(idx, a.by_c) * a.m : idx + (ksa_div(idx, a.by_m) + 1) * a.c;
}

// visible key ranges (Eq. 3) of query idx: text [lo_t, hi_t), summaries [lo_s, hi_s)
struct Visible { int lo_t, hi_t, lo_s, hi_s; };
__device__ __forceinline__ Visible visible(const DirectArgs &a, int q_space, int idx) {
    Visible r;
    if (q_space == KSA_SPACE_TEXT) {
        const int j = ksa_div(idx, a.by_c);
        const int first = j - a.C > 0 ? j - a.C : 0;
        r.lo_s = 0, r.hi_s = first * a.m, r.lo_t = first * a.c, r.hi_t = idx + 1;
    } else {
        const int j = ksa_div(idx, a.by_m);
        r.lo_s = a.self_only ? idx : j * a.m, r.hi_s = idx + 1, r.lo_t = j * a.c, r.hi_t = (j + 1) * a.c;
    }
    return r;
}

// GRAD = false: forward.  GRAD = true: dQ of the backward pass (see ksa_prefill_bwd.hip for the products) on the same key
// lists: S^T = K Q^T and dP^T = V dO^T, whose accumulator starts from minus delta, dS^T = P^T o dP^T in bf16 as the B operand
// of dQ^T += K^T dS^T.
// TEAMS = 2: eight waves, of which the second four take every other key tile, in buffers of their own, and add what they have to
// the first four's at the end.
template <int D, bool GRAD, int TEAMS>
__device__ __forceinline__ void direct(const DirectArgs &a, unsigned char *const lds_all) {
    using T = Tile<D>;
    static_assert(NW * 32 * T::STAGE_ROW <= 4 * T::BYTES, "the epilogue's staging area reuses the tile buffers");
    static_assert(TEAMS == 1 || NW * (32 * T::STAGE_ROW + (T::DB * 4 + 1) * 1024) <= TEAMS * 4 * T::BYTES, "... and the second team's results lie behind it");
    auto k_swizzle = [](int row) { return GRAD ? ksa_swz<D>(row) : k_swz<D>(row); };
    auto v_swizzle = [](int row) { return GRAD ? ksa_swz<D>(row) : v_swz<D>(row); };

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) % NW, team = TEAMS == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6) / NW;
    unsigned char *const lds = lds_all + team * 4 * T::BYTES;
    const int r = lane & 31, h = lane >> 5;
    // Workgroup index -> (query tile, slice of the group's heads, batch and KV head), the latter fastest: workgroup ids go
    // to the XCDs round-robin, so with a multiple of 8 (batch, KV head) pairs all tiles of a head share one L2.  Longest
    // key lists first: text tiles from the last rows down (they see the most summaries), the summary tiles, whose lists are
    // all as long, behind the text tiles with longer ones.
    const int rest = ksa_div(blockIdx.x, a.by_bh), bh = blockIdx.x - rest * a.n_bh;
    const int tile = ksa_div(rest, a.by_slices), slice = rest - tile * a.slices;
    const int b = ksa_div(bh, a.by_kv_heads), hkv = bh - b * a.n_kv_heads;
    const int past = tile - a.text_before;   // >= 0: a summary tile, or a text tile behind those
    const int q_space = past < 0 || past >= a.sum_tiles ? KSA_SPACE_TEXT : KSA_SPACE_SUMMARY;
    const int n_q = q_space == KSA_SPACE_TEXT ? a.n_text : a.n_sum;
    const int q_begin = (q_space == KSA_SPACE_SUMMARY ? past : a.text_tiles - 1 - (past < 0 ? tile : tile - a.sum_tiles)) * a.q_rows;
    const int q_end = min(q_begin + a.q_rows, n_q);
    const int hq = hkv * a.group + slice * a.stack + (wave & (a.stack - 1));
    const int w_begin = q_begin + (wave >> a.stack_shift) * 32;   // the wave's 32 rows
    const bool w_any = w_begin < q_end;

    // ---- the keys: all those some row of the tile sees (Eq. 3; ranges are monotone in the row) ----------------------
    // One list, summaries first: position x < n_s is summary s_begin + x, position x >= t_first is text
    // t_begin + (x - t_first).  A key tile is 64 positions of the list.  With t_first = n_s at most one tile is partly
    // filled and one may hold both kinds; where the rows of such a tile may lie further apart than a 32-bit offset
    // reaches, t_first is the next multiple of 64 and the positions in between are masked.
    const Visible first_row = visible(a, q_space, q_begin), last_row = visible(a, q_space, q_end - 1);
    const int s_begin = first_row.lo_s, n_s = max(last_row.hi_s - s_begin, 0);
    const int t_first = a.mixed_tiles ? n_s : (n_s + BN - 1) / BN * BN;
    const int t_begin = first_row.lo_t, n_keys = t_first + last_row.hi_t - t_begin;   // (a row sees its own chunk's text)
    const int n_tiles = (n_keys + BN - 1) / BN;

    // ---- the lane's query row ----------------------------------------------------------------------------------
    const int idx = min(w_begin + r, q_end - 1);   // lanes past the end repeat the last row and store nothing
    const int q_aug = row_of(a, q_space, idx);
    bf16x8 qreg[T::KS];
    {
        const __bf16 *qp = a.q + b * a.qs[0] + (int64_t)q_aug * a.qs[1] + hq * a.qs[2] + h * 8;
#pragma unroll
        for (int s = 0; s < T::KS; ++s) qreg[s] = *reinterpret_cast<const bf16x8 *>(qp + s * 16);
    }
    bf16x8 greg[GRAD ? T::KS : 1];
    float lse2 = 0.f, minus_delta = 0.f;
    if constexpr (GRAD) {
        const __bf16 *gp = a.g + b * a.gs[0] + (int64_t)q_aug * a.gs[1] + hq * a.gs[2] + h * 8;
#pragma unroll
        for (int s = 0; s < T::KS; ++s) greg[s] = *reinterpret_cast<const bf16x8 *>(gp + s * 16);
        const int64_t stat = ((int64_t)b * a.n_q_heads + hq) * (a.nt_pad + a.ns_pad) + (q_space == KSA_SPACE_TEXT ? idx : a.nt_pad + idx);
        lse2 = a.stats[ksa_stat_at(stat)], minus_delta = a.stats[ksa_stat_at(stat) + KSA_STAT_ROWS];
    }

    // ---- the request of a tile, in two parts -------------------------------------------------------------------
    // prepare: where the tile's rows are (scalar bases of its first row, one 32-bit byte offset per lane and load
    // instruction); issue: one of the 2 NI global -> LDS loads of a wave.  The loads of the next tile are dealt between
    // the score MFMAs of the tile in work, one per k step: a wave that issues them in one go stands still for about 1000
    // clocks (the vector memory path of a compute unit takes 64 bytes per clock), a third of a step.
    const __bf16 *kbase = a.k + b * a.ks[0] + hkv * a.ks[2];
    const __bf16 *vbase = a.v + b * a.ks[0] + hkv * a.ks[2];
    const unsigned lds0 = (unsigned)(size_t)lds, row_bytes = (unsigned)a.ks[1] * 2u;
    const __bf16 *rq_k = kbase, *rq_v = vbase;
    unsigned k_off[T::NI], v_off[T::NI];
    int off_state = -1;   // what the offsets were worked out for: 2 * (position of the first row in its chunk) + kind
    int fast_left = 0;        // so many tiles follow whose rows lie fast_step elements behind the previous tile's
    int64_t fast_step = 0;
    auto prepare = [&](int t) {
        if (fast_left > 0) {
            --fast_left, rq_k += fast_step, rq_v += fast_step;
            return;
        }
        const int x0 = t * BN;
        unsigned row_off[T::NI];   // of the row alone
        bool renew = true;
        int64_t row0 = 0;
        int state = -1;
        if (t >= n_tiles) {
            // no such tile: the loads fetch 16 bytes of the KV head's first row, into a buffer nobody reads
#pragma unroll
            for (int i = 0; i < T::NI; ++i) row_off[i] = 0;
        } else if (x0 >= t_first || x0 + BN <= n_s) {
            const bool s = x0 < t_first;
            const int per = s ? a.m : a.c, other = s ? a.c : a.m;
            const int first = s ? s_begin + x0 : t_begin + (x0 - t_first);
            const int j0 = ksa_div(first, KsaDivisor{s ? a.by_m.mul : a.by_c.mul, s ? a.by_m.shift : a.by_c.shift}), phase = first - j0 * per;
            row0 = (int64_t)first + (s ? a.c : 0) + (int64_t)j0 * other;
            state = x0 + BN > n_keys ? -1 : 2 * phase + (s ? 1 : 0);
            renew = state != off_state || state < 0;
            const unsigned mul = per < 64 ? (s ? a.small_m : a.small_c) : 1024u;
            const int chunks = (BN * mul) >> 16;   // 64 / per
            if (chunks * per == BN) {
                fast_left = (((s ? n_s : n_keys) - x0) / BN - 1) / TEAMS;
                fast_step = (int64_t)(BN + chunks * other) * a.ks[1] * TEAMS;
            }
            if (renew) {
                // Row k of the tile is k + j (rows of the other kind per chunk) rows behind the first, j = how many chunk
                // borders lie between the two: small numbers, so that j is one 24-bit product (chunks of less than 64
                // rows: 65536 / chunk rounded up is exact for k + phase < 128; longer ones have at most one border).
                const unsigned add = (per < 64 ? phase : 64 - min(64, per - phase)) * mul;
                const unsigned other_bytes = (unsigned)other * row_bytes;
#pragma unroll
                for (int i = 0; i < T::NI; ++i) {
                    const int row = RW * wave + T::RPI * i + lane / T::CH;
                    const unsigned k = min(row, n_keys - 1 - x0);   // positions past the end of the list: its last row, masked
                    row_off[i] = k * row_bytes + ((__umul24(k, mul) + add) >> 16) * other_bytes;
                }
            }
        } else {
            // the end of the summaries and (mixed_tiles) the beginning of the text
            const int t_row0 = row_of(a, KSA_SPACE_TEXT, t_begin), s_row0 = row_of(a, KSA_SPACE_SUMMARY, s_begin + x0);
            const int first = a.mixed_tiles ? min(s_row0, t_row0) : s_row0;
            row0 = first;
#pragma unroll
            for (int i = 0; i < T::NI; ++i) {
                const int row = RW * wave + T::RPI * i + lane / T::CH;
                const int x = min(x0 + row, a.mixed_tiles ? n_keys - 1 : n_s - 1);
                const bool s = x < n_s;
                const int at = s ? s_begin + x : t_begin + (x - t_first);
                const int j = ksa_div(at, KsaDivisor{s ? a.by_m.mul : a.by_c.mul, s ? a.by_m.shift : a.by_c.shift});
                row_off[i] = (unsigned)(at + (s ? a.c : 0) + j * (s ? a.c : a.m) - first) * row_bytes;
            }
        }
        if (renew) {
#pragma unroll
            for (int i = 0; i < T::NI; ++i) {
                const int row = RW * wave + T::RPI * i + lane / T::CH, pch = lane % T::CH;
                const bool any = t < n_tiles;
                k_off[i] = row_off[i] + (any ? (pch ^ k_swizzle(row)) << 4 : 0);
                v_off[i] = row_off[i] + (any ? (pch ^ v_swizzle(row)) << 4 : 0);
            }
        }
        off_state = state;
        rq_k = kbase + row0 * a.ks[1], rq_v = vbase + row0 * a.ks[1];
    };
    auto issue = [&](int buf, int x) {   // load instruction x of the prepared tile: first K, then V
        const int i = x % T::NI;
        const unsigned dst = lds0 + buf * 2 * T::BYTES + (x / T::NI) * T::BYTES + (RW * wave + T::RPI * i) * (D * 2);
        if (x < T::NI)
            lds_direct_load_16_s(rq_k, k_off[i], dst);
        else
            lds_direct_load_16_s(rq_v, v_off[i], dst);
    };
    prepare(team);
#pragma unroll
    for (int x = 0; x < 2 * T::NI; ++x) issue(0, x);
    prepare(team + TEAMS);

    const Visible vis = visible(a, q_space, idx);
    // In list positions: the row sees [s_lo, s_hi) of the summaries and [t_lo, t_hi) of the text; some row of the wave
    // sees a position of [ws_lo, ws_hi) or [wt_lo, wt_hi), every row of it those of [fs_lo, fs_hi) and [ft_lo, ft_hi).
    const Visible w_first = visible(a, q_space, min(w_begin, q_end - 1)), w_last = visible(a, q_space, min(w_begin + 31, q_end - 1));
    const int t_off = t_first - t_begin;
    const int s_lo = vis.lo_s - s_begin, s_hi = vis.hi_s - s_begin, t_lo = vis.lo_t + t_off, t_hi = vis.hi_t + t_off;
    const int ws_lo = w_first.lo_s - s_begin, ws_hi = w_last.hi_s - s_begin, wt_lo = w_first.lo_t + t_off, wt_hi = w_last.hi_t + t_off;
    const int fs_lo = w_last.lo_s - s_begin, ft_hi = w_first.hi_t + t_off;
    int fs_hi = w_first.hi_s - s_begin, ft_lo = w_last.lo_t + t_off;
    if (fs_hi >= ft_lo) ft_lo = fs_lo, fs_hi = ft_hi;   // the two meet at the border: one range
    // ... and in tiles: those the wave sees something of, and those every row of it sees whole
    auto tiles = [](int lo, int hi) { return (unsigned)max(hi - lo, 0); };
    const int ws_t = ws_lo / BN, wt_t = wt_lo / BN, fs_t = (fs_lo + BN - 1) / BN, ft_t = (ft_lo + BN - 1) / BN;
    const unsigned ws_n = w_any && ws_hi > ws_lo ? tiles(ws_t, (ws_hi + BN - 1) / BN) : 0u;
    const unsigned wt_n = w_any && wt_hi > wt_lo ? tiles(wt_t, (wt_hi + BN - 1) / BN) : 0u;
    const unsigned fs_n = tiles(fs_t, fs_hi / BN), ft_n = tiles(ft_t, ft_hi / BN);

    // ---- the softmax reference: fixed where |q| max |k| rules out overflow and underflow (see ksa_prefill.hip) -----
    const float sl = a.scale_log2e;
    // The last query tiles of either space keep running maxima if their key runs reach past the end of the index space
    // (KsaWorkItem::running_max): short texts consist of such tiles, whose rows see few keys, and the rounding of a row's
    // largest weight shows there.  Relative error of the outputs against fp64, running / fixed (d 128): 37 tokens 1.76e-3 /
    // 1.93e-3, 500 tokens with c 8, m 1, C 32 2.00e-3 / 2.12e-3.  Their log-sum-exp still comes from unrounded weights.
    const bool running_max = q_begin >= (q_space == KSA_SPACE_TEXT ? a.running_text : a.running_sum);
    float m_static = 0.f;
    bool static_ok = false;
    if (!GRAD && a.knorm_parts) {
        float kmax2 = 0.f;
        if (a.own_norms) {
            constexpr int WAVES = NW * TEAMS, ROWS = WAVES * 64 / T::CH, AT_ONCE = 4;   // loads of a lane that travel together
            __shared__ float best_of[WAVES];
            const __bf16 *const src = kbase + tid % T::CH * 8;
            for (int64_t row0 = tid / T::CH; row0 < a.aug_len + tid / T::CH; row0 += AT_ONCE * ROWS) {
                bf16x8 x[AT_ONCE];
#pragma unroll
                for (int i = 0; i < AT_ONCE; ++i) x[i] = *reinterpret_cast<const bf16x8 *>(src + min(row0 + i * ROWS, a.aug_len - 1) * a.ks[1]);
#pragma unroll
                for (int i = 0; i < AT_ONCE; ++i) kmax2 = fmaxf(kmax2, row_norm2<T::CH>(x[i]));
            }
            kmax2 = rows_max<T::CH>(kmax2);
            if (lane == 0) best_of[tid >> 6] = kmax2;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < WAVES; ++i) kmax2 = fmaxf(kmax2, best_of[i]);
        } else {
            const float *src = a.knorm_parts + (int64_t)bh * a.norm_parts;
#pragma unroll
            for (int i = 0; i < NORM_PARTS; i += 64) kmax2 = fmaxf(kmax2, src[min(i + lane, a.norm_parts - 1)]);   // (the last one repeats)
            kmax2 = dpp_max<0xB1>(kmax2);    // quad_perm [1,0,3,2]
            kmax2 = dpp_max<0x4E>(kmax2);    // quad_perm [2,3,0,1]
            kmax2 = dpp_max<0x141>(kmax2);   // row_half_mirror
            kmax2 = rows_max<8>(kmax2);
        }
        if (rest == 0 && tid == 0) a.knorm[bh] = kmax2;
        float n2 = 0.f;
#pragma unroll
        for (int s = 0; s < T::KS; ++s)
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                const bf16x2 x = {qreg[s][e], qreg[s][e + 1]};
                n2 = __builtin_amdgcn_fdot2_f32_bf16(x, x, n2, false);
            }
        n2 += other_half(n2);
        const float bound = __builtin_amdgcn_sqrtf(n2 * kmax2) * 1.002f;   // (the factor covers the rounding of all this)
        m_static = bound - a.static_shift;
        static_ok = !running_max && __builtin_amdgcn_ballot_w64(!(bound * sl <= 60.f)) == 0;
    }

    // byte addresses inside a buffer, relative to its start: see ksa_prefill.hip
    const int grp = lane >> 4, li = lane & 15;
    const int t_row = 4 * (grp >> 1) + (li >> 2), t_col = 16 * (grp & 1) + 4 * (li & 3);
    const int ll_k = r * (D * 2) + ((k_swizzle(r) ^ h) << 4);                                                   // rows
    const int ll_t = t_row * (D * 2) + (((t_col >> 3) ^ v_swizzle(t_row)) << 4) + ((t_col & 7) << 1);           // columns
    const int ll_v = T::BYTES + ll_t;

    // dQ: one key tile, 32 keys at a time (the registers of two blocks of S and dP would not fit)
    auto grad_tile = [&](int t, int buf, const unsigned char *tile_lds, f32x16 (&oacc)[T::DB]) {
        const int x0 = t * BN;
        const bool masked = (unsigned)(t - fs_t) >= fs_n && (unsigned)(t - ft_t) >= ft_n;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            f32x16 sacc, gacc;
#pragma unroll
            for (int g = 0; g < 16; ++g) sacc[g] = 0.f, gacc[g] = minus_delta;
            constexpr int AHEAD = 2;   // operands are read AHEAD k steps before the MFMAs that use them
            bf16x8 ka[T::KS], va[T::KS];
            auto read_rows = [&](int s) {
                const unsigned char *at = tile_lds + ((ll_k ^ (s << 5)) + kb * 32 * (D * 2));
                ka[s] = *reinterpret_cast<const bf16x8 *>(at), va[s] = *reinterpret_cast<const bf16x8 *>(at + T::BYTES);
            };
#pragma unroll
            for (int s = 0; s < AHEAD; ++s) read_rows(s);
#pragma unroll
            for (int s = 0; s < T::KS; ++s) {
                if (s + AHEAD < T::KS) read_rows(s + AHEAD);
                KSA_FENCE();
                sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[s], qreg[s], sacc, 0, 0, 0);
                gacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[s], greg[GRAD ? s : 0], gacc, 0, 0, 0);
                if (kb == 0) issue(buf ^ 1, s);
                KSA_FENCE();
            }
            if (kb == 0) prepare(t + 2 * TEAMS);
            if (masked) {   // as in the forward tile
                const int y0 = x0 + kb * 32, base_t = y0 + 4 * h - t_lo, base_s = y0 + 4 * h - s_lo;
                const unsigned span_t = (unsigned)max(t_hi - t_lo, 0), span_s = (unsigned)max(s_hi - s_lo, 0);
                if (y0 >= t_first || y0 + 32 <= n_s) {
                    const bool txt = y0 >= t_first;
                    if (y0 >= (txt ? ft_lo : fs_lo)) {
                        const int end = (txt ? t_hi : s_hi) - y0 - 4 * h;
#pragma unroll
                        for (int g = 0; g < 16; ++g) sacc[g] = 8 * (g / 4) + g % 4 < end ? sacc[g] : -INFINITY;
                    } else {
                        const int base = txt ? base_t : base_s;
                        const unsigned span = txt ? span_t : span_s;
#pragma unroll
                        for (int g = 0; g < 16; ++g) sacc[g] = (unsigned)(base + 8 * (g / 4) + g % 4) < span ? sacc[g] : -INFINITY;
                    }
                } else {
#pragma unroll
                    for (int g = 0; g < 16; ++g) {
                        const int o = 8 * (g / 4) + g % 4;
                        sacc[g] = ((unsigned)(base_t + o) < span_t || (unsigned)(base_s + o) < span_s) ? sacc[g] : -INFINITY;
                    }
                }
            }
            bf16x8 ds[2];
#pragma unroll
            for (int g = 0; g < 16; ++g) ds[g / 8][g % 8] = (__bf16)(__builtin_amdgcn_exp2f(fmaf(sacc[g], sl, -lse2)) * gacc[g]);
#pragma unroll
            for (int hf = 0; hf < 2; ++hf)
#pragma unroll
                for (int db = 0; db < T::DB; ++db) {
                    // rows R0 + t_row and R0 + 8 + t_row, R0 = 32 kb + 16 hf: the latter's swizzle differs by XOR 2
                    const unsigned char *at = tile_lds + (kb * 32 + hf * 16) * (D * 2);
                    const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s16x4))(at + (ll_t ^ (db << 6))));
                    const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s16x4))(at + ((ll_t ^ (((db * 4) ^ 2) << 4)) + 8 * (D * 2))));
                    const bf16x8 kt = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
                    oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kt, ds[hf], oacc[db], 0, 0, 0);
                }
        }
    };

    auto body = [&](auto track_tag, auto exact_tag) {
        constexpr bool TRACK = decltype(track_tag)::value, EXACT = decltype(exact_tag)::value;   // EXACT: l_exact is kept
        f32x16 oacc[T::DB];
        f32x4 l_sum = {0.f, 0.f, 0.f, 0.f};   // row sums: lane j < 16, register 0 (query j) and 1 (query j + 16)
        // l_sum comes from products in which the weights of row j + 16 are multiplied by zero, so one that is no number (a NaN
        // or an infinity in the query or in a key it sees) would reach row j.  With running maxima such a row is taken out
        // (m_ref = infinity, weights 0) and its result set to NaN at the end: 1 % of the time, a sum per lane takes 3 %.
        // Fixed reference: the lane's part of the row sum of the weights before rounding, for the log-sum-exp, and for the row
        // itself where l_sum is not a number and this sum is.  (A running maximum makes a row's largest weight 1, or close to
        // it; against a fixed reference it is any number, and a row of one or two keys would hand the backward pass a
        // log-sum-exp that is off by up to 2^-9.  3 % of the time.)
        float l_exact = 0.f;
        float m_ref = TRACK ? -1e30f : m_static;
#pragma unroll
        for (int db = 0; db < T::DB; ++db)
#pragma unroll
            for (int g = 0; g < 16; ++g) oacc[db][g] = 0.f;
        const unsigned ind1 = (lane == 0 || lane == 32 || lane == 17 || lane == 49) ? 0x3f803f80u : 0u;
        const bf16x8 ind = __builtin_bit_cast(bf16x8, u32x4{ind1, ind1, ind1, ind1});

        for (int round = 0; round * TEAMS < n_tiles; ++round) {
            const int t = round * TEAMS + team, buf = round & 1;   // (a t behind the last tile: nothing for this wave)
            __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wave's pieces of tile t have landed
            __syncthreads();                      // ... and everybody's; nobody reads the other buffer any more
            const int x0 = t * BN, x1 = x0 + BN;
            if ((unsigned)(t - ws_t) >= ws_n && (unsigned)(t - wt_t) >= wt_n) {   // nothing for this wave
#pragma unroll
                for (int x = 0; x < 2 * T::NI; ++x) issue(buf ^ 1, x);
                prepare(t + 2 * TEAMS);
                continue;
            }
            const unsigned char *tile_lds = lds + buf * 2 * T::BYTES;
            if constexpr (GRAD) {
                grad_tile(t, buf, tile_lds, oacc);
                continue;
            }

            f32x16 sacc[2];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int g = 0; g < 16; ++g) sacc[kb][g] = 0.f;
            // K operands are read AHEAD k steps before the MFMAs that use them
            constexpr int AHEAD = 3;
            bf16x8 ka[T::KS][2];
            auto read_k = [&](int s) {
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) ka[s][kb] = *reinterpret_cast<const bf16x8 *>(tile_lds + ((ll_k ^ (s << 5)) + kb * 32 * (D * 2)));
            };
#pragma unroll
            for (int s = 0; s < AHEAD; ++s) read_k(s);
#pragma unroll
            for (int s = 0; s < T::KS; ++s) {
                if (s + AHEAD < T::KS) read_k(s + AHEAD);
                KSA_FENCE();
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) sacc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[s][kb], qreg[s], sacc[kb], 0, 0, 0);
                static_assert(2 * T::NI == T::KS, "one load per k step");
                issue(buf ^ 1, s);
                KSA_FENCE();
            }
            prepare(t + 2 * TEAMS);
            __builtin_amdgcn_s_setprio(0);
            if ((unsigned)(t - fs_t) >= fs_n && (unsigned)(t - ft_t) >= ft_n) {
                // clip to what the row sees: score register g of block kb is position x0 + 32 kb + 4 h + 8 (g / 4) + g % 4
                const int base_t = x0 + 4 * h - t_lo, base_s = x0 + 4 * h - s_lo;
                const unsigned span_t = (unsigned)max(t_hi - t_lo, 0), span_s = (unsigned)max(s_hi - s_lo, 0);
                if (x0 >= t_first || x1 <= n_s) {   // one kind of key
                    const bool txt = x0 >= t_first;
                    if (x0 >= (txt ? ft_lo : fs_lo)) {   // ... whose first one every row sees: a compare with a constant each
                        const int end = (txt ? t_hi : s_hi) - x0 - 4 * h;
#pragma unroll
                        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                            for (int g = 0; g < 16; ++g) sacc[kb][g] = kb * 32 + 8 * (g / 4) + g % 4 < end ? sacc[kb][g] : -INFINITY;
                    } else {
                        const int base = txt ? base_t : base_s;
                        const unsigned span = txt ? span_t : span_s;
#pragma unroll
                        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                            for (int g = 0; g < 16; ++g)
                                sacc[kb][g] = (unsigned)(base + kb * 32 + 8 * (g / 4) + g % 4) < span ? sacc[kb][g] : -INFINITY;
                    }
                } else {
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                        for (int g = 0; g < 16; ++g) {
                            const int o = kb * 32 + 8 * (g / 4) + g % 4;
                            sacc[kb][g] = ((unsigned)(base_t + o) < span_t || (unsigned)(base_s + o) < span_s) ? sacc[kb][g] : -INFINITY;
                        }
                }
            }
            if constexpr (TRACK) {
                float mx = sacc[0][0];
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int g = 0; g < 16; ++g) mx = __builtin_elementwise_maximum(mx, sacc[kb][g]);   // NaN if one of them is
                mx = __builtin_elementwise_maximum(mx, other_half(mx));
                if (__builtin_amdgcn_ballot_w64(!((mx - m_ref) * sl <= RESCALE_THRESHOLD_LOG2)) != 0) {
                    const bool lost = !(mx < INFINITY);
                    if (__builtin_amdgcn_ballot_w64(lost) != 0) {
#pragma unroll
                        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                            for (int g = 0; g < 16; ++g) sacc[kb][g] = lost ? -INFINITY : sacc[kb][g];
                    }
                    const float m_new = lost ? INFINITY : fmaxf(m_ref, mx);
                    // (old - new) first: equal references (also the -1e30 start value) must give exactly 2^0
                    const float alpha = __builtin_amdgcn_exp2f((m_ref - m_new) * sl);
                    m_ref = m_new;
                    const float alpha_lo = __shfl(alpha, lane & 15), alpha_hi = __shfl(alpha, (lane & 15) + 16);
                    l_sum[0] *= alpha_lo, l_sum[1] *= alpha_hi;
                    if constexpr (EXACT) l_exact *= alpha;
#pragma unroll
                    for (int db = 0; db < T::DB; ++db)
#pragma unroll
                        for (int g = 0; g < 16; ++g) oacc[db][g] *= alpha;
                }
            }
            __builtin_amdgcn_s_setprio(1);   // the other workgroup's wave on this SIMD yields: measured 1 %
            // weights, rounded to bf16, in the B-operand layout of P V; row sums of the rounded weights (see sum_half())
            const float msl = m_ref * sl;
            bf16x8 pb[2][2];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int hf = 0; hf < 2; ++hf) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float w = __builtin_amdgcn_exp2f(fmaf(sacc[kb][8 * hf + e], sl, -msl));
                        if constexpr (EXACT) l_exact += w;
                        pb[kb][hf][e] = (__bf16)w;
                    }
                    l_sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ind, pb[kb][hf], l_sum, 0, 0, 0);
                }
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int hf = 0; hf < 2; ++hf)
#pragma unroll
                    for (int db = 0; db < T::DB; ++db) {
                        const int a_db = ll_v ^ (db << 6);
                        const int o0 = (kb * 32 + hf * 16) * (D * 2), o1 = o0 + 8 * (D * 2);
                        const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s16x4))(tile_lds + a_db + o0));
                        const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s16x4))(tile_lds + a_db + o1));
                        const bf16x8 va = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
                        oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb[kb][hf], oacc[db], 0, 0, 0);
                    }
        }

        // ---- O = O^T / l through a per-wave staging area in the tile buffers, whole rows stored; LSE ---------------
        __builtin_amdgcn_s_waitcnt(0x0F70);   // the loads behind the last tile have landed
        __syncthreads();                      // everybody is done with the tiles
        if constexpr (TEAMS == 2) {   // a wave of the second team holds the same rows as the one of the first, in the same lanes
            f32x4 *const given = reinterpret_cast<f32x4 *>(lds_all + NW * 32 * T::STAGE_ROW) + wave * ((T::DB * 4 + 1) * 64) + lane;
            if (team == 1 && w_any) {
#pragma unroll
                for (int x = 0; x < T::DB * 4; ++x)
                    given[x * 64] = f32x4{oacc[x / 4][x % 4 * 4], oacc[x / 4][x % 4 * 4 + 1], oacc[x / 4][x % 4 * 4 + 2], oacc[x / 4][x % 4 * 4 + 3]};
                if constexpr (!GRAD) given[T::DB * 4 * 64] = f32x4{l_sum[0], l_sum[1], l_exact, m_ref};
            }
            __syncthreads();
            if (team == 1) return;
            if (w_any) {
                float mine = 1.f, theirs = 1.f;   // what the two parts are multiplied by: with running maxima their references differ
                f32x4 more = {0.f, 0.f, 0.f, 0.f};
                if constexpr (!GRAD) more = given[T::DB * 4 * 64];
                if constexpr (TRACK) {
                    const float m_new = fmaxf(m_ref, more[3]);   // (equal references, also two infinite ones, must give exactly 1)
                    mine = m_ref == m_new ? 1.f : __builtin_amdgcn_exp2f((m_ref - m_new) * sl);
                    theirs = more[3] == m_new ? 1.f : __builtin_amdgcn_exp2f((more[3] - m_new) * sl);
                    m_ref = m_new;
                }
#pragma unroll
                for (int x = 0; x < T::DB * 4; ++x) {
                    const f32x4 o = given[x * 64];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float &acc = reinterpret_cast<float (&)[16]>(oacc[x / 4])[x % 4 * 4 + e];
                        acc = TRACK ? fmaf(o[e], theirs, acc * mine) : acc + o[e];
                    }
                }
                if constexpr (TRACK) {
#pragma unroll
                    for (int e = 0; e < 2; ++e) l_sum[e] = fmaf(more[e], __shfl(theirs, (lane & 15) + 16 * e), l_sum[e] * __shfl(mine, (lane & 15) + 16 * e));
                } else {
                    l_sum[0] += more[0], l_sum[1] += more[1];
                }
                l_exact = l_exact * mine + more[2] * theirs;
            }
        }
        if (!w_any) return;
        unsigned char *stg = lds_all + wave * (32 * T::STAGE_ROW);
        const float s0 = __shfl(l_sum[0], r & 15), s1 = __shfl(l_sum[1], r & 15);
        float l_row = (r & 16) ? s1 : s0;
        l_exact += other_half(l_exact);
        if constexpr (TRACK) {
            l_row = m_ref < INFINITY ? l_row : __builtin_nanf("");
            l_exact = EXACT && m_ref < INFINITY ? l_exact : l_row;
        } else {
            l_row = l_row == l_row ? l_row : l_exact;
        }
        const float inv = GRAD ? a.scale : 1.0f / l_row;
#pragma unroll
        for (int db = 0; db < T::DB; ++db)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                bf16x4 pk;
#pragma unroll
                for (int e = 0; e < 4; ++e) pk[e] = (__bf16)(oacc[db][g4 * 4 + e] * inv);
                *reinterpret_cast<bf16x4 *>(stg + r * T::STAGE_ROW + (db * 32 + g4 * 8 + h * 4) * 2) = pk;
            }
        const int piece = lane % T::CH;
        // Row k of the wave lies k + (chunk borders in between) * other rows behind its first: see prepare.
        const bool txt = q_space == KSA_SPACE_TEXT;
        const int per = txt ? a.c : a.m, other = txt ? a.m : a.c;
        const int j0 = ksa_div(w_begin, KsaDivisor{txt ? a.by_c.mul : a.by_m.mul, txt ? a.by_c.shift : a.by_m.shift}), phase = w_begin - j0 * per;
        const unsigned mul = per < 64 ? (txt ? a.small_c : a.small_m) : 1024u, add = (per < 64 ? phase : 64 - min(64, per - phase)) * mul;
        __bf16 *const obase = a.o + b * a.os[0] + ((int64_t)w_begin + (txt ? 0 : a.c) + (int64_t)j0 * other) * a.os[1] + hq * a.os[2] + piece * 8;
        u32x4 x[32 / T::RPI];
#pragma unroll
        for (int i = 0; i < 32 / T::RPI; ++i) x[i] = *reinterpret_cast<const u32x4 *>(stg + (T::RPI * i + lane / T::CH) * T::STAGE_ROW + piece * 16);
        auto store = [&](int i) {
            const int row = T::RPI * i + lane / T::CH;
            const unsigned d_rows = row + ((__umul24(row, mul) + add) >> 16) * (unsigned)other;   // (less than 2^30)
            *reinterpret_cast<u32x4 *>(obase + (uint64_t)d_rows * (uint64_t)a.os[1]) = x[i];
        };
        if (w_begin + 32 <= q_end) {
#pragma unroll
            for (int i = 0; i < 32 / T::RPI; ++i) store(i);
        } else {
#pragma unroll
            for (int i = 0; i < 32 / T::RPI; ++i)
                if (w_begin + T::RPI * i + lane / T::CH < q_end) store(i);
        }
        if constexpr (GRAD) return;
        if (a.lse && h == 0 && w_begin + r < q_end) {
            float msl = m_ref * sl;
            asm volatile("" : "+v"(msl));   // (not contracted with the sum below; split as in ksa_prefill.hip)
            const float t = msl + (float)__builtin_amdgcn_frexp_expf(l_exact);
            a.lse[((int64_t)b * a.n_q_heads + hq) * a.aug_len + q_aug] =
                fmaf(t, 0.6931471805599453f, __logf(__builtin_amdgcn_frexp_mantf(l_exact)));
        }
    };
    // the copies meet at the same barriers, so the choice is per wave
    if (GRAD || static_ok)
        body(std::false_type{}, std::true_type{});
    else if constexpr (!GRAD) {
        if (running_max && a.knorm_parts)
            body(std::true_type{}, std::true_type{});
        else
            body(std::true_type{}, std::false_type{});
    }
}

// Two workgroups per compute unit for head_dim 128 (64 KB of LDS, 256 registers each), three for head_dim 64 (16K tokens,
// 32/8 heads: 219 us; two: 235, four, with shorter operand read-ahead: 250).
template <int D>
__global__ __launch_bounds__(NW * 64, D == 128 ? 2 : 3) void ksa_prefill_direct_kernel(const DirectArgs a) {
    __shared__ __attribute__((aligned(1024))) unsigned char lds[4 * Tile<D>::BYTES];
    direct<D, false, 1>(a, lds);
}
template <int D>
__global__ __launch_bounds__(NW * 64, D == 128 ? 2 : 3) void ksa_bwd_dq_direct_kernel(const DirectArgs a) {
    __shared__ __attribute__((aligned(1024))) unsigned char lds[4 * Tile<D>::BYTES];
    direct<D, true, 1>(a, lds);
}
// ... and with eight waves in a workgroup (ksa_two_teams() in ksa_internal.h)
template <int D>
__global__ __launch_bounds__(2 * NW * 64, 2) void ksa_prefill_teams_kernel(const DirectArgs a) {
    __shared__ __attribute__((aligned(1024))) unsigned char lds[2 * 4 * Tile<D>::BYTES];
    direct<D, false, 2>(a, lds);
}
template <int D>
__global__ __launch_bounds__(2 * NW * 64, 2) void ksa_bwd_dq_teams_kernel(const DirectArgs a) {
    __shared__ __attribute__((aligned(1024))) unsigned char lds[2 * 4 * Tile<D>::BYTES];
    direct<D, true, 2>(a, lds);
}

// Largest squared K row norm of norm_run 64-key tiles of a (batch, KV head), the parts of the text space first.
// Bound by latency or HBM reads; squares as dot products of pairs and sums by lane moves (through LDS 2 x 4096 tokens 5.4 us, now 4.9;
// 20003 tokens, 16 heads, 92 MB 16.7, now 15.1; 512 tokens, whole prefill 12.25, now 11.87).
template <int D>
__global__ __launch_bounds__(256) void ksa_knorm_parts_kernel(const DirectArgs a, float *out) {
    constexpr int CH = D / 8, ROWS = 256 / CH;
    __shared__ float wave_best[4];
    const int b = blockIdx.z, hkv = blockIdx.y, tid = threadIdx.x, part = blockIdx.x;
    const int space = part < a.norm_text_parts ? KSA_SPACE_TEXT : KSA_SPACE_SUMMARY;
    const int k0 = (space == KSA_SPACE_TEXT ? part : part - a.norm_text_parts) * a.norm_run * BN;
    const int n_space = space == KSA_SPACE_TEXT ? a.n_text : a.n_sum;
    const int n_tiles = min(a.norm_run, (n_space - k0 + BN - 1) / BN);
    const __bf16 *kb = a.k + b * a.ks[0] + hkv * a.ks[2] + (tid % CH) * 8;
    float best = 0.f;
    for (int t = 0; t < n_tiles; ++t) {
#pragma unroll
        for (int i = 0; i < BN / ROWS; ++i) {
            const int key = min(k0 + BN * t + ROWS * i + tid / CH, n_space - 1);
            const bf16x8 x = *reinterpret_cast<const bf16x8 *>(kb + (int64_t)row_of(a, space, key) * a.ks[1]);
            best = fmaxf(best, row_norm2<CH>(x));
        }
    }
    best = rows_max<CH>(best);
    if ((tid & 63) == 0) wave_best[tid >> 6] = best;
    __syncthreads();
    if (tid == 0)
        out[((int64_t)b * a.n_kv_heads + hkv) * gridDim.x + part] = fmaxf(fmaxf(wave_best[0], wave_best[1]), fmaxf(wave_best[2], wave_best[3]));
}

bool two_teams(const DirectArgs &a, int head_dim, int64_t n_wg, bool grad) { return ksa_two_teams(head_dim, n_wg, a.stack, a.longest_list, grad); }

// Short texts: a launch of its own for the K norms takes 3 - 4 us, a workgroup reads all rows of its head in less.  us, norms before / by
// every workgroup: head_dim 64 (eight waves) 200 tokens 10.7 / 8.8, 512 11.1 / 10.0, 1500 rows 11.1 / 10.7, 3375 12.9 / 15.2; head_dim 128, eight
// waves 787 rows 19.3 / 18.7, 1152 25.7 / 26.0, four waves 216 rows 14.6 / 13.1, 576 15.3 / 15.5; head_dim 64, four waves (lists of one key tile)
// 900 rows 8.2 / 7.2, 1280 8.2 / 8.0.
bool takes_own_norms(const DirectArgs &a, int head_dim, int64_t n_wg) {
    return n_wg <= 256 && a.aug_len * head_dim <= (two_teams(a, head_dim, n_wg, false) ? 100 : head_dim == 64 ? 80 : 56) * 1024;
}

template <int D>
void launch(const DirectArgs &a, float *parts, int batch, int64_t n_wg, hipStream_t st) {
    if (a.knorm_parts && !a.own_norms) hipLaunchKernelGGL(ksa_knorm_parts_kernel<D>, dim3(a.norm_parts, a.n_kv_heads, batch), dim3(256), 0, st, a, parts);
    if (two_teams(a, D, n_wg, false))
        hipLaunchKernelGGL(ksa_prefill_teams_kernel<D>, dim3((unsigned)n_wg), dim3(2 * NW * 64), 0, st, a);
    else
        hipLaunchKernelGGL(ksa_prefill_direct_kernel<D>, dim3((unsigned)n_wg), dim3(NW * 64), 0, st, a);
}

// the parts of the arguments that describe the key lists (the strides are set); returns the number of workgroups
int64_t fill_lists(DirectArgs &a, const ksa_params &p, int32_t head_stack, int64_t aug_len) {
    a.n_text = p.n_text;
    a.n_sum = (p.n_text / p.chunk_len) * p.n_summary;
    a.c = p.chunk_len, a.m = p.n_summary, a.C = p.window_chunks;
    a.small_c = (65535 + a.c) / a.c, a.small_m = a.m > 0 ? (65535 + a.m) / a.m : 0;
    a.by_c = ksa_divisor(a.c), a.by_m = ksa_divisor(a.m > 0 ? a.m : 1);
    a.n_q_heads = p.n_q_heads, a.n_kv_heads = p.n_kv_heads;
    a.group = p.n_q_heads / p.n_kv_heads;
    a.n_bh = p.batch * p.n_kv_heads;
    a.by_bh = ksa_divisor(a.n_bh), a.by_kv_heads = ksa_divisor(a.n_kv_heads);
    a.stack = head_stack;
    a.stack_shift = log2_exact(head_stack);
    a.slices = a.group / head_stack;
    a.by_slices = ksa_divisor(a.slices);
    // Rows per query tile: 32 per wave.  A launch with fewer workgroups than compute units takes shorter tiles, down to the
    // rows of one wave (the other waves then only fetch): their key lists are shorter, and there are units to spare (512
    // tokens, 1 head, d 64: the 64 summary rows see 576 keys together, 288 by halves: 16.7 -> 13.4 us; 700 tokens in the
    // paper's form, 16 heads: 26.0 -> 20.5).
    a.q_rows = WG_PAIRS / head_stack;
    auto tiles_of = [&](int32_t rows) { return (rows + a.q_rows - 1) / a.q_rows; };
    while (a.q_rows > 32 && 2 * ((int64_t)tiles_of(a.n_text) + tiles_of(a.n_sum)) * a.slices * a.n_bh <= 256) a.q_rows /= 2;
    a.text_tiles = tiles_of(a.n_text);
    a.sum_tiles = tiles_of(a.n_sum);
    {   // a text tile's list has (chunks before the window) m summaries and at most (C + 1) c + q_rows text rows
        const int64_t sum_keys = a.m > 0 ? (int64_t)((a.q_rows + a.m - 1) / a.m) * a.c + a.q_rows : 0;
        auto longer = [&](int64_t tile) {
            const int64_t row = tile * a.q_rows, j = row / a.c;
            return (j > a.C ? (j - a.C) * a.m + (int64_t)(a.C + 1) * a.c : row) + a.q_rows > sum_keys;
        };
        int32_t lo = 0, hi = a.text_tiles;   // (lists do not get shorter from one text tile to the next)
        while (lo < hi) {
            const int32_t mid = lo + (hi - lo) / 2;
            if (longer(mid)) hi = mid; else lo = mid + 1;
        }
        a.text_before = a.text_tiles - lo;
        a.longest_list = (int32_t)ksa_longest_list(a.c, a.m, a.C, a.n_text, a.n_sum, a.q_rows);
    }
    a.self_only = (p.flags & KSA_FLAG_SUMMARY_SELF_ONLY) ? 1 : 0;
    a.mixed_tiles = ksa_mixed_tile_rows(a.c, a.m, a.q_rows) * a.ks[1] * 2 < ((int64_t)1 << 32) ? 1 : 0;   // 32-bit byte offsets
    a.aug_len = aug_len;
    return ((int64_t)a.text_tiles + a.sum_tiles) * a.slices * a.n_bh;
}

}  // namespace

int ksa_launch_prefill_direct(const KsaPrefillLaunch &L, float *knorm_parts, float *knorm, void *stream) {
    DirectArgs a;
    a.q = static_cast<const __bf16 *>(L.q);
    a.k = static_cast<const __bf16 *>(L.k);
    a.v = static_cast<const __bf16 *>(L.v);
    a.o = static_cast<__bf16 *>(L.o);
    a.lse = L.lse;
    for (int x = 0; x < 3; ++x) a.qs[x] = L.q_strides[x], a.ks[x] = L.kv_strides[x], a.os[x] = L.o_strides[x];
    // Chunk shapes that are no powers of two keep running maxima: with a fixed reference the largest weight of a row is no
    // longer 1 but any number, rounded to bf16 like the others, and the outputs' error against fp64 would rise (2.15e-3 to
    // 2.26e-3 relative); the other shapes have had the fixed reference all along.
    const bool fixed = log2_exact(L.p.chunk_len) >= 0 && (L.p.n_summary == 0 || log2_exact(L.p.n_summary) >= 0);
    a.knorm_parts = fixed ? knorm_parts : nullptr;
    a.running_text = L.running_text, a.running_sum = L.running_sum;
    a.knorm = knorm;
    a.scale_log2e = L.p.softmax_scale * 1.4426950408889634f;
    a.static_shift = 32.f / a.scale_log2e;
    const int64_t n_wg = fill_lists(a, L.p, L.head_stack, L.aug_len);
    if (n_wg >= (int64_t)1 << 30) return KSA_ERR_UNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int text_tiles = (a.n_text + BN - 1) / BN, sum_tiles = (a.n_sum + BN - 1) / BN;
    a.norm_run = std::max(1, (text_tiles + sum_tiles + NORM_PARTS - 3) / (NORM_PARTS - 2));   // (each space may add a short part)
    a.norm_text_parts = (text_tiles + a.norm_run - 1) / a.norm_run;
    a.norm_parts = a.norm_text_parts + (sum_tiles + a.norm_run - 1) / a.norm_run;
    a.own_norms = takes_own_norms(a, L.p.head_dim, n_wg);
    if (L.p.head_dim == 128)
        launch<128>(a, knorm_parts, L.p.batch, n_wg, st);
    else if (L.p.head_dim == 64)
        launch<64>(a, knorm_parts, L.p.batch, n_wg, st);
    else
        return KSA_ERR_UNSUPPORTED;
    return hipGetLastError() == hipSuccess ? KSA_OK : KSA_ERR_HIP;
}

int ksa_launch_dq_direct(const KsaPrefillBwdLaunch &L, const float *stats, void *stream) {
    DirectArgs a;
    a.q = static_cast<const __bf16 *>(L.q);
    a.k = static_cast<const __bf16 *>(L.k);
    a.v = static_cast<const __bf16 *>(L.v);
    a.g = static_cast<const __bf16 *>(L.d_o);
    a.o = static_cast<__bf16 *>(L.dq);
    a.lse = nullptr, a.knorm_parts = nullptr, a.knorm = nullptr, a.own_norms = 0, a.running_text = a.running_sum = a.norm_parts = a.norm_text_parts = a.norm_run = 0;
    for (int x = 0; x < 3; ++x) a.qs[x] = L.q_strides[x], a.ks[x] = L.kv_strides[x], a.gs[x] = L.o_strides[x], a.os[x] = L.dq_strides[x];
    a.stats = stats;
    const int64_t n_wg = fill_lists(a, L.p, L.head_stack, L.aug_len);
    if (n_wg >= (int64_t)1 << 30) return KSA_ERR_UNSUPPORTED;
    a.nt_pad = (a.n_text + 63) / 64 * 64, a.ns_pad = (a.n_sum + 63) / 64 * 64;
    a.scale = L.p.softmax_scale, a.scale_log2e = L.p.softmax_scale * 1.4426950408889634f;
    const bool two = two_teams(a, L.p.head_dim, n_wg, true);
    const dim3 grid((unsigned)n_wg), block(NW * 64 * (two ? 2 : 1));
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (L.p.head_dim == 128 && two)
        hipLaunchKernelGGL(ksa_bwd_dq_teams_kernel<128>, grid, block, 0, st, a);
    else if (L.p.head_dim == 128)
        hipLaunchKernelGGL(ksa_bwd_dq_direct_kernel<128>, grid, block, 0, st, a);
    else if (two)
        hipLaunchKernelGGL(ksa_bwd_dq_teams_kernel<64>, grid, block, 0, st, a);
    else
        hipLaunchKernelGGL(ksa_bwd_dq_direct_kernel<64>, grid, block, 0, st, a);
    return KSA_OK;
}

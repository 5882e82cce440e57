// KSA prefill backward for gfx950: dK and dV with two workgroups per compute unit (head_dim 64: three).
//
// Products as in ksa_prefill_bwd.hip: S = Q K^T and dP = G V^T (G = dLoss/dO), whose accumulator starts from minus delta,
// P = exp2(S scale log2(e) - lse2), dS = P o dP, dV^T += G^T P, dK^T += Q^T dS, with the wave's 32 keys and both gradients in
// registers and the query tiles (32 rows of one head: Q, G and two statistics per row) streamed through LDS.
//
// A workgroup takes KSA_DKV_KEYS = 128 keys of an index space, 32 per wave, and walks the query tiles that see them: the
// aligned 32-row blocks of the text rows, then of the summary rows, each from the last block down (the key tiles of a head
// then meet the same query tiles at about the same time), the query heads of the group innermost.  An entry of the
// schedule may be a piece of that sequence (KsaDkvEntry).
//
// Why this split: a workgroup that owns its compute unit (512 registers per lane, blocks of 64 rows: ksa_bwd_dkv_kernel) has
// one wave per SIMD, which issues everything itself: matrix unit busy 52 % at 128K tokens, and at 2 x 4096 tokens 40 % of the
// scores it works out lie outside the mask.  With 256 registers two waves share a SIMD and issue beside each other's matrix
// instructions, and a 32 x 32 block that none of a wave's keys is seen by is skipped.  Both accumulators are 128 registers,
// V 32, scores and dP of one block 32: of K's 32 the first operands come from LDS (K_LDS), read back lane by lane.  What the
// loop needs only now and then (the keys' visibility, the parameters of another chunk row) is worked out again from opaque
// copies of the lane number and of the argument pointer: kept in registers it pushed operands out to scratch, which costs
// 15 % (a reload waits for the tiles in flight).
// Where the tiles lie is worked out for 64 steps at a time, one per lane, and kept in LDS.  Taken from the step before, as it was,
// it was 100 scalar instructions with branches, 500 - 700 clocks per step, and 54 scalars that did not fit the scalar registers
// (now 9 and 160 clocks): 20003 tokens in the paper's form 1623 -> 1596 us (forward and backward; the kernel's clocks fall by 11 %,
// the power cap takes most of it back), 2 x 4096 345.8 -> 341.8, 6011 tokens, c 48, m 6, d 64, where a block's place was worked
// out from the start 158.4 -> 148.7, window 1024, d 64, 2 x 1536 158.0 -> 150.4.
// What bounds it: 128K tokens (32/8 heads, d 128, 35.6 TFLOP executed) the board's power cap, 32.5 ms, before 35.2; 2 x 4096
// tokens 131 us, before 205: chains of 90 and more steps of 0.9 - 1.2 us per workgroup; 20003 tokens in the paper's form 690 us,
// before 830.  Per step of 32 MFMAs (1024 clocks) a wave alone on its SIMD takes about 2300 clocks: the four phases 1700, the
// barrier 100, the first operands' way from LDS 250, the next request 160.
// A workgroup alone on its unit is slower than one of ksa_bwd_dkv_kernel, which takes the launches that wait for one: build_dkv in
// ksa_layout.cpp.
// Tried and dropped: query tiles of 64 rows (the offsets of twice as many loads spill); four stages in flight instead of three
// (equal); S and dP interleaved (the chain of eight dependent MFMAs costs nothing: 32 clocks each); operands read one, two or
// four MFMAs ahead (1 - 2 %); a look at every tile's log-sum-exp for values that are no numbers (2 %; now at clipped tiles only).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "ksa_device.h"
#include "ksa_internal.h"

namespace {

constexpr int NW = 4;              // waves per workgroup, 32 keys each
constexpr int BM = 32;             // query rows per tile
constexpr int STAGES = 3;          // tiles in LDS: the one in work and two that are on their way
static_assert(NW * 32 == KSA_DKV_KEYS, "the schedule counts key tiles of this size");
static_assert(BM == KSA_DKV_ROWS, "... and query tiles of this size");
static_assert(BM == KSA_STAT_ROWS, "a tile's statistics are one 64-lane load");
constexpr int RW = BM / NW;        // rows of a tile each wave fetches
constexpr int PLAN = 64;           // steps per part of the request plan: one per lane of the wave that works it out

// what the visibility of a key depends on
struct KeyView {
    int32_t n_text, n_sum, c, m, C, self_only;
    KsaDivisor by_c, by_m;
};

struct DkvArgs {
    const __bf16 *q, *k, *v, *g;
    const float *stats;            // row statistics (ksa_stat_at)
    __bf16 *dk, *dv;
    float *scratch;                // partial sums of split tiles; NULL: no tile is split
    const KsaDkvEntry *entries;
    int64_t qs[3], ks[3], gs[3], dks[3];   // {batch, row, head} strides in elements
    KeyView view;
    int32_t n_q_heads, n_kv_heads, group, n_bh, sum_tiles, nt_pad, ns_pad;
    uint32_t small_c, small_m;     // 65536 / c and 65536 / m, rounded up (used where c, m < 64)
    KsaDivisor by_bh, by_kv_heads, by_group;
    float scale, scale_log2e;
};

#define KSA_FENCE() __builtin_amdgcn_sched_barrier(0)

// 4 bytes per lane from a wave-uniform base (see lds_direct_load_16_s)
__device__ __forceinline__ void lds_direct_load_4_s(const float *sbase, unsigned voff_bytes, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" : : "v"(voff_bytes), "s"(sbase), "s"(lds_addr) : "memory");
}

// Query rows [lo, hi) of index space q_space that see key `key` of index space `space` (Eq. 3 read from the key's side).  A
// row's visible ranges never move backwards from one row to the next, so these are consecutive rows, and lo and hi do
// not decrease from one key to the next.
struct Seen { int lo, hi; };
__device__ __forceinline__ Seen seen_by(const KeyView &a, int space, int key, int q_space) {
    if (space == KSA_SPACE_TEXT) {
        const int j = ksa_div(key, a.by_c);
        if (q_space == KSA_SPACE_TEXT) return {key, (int)min(((int64_t)j + a.C + 1) * a.c, (int64_t)a.n_text)};
        return {min(j * a.m, a.n_sum), min((j + 1) * a.m, a.n_sum)};
    }
    const int j = ksa_div(key, a.by_m);
    if (q_space == KSA_SPACE_TEXT) return {(int)min(((int64_t)j + a.C + 1) * a.c, (int64_t)a.n_text), a.n_text};
    return {key, a.self_only ? key + 1 : min((j + 1) * a.m, a.n_sum)};
}

template <int D>
__global__ __launch_bounds__(NW * 64, D == 128 ? 2 : 3) void ksa_bwd_dkv_direct_kernel(const DkvArgs a) {
    constexpr int KS = D / 16, DB = D / 32, BYTES = BM * D * 2, CH = D / 8, RPI = 64 / CH, NI = RW / RPI;
    constexpr int STAGE_ROW = D * 2 + 16;
    static_assert(RW % RPI == 0 && NI >= 1, "a wave's share of a tile is a whole number of load instructions");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[STAGES * 2 * BYTES];   // Q and G tiles, row-major, swizzled by ksa_swz
    __shared__ __attribute__((aligned(256))) float st[STAGES * 2 * BM];                // ... and their rows' statistics
    __shared__ __attribute__((aligned(16))) float own_lse[NW][BM];
    // the first K_LDS of a lane's K operands: kept in registers they would not fit
    constexpr int K_LDS = D == 128 ? 6 : 2;
    __shared__ __attribute__((aligned(1024))) bf16x8 k_lds[K_LDS > 0 ? K_LDS : 1][NW * 64];
    static_assert(NW * 32 * STAGE_ROW <= STAGES * 2 * BYTES, "the epilogue's staging area reuses the tile buffers");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 31, h = lane >> 5;
    // The lane number, opaque: what the tile loop needs only now and then is worked out again from it there, or the compiler
    // would keep it in registers that the loop does not have.
    auto lane_again = [&]() {
        int x = tid;
        asm volatile("" : "+v"(x));
        return x & 63;
    };
    const KeyView view = a.view;
    // ... and likewise the kernel's arguments: read again where they are needed in the loop
    auto args_again = [&]() {
        auto p = (const __attribute__((address_space(4))) DkvArgs *)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(p));
        return p;
    };
    // Workgroup index -> (entry, batch and KV head), the latter fastest: see ksa_prefill_direct.hip.
    int t = ksa_div(blockIdx.x, a.by_bh);
    const int bh = blockIdx.x - t * a.n_bh;
    const int b = ksa_div(bh, a.by_kv_heads), hkv = bh - b * a.n_kv_heads;
    int step_begin = 0, step_end = 0x7fffffff, slot = -1;
    if (a.scratch) {
        const KsaDkvEntry ent = a.entries[t];
        t = ent.tile, step_begin = ent.step_begin, step_end = ent.step_end, slot = ent.slot;
    }
    const int space = t >= a.sum_tiles ? KSA_SPACE_TEXT : KSA_SPACE_SUMMARY;
    const int n_space = space == KSA_SPACE_TEXT ? view.n_text : view.n_sum;
    const int k0 = (space == KSA_SPACE_TEXT ? t - a.sum_tiles : t) * KSA_DKV_KEYS;
    const int k_last = min(k0 + KSA_DKV_KEYS, n_space) - 1;
    // augmented row (Eq. 1) of a key
    const KsaDivisor by_own = space == KSA_SPACE_TEXT ? view.by_c : view.by_m;
    const int own_other = space == KSA_SPACE_TEXT ? view.m : view.c;
    static_assert(KSA_SPACE_TEXT == 0 && KSA_SPACE_SUMMARY == 1, "a run's number is its index space");
    auto key_row = [&](int idx) { return idx + (ksa_div(idx, by_own) + space) * own_other; };

    // ---- the lane's key: B operands of S = Q K^T and of G V^T (lanes past the end repeat the last one and store nothing)
    const int w_key0 = k0 + wave * 32;
    const bool w_any = w_key0 < n_space;
    const int key = min(w_key0 + r, n_space - 1);
    bf16x8 kreg[KS], vreg[KS];
    {
        const int64_t at = b * a.ks[0] + (int64_t)key_row(key) * a.ks[1] + hkv * a.ks[2] + h * 8;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            kreg[s] = *reinterpret_cast<const bf16x8 *>(a.k + at + s * 16);
            vreg[s] = *reinterpret_cast<const bf16x8 *>(a.v + at + s * 16);
        }
    }

    // ---- the sequence of query tiles: run 0 is the text rows, run 1 the summary rows, a step one head of one block ------
    int run_end[2], blk_n[2];      // rows before run_end, the last blk_n blocks of them
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const int lo = seen_by(view, space, k0, x).lo, hi = seen_by(view, space, k_last, x).hi;
        run_end[x] = hi;
        blk_n[x] = hi > lo ? (hi + BM - 1) / BM - lo / BM : 0;
    }
    const int steps0 = blk_n[0] * a.group;
    const int n_steps = min(steps0 + blk_n[1] * a.group, step_end) - step_begin;   // > 0: a key is seen by its own row

    // ---- the requests: one wave works out 64 of them at a time, one per lane, into LDS; a step reads the next one ---------
    struct Request {
        const char *q, *g;         // row `first` of the tile
        const char *stats;         // its statistics: 32 of the one kind, then 32 of the other
        uint32_t first;            // the tile's first row (a multiple of BM) with the run in bit 0
        uint32_t pattern;          // what the tile's other rows' places depend on: run | last row << 1 | border << 6
    };
    static_assert(sizeof(Request) == 32, "two 16-byte reads");
    __shared__ __attribute__((aligned(16))) unsigned char plan[2 * PLAN * sizeof(Request)];   // of two parts by turns
    auto plan_part = [&](int n0) {   // requests n0 .. n0 + 63; behind the last one: it again, into a stage nobody reads
        const auto *p = args_again();
        const int n = n0 + lane_again(), s = step_begin + min(n, n_steps - 1);
        const bool x = s >= steps0;
        const int in_run = s - (x ? steps0 : 0), ti = ksa_div(in_run, KsaDivisor{p->by_group.mul, p->by_group.shift});
        const int hq = hkv * p->group + in_run - ti * p->group;
        const int c = p->view.c, m = p->view.m, per = x ? m : c, other = x ? c : m, end = x ? run_end[1] : run_end[0];
        const int first = ((int)((unsigned)(end - 1) / BM) - ti) * BM;   // the blocks of a run from its last one down
        // (both quotients: a choice between the divisors would be a load per lane, which waits for the tiles in flight)
        const int by_c = ksa_div(first, KsaDivisor{p->view.by_c.mul, p->view.by_c.shift});
        const int by_m = ksa_div(first, KsaDivisor{p->view.by_m.mul, p->view.by_m.shift});
        const int j0 = x ? by_m : by_c;
        const int phase = first - j0 * per;
        const int64_t row0 = (int64_t)first + (x ? c : 0) + (int64_t)j0 * other;
        // Row k of the tile lies k + (chunk borders in between) * other rows behind the first: see ksa_prefill_direct.hip.  Chunks of
        // 64 rows and more have at most one border, at `border` = 64 - its distance; none in the tile counts as 0.
        int border = per < 64 ? phase : 64 - min(64, per - phase);
        if (per >= 64 && border <= 64 - BM) border = 0;
        Request r;
        r.q = (const char *)(p->q + b * p->qs[0] + row0 * p->qs[1] + hq * p->qs[2]);
        r.g = (const char *)(p->g + b * p->gs[0] + row0 * p->gs[1] + hq * p->gs[2]);
        r.stats = (const char *)(p->stats + 2 * ((int64_t)(b * p->n_q_heads + hq) * (p->nt_pad + p->ns_pad) + (x ? p->nt_pad : 0) + first));
        r.first = (uint32_t)first | (x ? 1u : 0u);
        r.pattern = (x ? 1u : 0u) | (uint32_t)(min(BM, end - first) - 1) << 1 | (uint32_t)border << 6;   // (rows behind the run may hold NaN)
        *reinterpret_cast<Request *>(plan + (n % (2 * PLAN)) * sizeof(Request)) = r;
    };
    if (wave < 2) plan_part(wave * PLAN);
#pragma unroll
    for (int s = 0; s < K_LDS; ++s) k_lds[s][tid] = kreg[s];
    __syncthreads();

    const unsigned lds0 = (unsigned)(size_t)lds, st0 = (unsigned)(size_t)&st[0];
    u32x4 next_lo, next_hi;        // the request behind the prepared one, as read from LDS
    auto read_request = [&](int n) {
        const unsigned char *at = plan + (n % (2 * PLAN)) * sizeof(Request);
        next_lo = *reinterpret_cast<const u32x4 *>(at), next_hi = *reinterpret_cast<const u32x4 *>(at + 16);
    };
    const char *rq_q, *rq_g, *rq_st;
    unsigned q_off[NI], g_off[NI], rq_first, rq_pattern = ~0u;
    auto take_request = [&]() {    // the one read last becomes the prepared one
        auto scalar = [](unsigned x) { return (unsigned)__builtin_amdgcn_readfirstlane((int)x); };
        auto pointer = [&](unsigned lo, unsigned hi) { return (const char *)((uint64_t)scalar(hi) << 32 | scalar(lo)); };
        rq_q = pointer(next_lo[0], next_lo[1]), rq_g = pointer(next_lo[2], next_lo[3]), rq_st = pointer(next_hi[0], next_hi[1]);
        rq_first = scalar(next_hi[2]);
        const unsigned pattern = scalar(next_hi[3]);
        if (pattern == rq_pattern) return;
        rq_pattern = pattern;
        const auto *p = args_again();
        const bool x = pattern & 1;
        const int per = x ? p->view.m : p->view.c, limit = (pattern >> 1) & 31;
        const unsigned other = (unsigned)(x ? p->view.c : p->view.m), mul = per < 64 ? (x ? p->small_m : p->small_c) : 1024u, add = (pattern >> 6) * mul;
        const unsigned q_row_bytes = (unsigned)p->qs[1] * 2u, g_row_bytes = (unsigned)p->gs[1] * 2u;
        const int lane = lane_again();
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int row = RW * wave + RPI * i + lane / CH;
            const unsigned k = min(row, limit);   // rows behind the run: its last one, masked
            const unsigned d_rows = k + ((__umul24(k, mul) + add) >> 16) * other;
            const unsigned col = (unsigned)(((lane % CH) ^ ksa_swz<D>(row)) << 4);
            q_off[i] = d_rows * q_row_bytes + col, g_off[i] = d_rows * g_row_bytes + col;
        }
    };
    constexpr int LOADS = 2 * NI + 1;
    auto issue = [&](int stage, int x) {   // load x of the prepared tile: Q and G by turns, then the statistics
        const unsigned dst = lds0 + stage * 2 * BYTES + (RW * wave + RPI * (x / 2)) * (D * 2);
        if (x == 2 * NI)
            lds_direct_load_4_s((const float *)rq_st, lane * 4, st0 + stage * 2 * BM * 4);
        else if (x % 2 == 0)
            lds_direct_load_16_s((const __bf16 *)rq_q, q_off[x / 2], dst);
        else
            lds_direct_load_16_s((const __bf16 *)rq_g, g_off[x / 2], dst + BYTES);
    };
    unsigned tile_first[STAGES - 1];   // `first` of the tiles that are on their way
    f32x16 dk[DB], dv[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) dk[db][e] = 0.f, dv[db][e] = 0.f;

    // K and V have arrived before the first request: the counted waits below are about tile requests only
    __builtin_amdgcn_s_waitcnt(0x0F70);
#pragma unroll
    for (int x = 0; x < STAGES; ++x) {
        read_request(x);
        take_request();
        if (x == STAGES - 1) break;
        tile_first[x] = rq_first;
#pragma unroll
        for (int y = 0; y < LOADS; ++y) issue(x, y);
    }

    // rows that see some key of the wave, and those that see every one of them, in the run of the tile in work
    const float sl = a.scale_log2e;
    int run = -1, some_lo = 0, some_hi = 0, all_lo = 0, all_hi = 0;
    auto enter_run = [&](int x) {
        run = x;
        const Seen first = seen_by(view, space, min(w_key0, n_space - 1), x), last = seen_by(view, space, min(w_key0 + 31, n_space - 1), x);
        some_lo = first.lo, some_hi = w_any ? last.hi : 0, all_lo = last.lo, all_hi = first.hi;
    };

    const int grp = lane >> 4, li = lane & 15;
    const int t_row = 4 * (grp >> 1) + (li >> 2), t_col = 16 * (grp & 1) + 4 * (li & 3);
    unsigned at_r = r * (D * 2) + ((h ^ ksa_swz<D>(r)) << 4);                                               // rows
    unsigned at_t = t_row * (D * 2) + (((t_col >> 3) ^ ksa_swz<D>(t_row)) << 4) + ((t_col & 7) << 1);       // columns

    // One tile: scores | dP with the exponentials between its MFMAs | dV with dS between its MFMAs | dK.  LDS operands are
    // read AHEAD MFMAs before the one that uses them.
    auto compute = [&](int stage, int req, int first, int step) {
        const float *const stats = &st[stage * 2 * BM + 4 * h];
        const float *lse = stats;
        const bool clip = (int)(first < all_lo) | (int)(first + BM > all_hi);
        f32x16 sacc, gacc;
#pragma unroll
        for (int e = 0; e < 16; ++e) sacc[e] = 0.f;
        constexpr int NM = 4 * KS, SLOTS = KS / 2;
        constexpr int AHEAD = D == 128 ? 3 : 2;
        bf16x8 op[NM], kop[K_LDS > 0 ? K_LDS : 1];
        auto read_op = [&](int x) {
            if (x < 2 * KS) {   // rows of Q, then of G
                op[x] = *reinterpret_cast<const bf16x8 *>(lds + (x / KS) * BYTES + (at_r ^ ((x % KS) << 5)));
                if (x < K_LDS) kop[x] = k_lds[x][tid];
            } else {            // columns of G, then of Q: rows R0 + t_row and R0 + 8 + t_row, whose swizzle differs by XOR 2
                const int y = x % KS, hf = y / DB, db = y % DB;
                const unsigned char *at = lds + (x < 3 * KS ? BYTES : 0) + hf * 16 * (D * 2);
                const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s16x4))(at + (at_t ^ (db << 6))));
                const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s16x4))(at + ((at_t ^ (((db * 4) ^ 2) << 4)) + 8 * (D * 2))));
                op[x] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        };
        bf16x8 pp[2], pd[2];
        float p[16];
        f32x4 l4[4];
        auto read_l = [&](int g4) { l4[g4] = *reinterpret_cast<const f32x4 *>(lse + 8 * g4); };
        auto weight = [&](int g) {
            if (g % 4 == 0 && g < 12) read_l(g / 4 + 1);   // one group ahead
            p[g] = __builtin_amdgcn_exp2f(fmaf(sacc[g], sl, -l4[g / 4][g % 4]));
            if (g % 2 == 1) pp[g / 8][g % 8 - 1] = (__bf16)p[g - 1], pp[g / 8][g % 8] = (__bf16)p[g];
        };
        auto grad = [&](int g) {
            p[g] *= gacc[g];
            if (g % 2 == 1) pd[g / 8][g % 8 - 1] = (__bf16)p[g - 1], pd[g / 8][g % 8] = (__bf16)p[g];
        };
#pragma unroll
        for (int x = 0; x < AHEAD; ++x) read_op(x);
        auto half_phase = [&](auto tag) {
            constexpr int ph = decltype(tag)::value / 2, half = decltype(tag)::value % 2;
#pragma unroll
            for (int y = half * SLOTS; y < (half + 1) * SLOTS; ++y) {
                const int x = ph * KS + y;
                if (x + AHEAD < NM) read_op(x + AHEAD);
                if (x == NM - SLOTS) read_request(step + STAGES);
                if (ph == 0 && y >= KS - 4) {   // dP starts from minus delta
                    const int g4 = y - (KS - 4);
                    const f32x4 nd = *reinterpret_cast<const f32x4 *>(stats + BM + 8 * g4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) gacc[4 * g4 + e] = nd[e];
                }
                if (ph == 1 && y == 0) read_l(0);
                KSA_FENCE();
                if constexpr (ph == 0) sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[x], y < K_LDS ? kop[y < K_LDS ? y : 0] : kreg[y], sacc, 0, 0, 0);
                if constexpr (ph == 1) gacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[x], vreg[y], gacc, 0, 0, 0);
                if constexpr (ph == 2) dv[y % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[x], pp[y / DB], dv[y % DB], 0, 0, 0);
                if constexpr (ph == 3) dk[y % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[x], pd[y / DB], dk[y % DB], 0, 0, 0);
                if constexpr (ph == 0) {
                    if (y < LOADS) issue(req, y);
                }
                // What the vector unit does behind this MFMA.  (Scores reach the register file behind two MFMAs of the next
                // phase; the products of rows 16 hf .. 16 hf + 15 need their weights.)
                if constexpr (ph == 1) {
                    for (int g = y < 2 ? 16 : (y - 2) * 10 / (KS - 2); g < (y - 1) * 10 / (KS - 2); ++g) weight(g);
                }
                if constexpr (ph == 2) {
                    if (y < SLOTS) { for (int g = 10 + y * 6 / SLOTS; g < 10 + (y + 1) * 6 / SLOTS; ++g) weight(g); }
                    else { for (int g = (y - SLOTS) * 8 / SLOTS; g < (y - SLOTS + 1) * 8 / SLOTS; ++g) grad(g); }
                }
                if constexpr (ph == 3) {
                    if (y < SLOTS) { for (int g = 8 + y * 8 / SLOTS; g < 8 + (y + 1) * 8 / SLOTS; ++g) grad(g); }
                }
                KSA_FENCE();
            }
        };
        auto phase = [&](auto tag) {
            constexpr int ph = decltype(tag)::value;
            half_phase(std::integral_constant<int, 2 * ph>{});
            half_phase(std::integral_constant<int, 2 * ph + 1>{});
        };
        phase(std::integral_constant<int, 0>{});
        if (__builtin_expect(clip, 0)) {   // register g is row first + 8 (g / 4) + 4 h + g % 4
            const int l = lane_again();
            const float row_lse = st[stage * 2 * BM + (l & 31)];
            if (__builtin_amdgcn_ballot_w64(!(row_lse > -INFINITY)) != 0) {
                // Rows whose log-sum-exp is no number: their weights are none, too, but for those of keys that they do not see,
                // which stay zeros (exp2 of minus infinity).
                own_lse[wave][l & 31] = row_lse > -INFINITY ? row_lse : 0.f;
#pragma unroll
                for (int g = 0; g < 16; ++g) sacc[g] = lse[8 * (g / 4) + g % 4] > -INFINITY ? sacc[g] : __builtin_nanf("");
                lse = &own_lse[wave][4 * (l >> 5)];
            }
            const auto *p = args_again();
            const KeyView view = {p->view.n_text, p->view.n_sum, p->view.c, p->view.m, p->view.C, p->view.self_only,
                                  {p->view.by_c.mul, p->view.by_c.shift}, {p->view.by_m.mul, p->view.by_m.shift}};
            const Seen mine = seen_by(view, space, min(w_key0 + (l & 31), n_space - 1), run);
            const int base = first + 4 * (l >> 5) - mine.lo;
            const unsigned n = (unsigned)max(mine.hi - mine.lo, 0);
#pragma unroll
            for (int g = 0; g < 16; ++g) sacc[g] = (unsigned)(base + 8 * (g / 4) + g % 4) < n ? sacc[g] : -INFINITY;
        }
        phase(std::integral_constant<int, 1>{});
        phase(std::integral_constant<int, 2>{});
        phase(std::integral_constant<int, 3>{});
    };

    static_assert(LOADS <= KS, "one load behind each MFMA of the scores");
    int stage = 0;
    for (int step = 0; step < n_steps; ++step) {
        constexpr int YOUNGER = (STAGES - 2) * LOADS;   // this wave's pieces of the tile have landed once only younger loads are outstanding
        static_assert(YOUNGER < 16, "the low bits of the count");
        __builtin_amdgcn_s_waitcnt(0x0F70 | YOUNGER);
        __syncthreads();   // ... and everybody's; nobody reads the stage any more that the next request overwrites
        const int first = (int)(tile_first[0] & ~1u), x = (int)(tile_first[0] & 1u), req = stage == 0 ? STAGES - 1 : stage - 1;
#pragma unroll
        for (int y = 0; y + 1 < STAGES - 1; ++y) tile_first[y] = tile_first[y + 1];
        tile_first[STAGES - 2] = rq_first;
        if (step % PLAN == 0 && step > 0 && wave == step / PLAN % NW) plan_part(step + PLAN);
        if (x != run) enter_run(x);
        if (first >= some_hi || first + BM <= some_lo) {   // nothing for this wave
#pragma unroll
            for (int y = 0; y < LOADS; ++y) issue(req, y);
            read_request(step + STAGES);
        } else {
            compute(stage, req, first, step);
        }
        take_request();
        const int by = stage == STAGES - 1 ? -stage * 2 * BYTES : 2 * BYTES;
        at_r += by, at_t += by, stage = stage == STAGES - 1 ? 0 : stage + 1;
    }

    __builtin_amdgcn_s_waitcnt(0x0F70);   // the loads behind the last tile have landed
    if (slot >= 0) {   // a piece: the partial sums as they sit in the registers, one 16-byte store per lane and four of them
        f32x4 *out = reinterpret_cast<f32x4 *>(a.scratch) + ((int64_t)slot * a.n_bh + bh) * (KSA_DKV_KEYS * D / 2) + wave * (D * 16) + lane_again();
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                f32x4 xk, xv;
#pragma unroll
                for (int e = 0; e < 4; ++e) xk[e] = dk[db][g4 * 4 + e], xv[e] = dv[db][g4 * 4 + e];
                out[(db * 4 + g4) * 128] = xk, out[(db * 4 + g4) * 128 + 64] = xv;
            }
        return;
    }
    __syncthreads();   // everybody is done with the tiles: each wave's 32 x D block goes through them, whole rows are stored
    unsigned char *stg = lds + wave * (32 * STAGE_ROW);
    const int lane_end = lane_again(), piece = lane_end % CH;
    auto store = [&](__bf16 *out, const f32x16 (&acc)[DB], float scale) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                bf16x4 pk;
#pragma unroll
                for (int e = 0; e < 4; ++e) pk[e] = (__bf16)(acc[db][g4 * 4 + e] * scale);
                *reinterpret_cast<bf16x4 *>(stg + (lane_end & 31) * STAGE_ROW + (db * 32 + g4 * 8 + (lane_end >> 5) * 4) * 2) = pk;
            }
        __bf16 *const col = out + b * a.dks[0] + hkv * a.dks[2] + piece * 8;
#pragma unroll
        for (int i = 0; i < 32 / RPI; ++i) {
            const int row = RPI * i + lane_end / CH;
            const u32x4 x = *reinterpret_cast<const u32x4 *>(stg + row * STAGE_ROW + piece * 16);
            if (w_key0 + row < n_space) *reinterpret_cast<u32x4 *>(col + (int64_t)key_row(w_key0 + row) * a.dks[1]) = x;
        }
    };
    store(a.dk, dk, a.scale);
    store(a.dv, dv, 1.f);
}

}  // namespace

void ksa_launch_dkv_direct(const KsaPrefillBwdLaunch &L, const float *stats, float *scratch, int entries, void *stream) {
    DkvArgs a;
    a.q = static_cast<const __bf16 *>(L.q);
    a.k = static_cast<const __bf16 *>(L.k);
    a.v = static_cast<const __bf16 *>(L.v);
    a.g = static_cast<const __bf16 *>(L.d_o);
    a.stats = stats;
    a.dk = static_cast<__bf16 *>(L.dk);
    a.dv = static_cast<__bf16 *>(L.dv);
    a.scratch = scratch;
    a.entries = L.dkv_entries;
    for (int x = 0; x < 3; ++x) a.qs[x] = L.q_strides[x], a.ks[x] = L.kv_strides[x], a.gs[x] = L.o_strides[x], a.dks[x] = L.dkv_strides[x];
    const ksa_params &p = L.p;
    a.view.n_text = p.n_text, a.view.n_sum = (p.n_text / p.chunk_len) * p.n_summary;
    a.view.c = p.chunk_len, a.view.m = p.n_summary, a.view.C = p.window_chunks;
    a.view.self_only = (p.flags & KSA_FLAG_SUMMARY_SELF_ONLY) ? 1 : 0;
    a.n_q_heads = p.n_q_heads, a.n_kv_heads = p.n_kv_heads, a.group = p.n_q_heads / p.n_kv_heads;
    a.n_bh = p.batch * p.n_kv_heads;
    a.sum_tiles = (a.view.n_sum + KSA_DKV_KEYS - 1) / KSA_DKV_KEYS;
    a.nt_pad = (a.view.n_text + 63) / 64 * 64, a.ns_pad = (a.view.n_sum + 63) / 64 * 64;
    a.small_c = (65535 + a.view.c) / a.view.c, a.small_m = a.view.m > 0 ? (65535 + a.view.m) / a.view.m : 0;
    a.view.by_c = ksa_divisor(a.view.c), a.view.by_m = ksa_divisor(a.view.m > 0 ? a.view.m : 1);
    a.by_bh = ksa_divisor(a.n_bh), a.by_kv_heads = ksa_divisor(a.n_kv_heads), a.by_group = ksa_divisor(a.group);
    a.scale = p.softmax_scale, a.scale_log2e = p.softmax_scale * 1.4426950408889634f;
    const dim3 grid((unsigned)(entries * a.n_bh)), block(NW * 64);
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (p.head_dim == 128)
        hipLaunchKernelGGL(ksa_bwd_dkv_direct_kernel<128>, grid, block, 0, st, a);
    else
        hipLaunchKernelGGL(ksa_bwd_dkv_direct_kernel<64>, grid, block, 0, st, a);
}

// KSA decode for gfx950: one new text token per sequence attends over the summary KV cache
// (section 2.3.1).  The work is bandwidth bound: every visible K and V row is read from HBM exactly once
// per KV head and serves all Hq/Hkv query heads of that head.
//
// Split-K: a workgroup streams one span of the visible rows of one (sequence, KV head).  Of head_dim bf16 a V row is read by
// head_dim / 8 adjacent lanes with one 16-byte load each; U such loads of K and of V are in flight per lane.  Each lane keeps
// its 8 columns of the output for all query heads of the group, and every lane group runs its own online softmax on the rows
// it saw.  The lane groups of a wave are merged by lane swaps, the waves through LDS, into one partial (max, sum, o) per query
// head; a second kernel merges the spans of a sequence by log-sum-exp.  With one span per sequence (a summary token's few
// rows, small caches) the workgroup stores the result itself and there is no second kernel.  How many spans: plan_decode() in
// ksa_api.cpp.  With a million rows and more they are dealt by the sequences' lengths, which only the device knows: every workgroup
// works out its own from all positions (batch 64 at 128K, lengths 1 : 4: 511 us, dealt 457; all alike 658, 655).
//
// Scores: with four and eight query heads per KV head from the matrix unit, S^T = K Q^T with v_mfma_f32_16x16x32_bf16: 16 cache
// rows by G heads (repeated over the 16 columns), fp32 sums of exact products.  Lane l receives the scores of rows
// 4 (l / 16) + i, i < 4, for head l % G; the V rows it loads are dealt so that they are these same rows, and the (fp32) weights
// of the other heads are a DPP move away.  With one and two heads they are dot products on the vector unit, 8 columns per lane
// and a 4-step DPP all-reduce over the row's lanes.
// What bounds it: HBM reads where the launch fills the chip (batch 64 at a 128K context, 4.33 GB: 655 us, 6.6 TB/s; scores on the
// vector unit 670; with few rows the two launches and their chains of loads: 2000 rows, batch 1, 8/4 heads 7.5, before 16.0, when
// spans had 768 rows at least).  With eight heads the vector unit was the bound: batch 32, 64K context, 8/1 heads 58.1 / 37.2 us, window
// 1024 with batch 64 41.1 / 28.2; batch 3, 20K, d 64 22.3 / 16.6.  With four: 32K, batch 4 and append 26.1 / 24.7, 128K, batch 1
// 23.9 / 22.6.  With one head the matrix unit's operand reads (64 bytes of 16 rows instead of four whole rows) lost: batch 32,
// 32K, 16/16 heads 163.9 us on the vector unit, 169.0.  With two heads likewise where there are few spans (vector / matrix unit,
// 64K, batch 8 30.4 / 32.9, d 64, batch 16 27.9 / 30.6, 128K in the paper's form, batch 1 17.2 / 18.8); level or behind on full
// launches (64K, batch 32 86.7 / 87.3, 128K, batch 16 176.5 / 171.9, window 1024, batch 64 29.8 / 24.1).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <utility>

#include "ksa_device.h"
#include "ksa_internal.h"

// Scratch memory of ksa_decode_fwd_static: the partial (o, max, sum) records of the spans, which ksa_decode_fwd
// keeps in the caller's workspace.  Every GPU the library runs on holds its own copy of the array, at its own
// address, until the process ends.  In host code the array's name is only a handle for hipGetSymbolAddress; the
// device address it returns (ksa_decode_static_scratch below) is what kernels and HIP calls are given.
static __device__ __align__(256) unsigned char scratch[KSA_DECODE_STATIC_SCRATCH_BYTES];

namespace {

constexpr int U = 4;         // row loads in flight per lane, K and V each

struct DecodeArgs {
    const __bf16 *q, *k, *v;
    const int32_t *pos;
    __bf16 *o;
    float *lse;
    float *ws;
    int64_t cs[3];   // {batch, head, row} strides of the caches in elements
    int32_t n_splits, s_cap;   // n_splits: spans per sequence; 0: the n_spans of a KV head are dealt by the sequences' lengths
    int32_t n_spans;           // per KV head, all sequences together
    int32_t batch;
    int32_t kind, self_only;   // KSA_ROW_TEXT / KSA_ROW_SUMMARY query; flag bit 0 of the parameters
    int32_t c, m, C, n_text;
    int32_t n_q_heads, n_kv_heads;
    KsaDivisor by_c, by_m, by_slots;   // chunk_len, n_summary, window_chunks + 1
    float scale_log2e;
    float q_scale, score_scale;   // scale_log2e in two factors, the first a power of two
};

struct Ranges {
    int off0, n0, off1, n1, off2, n2;   // summaries [off0, off0+n0), ring [off1, off1+n1), ring [off2, off2+n2)
};

// Is p a position the query kind can have?  (text index / summary ordinal)
__device__ __forceinline__ bool valid_pos(const DecodeArgs &a, int p) {
    return p >= 0 && p < (a.kind == KSA_ROW_TEXT ? a.n_text : a.s_cap);
}

// Rows the query reads (Eq. 3 mapped onto the cache geometry); all zero if p is invalid.
// Text token at text index p: the summaries of the chunks that have left the window and the text of the window up to
// itself.  Summary token with ordinal p = j m + slot: the summaries of its chunk up to itself (only itself with
// self_only) and the text of its chunk, one whole ring slot.
__device__ __forceinline__ Ranges visible_rows(const DecodeArgs &a, int p) {
    Ranges R = {0, 0, 0, 0, 0, 0};
    if (!valid_pos(a, p)) return R;
    if (a.kind == KSA_ROW_SUMMARY) {
        const int j = ksa_div(p, a.by_m), slot = p - j * a.m;
        R.off0 = a.self_only ? p : j * a.m;
        R.n0 = a.self_only ? 1 : slot + 1;
        R.off1 = a.s_cap + (j - ksa_div(j, a.by_slots) * (a.C + 1)) * a.c;
        R.n1 = a.c;
        return R;
    }
    const int j = ksa_div(p, a.by_c), r = p - j * a.c;
    const int slot = j - ksa_div(j, a.by_slots) * (a.C + 1);
    R.n0 = (j - a.C > 0 ? j - a.C : 0) * a.m;
    R.off1 = a.s_cap;
    R.n1 = slot * a.c + r + 1;
    R.off2 = a.s_cap + (slot + 1) * a.c;
    R.n2 = j >= a.C ? (a.C - slot) * a.c : 0;
    return R;
}

__device__ __forceinline__ int phys_row(const Ranges &R, int v) {
    if (v < R.n0) return R.off0 + v;
    v -= R.n0;
    if (v < R.n1) return R.off1 + v;
    return R.off2 + (v - R.n1);
}

// how far behind its position v among the visible rows a row lies in the cache
__device__ __forceinline__ int row_shift(const Ranges &R, int v) {
    const int ring = v < R.n0 + R.n1 ? R.off1 - R.n0 : R.off2 - R.n0 - R.n1;
    return v < R.n0 ? R.off0 : ring;
}

// A score lives in the lane of its query head: lane l holds head l % G.  The value of head g among a lane's neighbours that hold
// the same rows: the 16 lanes of a row of lanes, with D = 64 its halves.
template <int D, int G, int g>
__device__ __forceinline__ float of_head(float x) {
    const int u = __builtin_bit_cast(int, x);
    if constexpr (G == 1) return x;
    else if constexpr (G <= 4) return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, u, g * 0x55, 0xf, 0xf, true));   // quad_perm [g,g,g,g]
    else {
        const int lo = __builtin_amdgcn_update_dpp(0, u, 0x150 + g, 0xf, 0xf, true);   // row_newbcast: lane g of the 16
        if constexpr (D == 128) return __builtin_bit_cast(float, lo);
        else return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(lo, u, 0x158 + g, 0xf, 0xc, false));   // ... 8 + g for the upper 8
    }
}
template <int D, int G, typename F, int... g>
__device__ __forceinline__ void heads_of(float x, F &&use, std::integer_sequence<int, g...>) {
    (use(g, of_head<D, G, g>(x)), ...);
}
template <int D, int G, typename F>
__device__ __forceinline__ void for_heads(float x, F &&use) {   // use(g, value of head g)
    heads_of<D, G>(x, use, std::make_integer_sequence<int, G>{});
}

// eight bf16 -> eight fp32 (a bf16 is the high half of an fp32)
__device__ __forceinline__ void unpack8(const u32x4 &x, float f[8]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        f[2 * e] = __builtin_bit_cast(float, x[e] << 16);
        f[2 * e + 1] = __builtin_bit_cast(float, x[e] & 0xffff0000u);
    }
}

template <int D>
__device__ __forceinline__ void store_result(const DecodeArgs &a, int b, int hq, int col, bool valid, float acc, float den, float M) {
    const float out = valid ? acc / den : __builtin_nanf("");
    a.o[((int64_t)b * a.n_q_heads + hq) * D + col] = (__bf16)out;
    if (a.lse && col == 0)
        a.lse[(int64_t)b * a.n_q_heads + hq] = valid ? M * 0.6931471805599453f + __logf(den) : __builtin_nanf("");
}

// values of lane l ^ 16 (rows of 16 lanes swapped pairwise) and of lane l ^ 32
__device__ __forceinline__ float swap16(float x) {
    const unsigned u = __builtin_bit_cast(unsigned, x);
    auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return __builtin_bit_cast(float, (threadIdx.x & 16) ? r[0] : r[1]);
}
__device__ __forceinline__ float swap32(float x) {
    const unsigned u = __builtin_bit_cast(unsigned, x);
    auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __builtin_bit_cast(float, (threadIdx.x & 32) ? r[0] : r[1]);
}
__device__ __forceinline__ float swap8(float x) {   // lane l ^ 8: row_ror 8
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x128, 0xf, 0xf, false));
}

// Spans dealt by length: how the n_spans of a KV head are shared out among at most 64 sequences; lane l holds sequence l's part.
// Sequence b takes n_b = max(1, ceil(N_b / per)) of them, `per` nearly the smallest for which they are enough.  With T rows in all,
// per = T / (n_spans - batch) always is: sum(n_b) <= T / per + batch (plan_decode() gives two and more per sequence).
// The merge kernel works the same out again, and every instantiation of both has to come to the same numbers: one span more or less for
// one sequence and the merge would read the records of others.  So nothing here is left to the compiler's choice: sums in a given order,
// and no product fused into a sum.
struct Deal {
    Ranges R;
    int n, behind;   // spans of the sequence; of it and of those in front of it
};
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_scan(int x) { return x + __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xf, false); }
__device__ __forceinline__ Deal deal_spans(const DecodeArgs &a) {
#pragma clang fp contract(off)
    const int lane = threadIdx.x & 63;
    const bool any = lane < a.batch;
    Deal d;
    d.R = visible_rows(a, a.pos[min(lane, a.batch - 1)]);
    const int N = d.R.n0 + d.R.n1 + d.R.n2;
    if (__builtin_amdgcn_ballot_w64(N != __builtin_amdgcn_readfirstlane(N)) == 0) {   // all alike (lanes without a sequence repeat the last one)
        d.n = (int)((unsigned)a.n_spans / (unsigned)a.batch);
        d.behind = min(lane + 1, a.batch) * d.n;
        return d;
    }
    const float rows = any ? (float)N : 0.f;
    auto total = [](float x) {
        x = row_allreduce<16>(x);
        x += swap16(x);
        return x + swap32(x);
    };
    auto spans = [&](float per) { return any ? fmaxf(ceilf(rows * __builtin_amdgcn_rcpf(per)), 1.f) : 0.f; };
    // (the factors keep a quotient that should be whole from being rounded up to the next number)
    const float all = fmaxf(total(rows), 1.f), most = (float)a.n_spans;
    float lo = all * __builtin_amdgcn_rcpf(most) * 1.0001f, hi = all * __builtin_amdgcn_rcpf(most - (float)a.batch) * 1.0002f;
    float per = lo;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (total(spans(per)) <= most) hi = per; else lo = per;
        per = 0.5f * (lo + hi);
    }
    d.n = (int)spans(hi);
    int x = d.n;   // sums over the lanes up to this one
    x = dpp_scan<0x111, 0xf>(x);   // row_shr 1, 2, 4, 8
    x = dpp_scan<0x112, 0xf>(x);
    x = dpp_scan<0x114, 0xf>(x);
    x = dpp_scan<0x118, 0xf>(x);
    x = dpp_scan<0x142, 0xa>(x);   // row_bcast 15: the last lane of rows 0 and 2 to rows 1 and 3
    x = dpp_scan<0x143, 0xc>(x);   // row_bcast 31
    d.behind = x;
    return d;
}

// What a workgroup works on: rows [v0, v1) of the visible rows R of sequence b for KV head hkv; b < 0: nothing.  Wave-uniform.
struct Span {
    Ranges R;
    int b, hkv, v0, v1;
    int record;   // number of the span's record among those of a query head
};
template <bool DEAL>
__device__ __forceinline__ Span find_span(const DecodeArgs &a) {
    Span s;
    const int x = blockIdx.x;
    if constexpr (!DEAL) {
        s.b = blockIdx.z, s.hkv = blockIdx.y, s.record = s.b * a.n_splits + x;
        s.R = visible_rows(a, a.pos[s.b]);
        const int N = s.R.n0 + s.R.n1 + s.R.n2, per = (N + a.n_splits - 1) / a.n_splits;
        s.v0 = x * per, s.v1 = min(N, s.v0 + per);
        return s;
    }
    // one wave deals (all of them took the launch 4 % at batch 64); workgroups by sequence, KV head, span, the last fastest
    __shared__ int found[9];
    if (threadIdx.x < 64) {
        const Deal d = deal_spans(a);
        const uint64_t from = __builtin_amdgcn_ballot_w64(d.behind * a.n_kv_heads > x);   // (lanes behind the last sequence hold the sum of all)
        const int at = from ? __builtin_ctzll(from) : 0;
        if ((int)threadIdx.x == at) {
            found[0] = from ? at : -1, found[1] = d.R.off0, found[2] = d.R.n0, found[3] = d.R.off1, found[4] = d.R.n1, found[5] = d.R.off2;
            found[6] = d.R.n2, found[7] = d.n, found[8] = d.behind;
        }
    }
    __syncthreads();
    auto get = [&](int y) { return __builtin_amdgcn_readfirstlane(found[y]); };
    s.b = get(0);
    s.R = {get(1), get(2), get(3), get(4), get(5), get(6)};
    const int N = s.R.n0 + s.R.n1 + s.R.n2, n = get(7), first = get(8) - n;
    const int in_b = x - first * a.n_kv_heads;
    s.hkv = (int)((unsigned)in_b / (unsigned)n);
    const int split = in_b - s.hkv * n;
    const int per = (N + n - 1) / n;
    s.v0 = split * per, s.v1 = min(N, s.v0 + per);
    s.record = first + split;
    return s;
}

// the waves' partial results -> the workgroup's: its record in the workspace, or with one span per sequence the result
template <int D, int G, int NT>
__device__ __forceinline__ void merge_waves(const DecodeArgs &a, const Span &s, const float (&sh_o)[NT / 64][G][D],
                                            const float (&sh_m)[NT / 64][G], const float (&sh_l)[NT / 64][G]) {
    constexpr int NW = NT / 64;
    __syncthreads();
    for (int x = (int)threadIdx.x; x < G * D; x += NT) {
        const int g = x / D, col = x % D;
        float M = sh_m[0][g];
#pragma unroll
        for (int y = 1; y < NW; ++y) M = fmaxf(M, sh_m[y][g]);
        float acc = 0.f, den = 0.f;
#pragma unroll
        for (int y = 0; y < NW; ++y) {
            const float w = __builtin_amdgcn_exp2f(sh_m[y][g] - M);
            acc += sh_o[y][g][col] * w, den += sh_l[y][g] * w;
        }
        const int hq = s.hkv * G + g;
        if (a.n_splits == 1) {
            store_result<D>(a, s.b, hq, col, valid_pos(a, a.pos[s.b]), acc, den, M);
        } else {
            float *rec = a.ws + ((int64_t)hq * a.n_spans + s.record) * (D + 2);
            rec[col] = acc;
            if (col == 0) rec[D] = M, rec[D + 1] = den;
        }
    }
}

// partial record in the workspace: [D] unnormalised o, then running max (log2 domain), then running sum
template <int D, int G, int NT, bool DEAL>
__global__ __launch_bounds__(NT) void ksa_decode_split_kernel(const DecodeArgs a) {
    constexpr int LPR = D / 8;          // lanes per cache row
    constexpr int RPW = 64 / LPR;       // rows per wavefront load
    constexpr int NW = NT / 64;
    constexpr int R_IT = NW * RPW * U;  // rows per workgroup iteration

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int chunk = lane % LPR, gi = lane / LPR;

    const Span span = find_span<DEAL>(a);
    const int b = span.b, hkv = span.hkv, v0 = span.v0, v1 = span.v1;
    if (DEAL && b < 0) return;
    const Ranges R = span.R;

    float qf[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const u32x4 raw = *reinterpret_cast<const u32x4 *>(a.q + ((int64_t)b * a.n_q_heads + hkv * G + g) * D + chunk * 8);
        unpack8(raw, qf[g]);
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[g][e] *= a.scale_log2e;
    }
    float m_run[G], l_run[G], o[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        m_run[g] = -1e30f;
        l_run[g] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[g][e] = 0.f;
    }

    const __bf16 *kb = a.k + b * a.cs[0] + hkv * a.cs[1] + chunk * 8;
    const __bf16 *vb = a.v + b * a.cs[0] + hkv * a.cs[1] + chunk * 8;

    for (int base = v0 + wave * (RPW * U); base < v1; base += R_IT) {
        u32x4 kk[U], vv[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int vr = base + u * RPW + gi;
            ok[u] = vr < v1;
            const int64_t off = (int64_t)phys_row(R, ok[u] ? vr : v1 - 1) * a.cs[2];
            kk[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(kb + off));
            vv[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(vb + off));
        }
        float s[U][G];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float kf[8];
            unpack8(kk[u], kf);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float acc = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) acc = fmaf(qf[g][e], kf[e], acc);
                acc = row_allreduce<LPR>(acc);
                s[u][g] = ok[u] ? acc : -INFINITY;
            }
        }
        float p[U][G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float mx = s[0][g];
#pragma unroll
            for (int u = 1; u < U; ++u) mx = fmaxf(mx, s[u][g]);
            const float m_new = fmaxf(m_run[g], mx);
            const float alpha = __builtin_amdgcn_exp2f(m_run[g] - m_new);
            m_run[g] = m_new;
            float sum = 0.f;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                p[u][g] = __builtin_amdgcn_exp2f(s[u][g] - m_new);
                sum += p[u][g];
            }
            l_run[g] = l_run[g] * alpha + sum;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[g][e] *= alpha;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float vf[8];
            unpack8(vv[u], vf);
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int e = 0; e < 8; ++e) o[g][e] = fmaf(p[u][g], vf[e], o[g][e]);
        }
    }

    // ---- merge the lane groups of each wave, then the waves -----------------------------------------
    __shared__ float sh_o[NW][G][D];
    __shared__ float sh_m[NW][G], sh_l[NW][G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        float M = m_run[g];
        if (LPR == 8) M = fmaxf(M, swap8(M));
        M = fmaxf(M, swap16(M));
        M = fmaxf(M, swap32(M));
        const float f = __builtin_amdgcn_exp2f(m_run[g] - M);
        auto merge = [&](float x) {
            x *= f;
            if (LPR == 8) x += swap8(x);
            x += swap16(x);
            return x + swap32(x);
        };
        const float l = merge(l_run[g]);
#pragma unroll
        for (int e = 0; e < 8; ++e) o[g][e] = merge(o[g][e]);
        if (gi == 0) {
#pragma unroll
            for (int e = 0; e < 8; ++e) sh_o[wave][g][chunk * 8 + e] = o[g][e];
            if (chunk == 0) sh_m[wave][g] = M, sh_l[wave][g] = l;
        }
    }
    merge_waves<D, G, NT>(a, span, sh_o, sh_m, sh_l);
}

// the same with scores from the matrix unit: four and eight query heads per KV head
template <int D, int G, int NT, bool DEAL>
__global__ __launch_bounds__(NT) void ksa_decode_split_matrix_kernel(const DecodeArgs a) {
    constexpr int LPR = D / 8;          // lanes per V row
    constexpr int RPW = 64 / LPR;       // V rows per wavefront load
    constexpr int KB = RPW * U / 16;    // blocks of 16 rows per wavefront and iteration
    constexpr int KS = D / 32;          // k steps of the score MFMA
    constexpr int NW = NT / 64;
    constexpr int R_IT = NW * RPW * U;  // rows per workgroup iteration
    static_assert(KB * KS == U && U == 4, "as many loads of K as of V");

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int chunk = lane % LPR, gi = lane / LPR;
    const int v_row = (D == 64 ? 16 * (gi & 1) : 0) + 4 * (lane >> 4);   // the lane's V rows: v_row .. v_row + 3

    const Span span = find_span<DEAL>(a);
    const int b = span.b, hkv = span.hkv, v0 = span.v0, v1 = span.v1;
    if (DEAL && b < 0) return;
    const Ranges R = span.R;

    bf16x8 qreg[KS];
    {
        const __bf16 *qp = a.q + ((int64_t)b * a.n_q_heads + hkv * G + lane % G) * D + (lane >> 4) * 8;
#pragma unroll
        for (int s = 0; s < KS; ++s) qreg[s] = *reinterpret_cast<const bf16x8 *>(qp + s * 32);
    }
    float m_run, l_run, o[G][8], largest;   // largest: of the lane's products; a NaN stays

    const __bf16 *kb = a.k + b * a.cs[0] + hkv * a.cs[1] + (lane >> 4) * 8;
    const __bf16 *vb = a.v + b * a.cs[0] + hkv * a.cs[1] + chunk * 8;

    const int64_t row = a.cs[2];
    auto walk = [&](const bf16x8 (&q)[KS], float to_score) {
        m_run = -1e30f, l_run = 0.f, largest = 0.f;
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int e = 0; e < 8; ++e) o[g][e] = 0.f;
        for (int base = v0 + wave * (RPW * U); base < v1; base += R_IT) {
            // Nearly all blocks lie in one piece of the cache and before the end: then a scalar offset moves the lane's addresses.
            // (The shift never decreases from one visible row to the next, so equal ends mean one piece.)
            const int end = base + RPW * U, shift = row_shift(R, base);
            const bool whole = end <= v1 && row_shift(R, end - 1) == shift;
            int64_t k_at[KB], v_at[U];
            if (whole) {
                const int64_t first = (int64_t)(base + shift) * row;
#pragma unroll
                for (int x = 0; x < KB; ++x) k_at[x] = (lane & 15) * row + (first + 16 * x * row);
#pragma unroll
                for (int u = 0; u < U; ++u) v_at[u] = v_row * row + (first + u * row);
            } else {
                auto offset = [&](int v) { v = min(v, v1 - 1); return (int64_t)(v + row_shift(R, v)) * row; };
#pragma unroll
                for (int x = 0; x < KB; ++x) k_at[x] = offset(base + 16 * x + (lane & 15));
#pragma unroll
                for (int u = 0; u < U; ++u) v_at[u] = offset(base + v_row + u);
            }
            u32x4 kk[KB][KS], vv[U];
#pragma unroll
            for (int x = 0; x < KB; ++x)
#pragma unroll
                for (int s = 0; s < KS; ++s) kk[x][s] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(kb + k_at[x] + s * 32));
#pragma unroll
            for (int u = 0; u < U; ++u) vv[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(vb + v_at[u]));
            __builtin_amdgcn_sched_barrier(0);   // all loads of the block are on their way
            f32x4 acc[KB];
#pragma unroll
            for (int x = 0; x < KB; ++x) {
                acc[x] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < KS; ++s)
                    acc[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kk[x][s]), q[s], acc[x], 0, 0, 0);
                largest = __builtin_elementwise_maximum(__builtin_elementwise_maximum(largest, fabsf(acc[x][0])), fabsf(acc[x][1]));
                largest = __builtin_elementwise_maximum(__builtin_elementwise_maximum(largest, fabsf(acc[x][2])), fabsf(acc[x][3]));
            }
            float p[U], mx = m_run;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float s = (KB == 1 || !(gi & 1) ? acc[0][u] : acc[KB - 1][u]) * to_score;
                p[u] = base + v_row + u < v1 ? s : -INFINITY;
                mx = fmaxf(mx, p[u]);
            }
            if (__builtin_amdgcn_ballot_w64(mx > m_run) != 0) {
                const float alpha = __builtin_amdgcn_exp2f(m_run - mx);
                l_run *= alpha, m_run = mx;
                for_heads<D, G>(alpha, [&](int g, float x) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[g][e] *= x;
                });
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                p[u] = __builtin_amdgcn_exp2f(p[u] - m_run);
                l_run += p[u];
                float vf[8];
                unpack8(vv[u], vf);
                for_heads<D, G>(p[u], [&](int g, float x) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[g][e] = fmaf(x, vf[e], o[g][e]);
                });
            }
        }
    };
    walk(qreg, a.scale_log2e);
    // Products that overflow may be scores that do not: the wave's rows once more with the scale's power of two in q (exact).  A
    // sum that was infinite at any time is so in the end, or a NaN.  (The look at the products costs the smallest launches 1 - 2 %:
    // one span of 1500 rows, 16 workgroups 21.3 / 21.7 us; scaling every q before the loop 4 %, in it 4 %, a look per block 4 %.)
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(largest < INFINITY)) != 0, 0)) {
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int e = 0; e < 8; ++e) qreg[s][e] = (__bf16)((float)qreg[s][e] * a.q_scale);
        walk(qreg, a.score_scale);
    }

    // ---- merge the lane groups of each wave, then the waves -----------------------------------------
    __shared__ float sh_o[NW][G][D];
    __shared__ float sh_m[NW][G], sh_l[NW][G];
    float M = m_run;
    if (LPR == 8) M = fmaxf(M, swap8(M));
    M = fmaxf(M, swap16(M));
    M = fmaxf(M, swap32(M));
    const float f = __builtin_amdgcn_exp2f(m_run - M);
    auto merge = [&](float x) {
        if (LPR == 8) x += swap8(x);
        x += swap16(x);
        return x + swap32(x);
    };
    const float l = merge(l_run * f);
    if (lane < G) sh_m[wave][lane] = M, sh_l[wave][lane] = l;
    for_heads<D, G>(f, [&](int g, float x) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float sum = merge(o[g][e] * x);
            if (gi == 0) sh_o[wave][g][chunk * 8 + e] = sum;
        }
    });
    merge_waves<D, G, NT>(a, span, sh_o, sh_m, sh_l);
}

// One workgroup per (batch, query head): log-sum-exp merge of the spans.  Part y of its MP parts of D threads takes spans
// MU y .. MU y + MU - 1 of every MP MU, whose loads travel together, the first ones beside those of the maxima and sums; the weights of
// 64 spans live in the lanes of every wave.
constexpr int MU = 8;
template <int D, bool DEAL, int MP>
__global__ __launch_bounds__(MP * D) void ksa_decode_merge_kernel(const DecodeArgs a) {
    const int hq = blockIdx.x, b = blockIdx.y, col = threadIdx.x % D, lane = threadIdx.x & 63;
    const int part = __builtin_amdgcn_readfirstlane(threadIdx.x / D);
    int first = b * a.n_splits, n = a.n_splits;
    if constexpr (DEAL) {
        __shared__ int found[2];
        if (threadIdx.x < 64) {
            const Deal d = deal_spans(a);
            if ((int)threadIdx.x == b) found[0] = d.n, found[1] = d.behind - d.n;   // (the first wave's lane: at most 64 sequences)
        }
        __syncthreads();
        n = __builtin_amdgcn_readfirstlane(found[0]), first = __builtin_amdgcn_readfirstlane(found[1]);
    }
    const float *rec = a.ws + ((int64_t)hq * a.n_spans + first) * (D + 2);
    auto at = [&](int s) { return rec + (int64_t)min(s, n - 1) * (D + 2); };
    float o[MU];
    auto load = [&](int s) {
#pragma unroll
        for (int u = 0; u < MU; ++u) o[u] = at(s + u)[col];
    };
    auto stats = [&](int s, float &m, float &l) { m = at(s + lane)[D], l = s + lane < n ? at(s + lane)[D + 1] : 0.f; };
    float m, l, acc = 0.f, den = 0.f;
    stats(0, m, l);
    load(MU * part);
    const bool valid = valid_pos(a, a.pos[b]);
    float M = m;
    for (int s = 64; s < n; s += 64) M = fmaxf(M, at(s + lane)[D]);
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) M = fmaxf(M, __shfl_xor(M, d));
    for (int s = 0; s < n; s += 64) {
        if (s > 0) stats(s, m, l);
        const float w = __builtin_amdgcn_exp2f(m - M);
        den += l * w;
        for (int x = MU * part; x < min(64, n - s); x += MP * MU) {
            if (s + x != MU * part) load(s + x);
#pragma unroll
            for (int u = 0; u < MU; ++u)
                if (s + x + u < n) acc += o[u] * __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, w), x + u));
        }
    }
    if constexpr (MP > 1) {
        __shared__ float parts[MP][D];
        parts[part][col] = acc;
        __syncthreads();
        if (part > 0) return;
#pragma unroll
        for (int y = 1; y < MP; ++y) acc += parts[y][col];
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) den += __shfl_xor(den, d);
    store_result<D>(a, b, hq, col, valid, acc, den, M);
}

template <int D, int G, int NT, bool DEAL>
void launch(const DecodeArgs &a, hipStream_t st) {
    const dim3 grid = DEAL ? dim3(a.n_spans * a.n_kv_heads) : dim3(a.n_splits, a.n_kv_heads, a.batch);
    if constexpr (G >= 4)
        hipLaunchKernelGGL((ksa_decode_split_matrix_kernel<D, G, NT, DEAL>), grid, dim3(NT), 0, st, a);
    else
        hipLaunchKernelGGL((ksa_decode_split_kernel<D, G, NT, DEAL>), grid, dim3(NT), 0, st, a);
    if (a.n_splits == 1) return;
    const dim3 outputs(a.n_q_heads, a.batch);
    if (a.n_spans > 8 * a.batch)
        hipLaunchKernelGGL((ksa_decode_merge_kernel<D, DEAL, 4>), outputs, dim3(4 * D), 0, st, a);
    else
        hipLaunchKernelGGL((ksa_decode_merge_kernel<D, DEAL, 1>), outputs, dim3(D), 0, st, a);
}

template <int D, int G>
void launch_group(const DecodeArgs &a, bool wide, hipStream_t st) {
    if (a.n_splits == 0)
        launch<D, G, 256, true>(a, st);   // (a million rows and more)
    else if (wide)
        launch<D, G, G == 8 ? 512 : 1024, false>(a, st);
    else
        launch<D, G, 256, false>(a, st);
}

template <int D>
int launch_all(const DecodeArgs &a, bool wide, hipStream_t st) {
    switch (a.n_q_heads / a.n_kv_heads) {
        case 1: launch_group<D, 1>(a, wide, st); break;
        case 2: launch_group<D, 2>(a, wide, st); break;
        case 4: launch_group<D, 4>(a, wide, st); break;
        case 8: launch_group<D, 8>(a, wide, st); break;
        default: return KSA_ERR_UNSUPPORTED;
    }
    return hipGetLastError() == hipSuccess ? KSA_OK : KSA_ERR_HIP;
}

}  // namespace

// The spans per sequence that the least workspace of a call without a number of its own holds records for: about 1536 workgroups, none
// with less than 768 rows.  What such a call takes is plan_decode() in ksa_api.cpp.
int ksa_decode_default_splits(const ksa_params *p) {
    const int64_t groups = (int64_t)p->batch * p->n_kv_heads;
    const int64_t rows = (int64_t)(p->n_text / p->chunk_len) * p->n_summary + (int64_t)(p->window_chunks + 1) * p->chunk_len;
    int64_t want = (1536 + groups - 1) / groups;
    const int64_t most = rows / 768 > 1 ? rows / 768 : 1;
    if (want > most) want = most;
    if (want < 1) want = 1;
    if (want > 64) want = 64;
    return (int)want;
}

// Device address of `scratch` on the current device, resolved once per device (with that device current).
int ksa_decode_static_scratch(float **ptr) {
    constexpr int MAX_DEVICES = 64;
    static void *addr[MAX_DEVICES] = {};
    static std::mutex lock;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return KSA_ERR_HIP;
    std::lock_guard<std::mutex> guard(lock);
    if (!addr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return KSA_ERR_HIP;
        addr[dev] = p;
    }
    *ptr = static_cast<float *>(addr[dev]);
    return KSA_OK;
}

int ksa_launch_decode(const KsaDecodeLaunch &L, void *stream) {
    DecodeArgs a;
    a.q = static_cast<const __bf16 *>(L.q);
    a.k = static_cast<const __bf16 *>(L.k_cache);
    a.v = static_cast<const __bf16 *>(L.v_cache);
    a.pos = L.pos;
    a.o = static_cast<__bf16 *>(L.o);
    a.lse = L.lse;
    a.ws = L.workspace;
    for (int x = 0; x < 3; ++x) a.cs[x] = L.cache_strides[x];
    a.n_splits = L.n_splits, a.n_spans = L.n_spans;
    a.s_cap = L.summary_capacity;
    a.kind = L.kind;
    a.self_only = (L.p.flags & 1u) ? 1 : 0;
    a.c = L.p.chunk_len;
    a.m = L.p.n_summary;
    a.C = L.p.window_chunks;
    a.n_text = L.p.n_text;
    a.by_c = ksa_divisor(a.c), a.by_m = ksa_divisor(std::max(a.m, 1)), a.by_slots = ksa_divisor(a.C + 1);
    a.n_q_heads = L.p.n_q_heads;
    a.n_kv_heads = L.p.n_kv_heads;
    a.scale_log2e = L.p.softmax_scale * 1.4426950408889634f;
    // with the first factor in q the products are no larger than the scaled scores and at least half as large, so that they do
    // not overflow where those would not (a scale of 1 / sqrt(128): from 2.7e39 on, unscaled products from 3.4e38)
    int exponent = 0;
    (void)std::frexp(a.scale_log2e, &exponent);
    a.q_scale = std::ldexp(1.f, std::max(std::min(exponent - 1, 0), -8)), a.score_scale = a.scale_log2e / a.q_scale;
    a.batch = L.p.batch;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (L.p.head_dim == 128) return launch_all<128>(a, L.wide, st);
    if (L.p.head_dim == 64) return launch_all<64>(a, L.wide, st);
    return KSA_ERR_UNSUPPORTED;
}

// KSA prefill backward, split dK / dV key tiles: adds up the fp32 partial sums that the pieces of a tile left behind
// (ksa_bwd_dkv_kernel, ksa_bwd_dkv_direct_kernel) in the order of the pieces and stores dK and dV.
// Bound by memory: 2 x 4096 tokens, 32/8 heads, d 128 read 19 MB of partial sums.  The records are laid out as the pieces'
// registers sit in their lanes (16 bytes per lane, 1 KiB per wavefront access), so both sides move whole lines; a
// workgroup takes one 32-column block of a tile, which gives the few split tiles enough workgroups.
#include <hip/hip_runtime.h>

#include "ksa_device.h"
#include "ksa_internal.h"

namespace {

// thread = (wave, lane) of the pieces' workgroups
template <int D>
__global__ __launch_bounds__(KSA_DKV_KEYS * 2) void ksa_bwd_dkv_sum_kernel(const KsaDkvSumArgs a) {
    const int bh = blockIdx.x % a.n_bh, hkv = bh % a.n_kv_heads, b = bh / a.n_kv_heads, db = blockIdx.y;
    const KsaDkvSplit sp = a.splits[blockIdx.x / a.n_bh];
    const bool summary = sp.tile < a.sum_tiles;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, h = lane >> 5;
    const int key = (summary ? sp.tile : sp.tile - a.sum_tiles) * KSA_DKV_KEYS + wave * 32 + (lane & 31);
    constexpr int RECORD = KSA_DKV_KEYS * D / 2;   // 16-byte pieces per record
    const f32x4 *in = reinterpret_cast<const f32x4 *>(a.scratch) + ((int64_t)sp.first_slot * a.n_bh + bh) * RECORD + wave * (D * 16) + db * 512 + lane;
    f32x4 sk[4], sv[4];
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) sk[g4] = in[g4 * 128], sv[g4] = in[g4 * 128 + 64];
    for (int x = 1; x < sp.n_slots; ++x) {
        in += (int64_t)a.n_bh * RECORD;
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
            const f32x4 xk = in[g4 * 128], xv = in[g4 * 128 + 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) sk[g4][e] += xk[e], sv[g4][e] += xv[e];
        }
    }
    if (key >= (summary ? a.n_sum : a.n_text)) return;
    const int row = summary ? key + (key / a.m + 1) * a.c : key + key / a.c * a.m;   // augmented row (Eq. 1)
    const int64_t at = b * a.strides[0] + row * a.strides[1] + hkv * a.strides[2] + db * 32 + h * 4;
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
        bf16x4 pk, pv;
#pragma unroll
        for (int e = 0; e < 4; ++e) pk[e] = (__bf16)(sk[g4][e] * a.scale), pv[e] = (__bf16)sv[g4][e];
        *reinterpret_cast<bf16x4 *>(static_cast<__bf16 *>(a.dk) + at + g4 * 8) = pk;
        *reinterpret_cast<bf16x4 *>(static_cast<__bf16 *>(a.dv) + at + g4 * 8) = pv;
    }
}

}  // namespace

void ksa_launch_dkv_sum(const KsaDkvSumArgs &a, void *stream) {
    const dim3 grid((unsigned)(a.n_splits * a.n_bh), a.head_dim / 32), block(KSA_DKV_KEYS * 2);
    if (a.head_dim == 128)
        hipLaunchKernelGGL(ksa_bwd_dkv_sum_kernel<128>, grid, block, 0, static_cast<hipStream_t>(stream), a);
    else
        hipLaunchKernelGGL(ksa_bwd_dkv_sum_kernel<64>, grid, block, 0, static_cast<hipStream_t>(stream), a);
}

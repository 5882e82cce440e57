// Device-side pieces shared by the prefill forward and backward kernels: vector types, the row maps of the
// augmented sequence and the global -> LDS load.  Header-only, included by .hip files.
#ifndef KSA_DEVICE_H_
#define KSA_DEVICE_H_

#include <hip/hip_runtime.h>

#include "ksa.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

#define LDS_PTR(T) __attribute__((address_space(3))) T *

__device__ __forceinline__ int div_by(int x, int d, int shift) { return shift >= 0 ? (x >> shift) : (x / d); }

// Augmented row (Eq. 1) of compact text index / summary ordinal idx.  Args carries c, m, w = c + m and the
// shifts c_shift, m_shift (log2 when a power of two, else -1).
template <class Args>
__device__ __forceinline__ int aug_row(const Args &a, int space, int idx) {
    if (space == KSA_SPACE_TEXT) {
        const int j = div_by(idx, a.c, a.c_shift);
        return j * a.w + (idx - j * a.c);
    }
    const int j = div_by(idx, a.m, a.m_shift);
    return j * a.w + a.c + (idx - j * a.m);
}

// global -> LDS without VGPR staging: every lane fetches 16 bytes from the wave-uniform base address plus its own unsigned byte
// offset (nothing but the load itself goes through the vector issue port), and the wave's 64 pieces land back to back (lane
// order) from the wave-uniform LDS address.
// Written as inline assembly on purpose: for the builtin the compiler assumes that any later LDS read may alias the
// data in flight and puts s_waitcnt vmcnt(0) in front of it, which serialises the loads with the MFMA work they are
// meant to overlap.  Here the waits are explicit (s_waitcnt before the workgroup barrier that publishes a tile).
// M0 carries the LDS address; no other code of these kernels uses M0.
__device__ __forceinline__ void lds_direct_load_16_s(const __bf16 *sbase, unsigned voff_bytes, unsigned lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(voff_bytes), "s"(sbase), "s"(lds_addr)
                 : "memory");
}

template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
    const int y = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, false);
    return x + __builtin_bit_cast(float, y);
}
// sum over 8 or 16 adjacent lanes (a row of head_dim 64 or 128 in 16-byte pieces); every one of them ends with the total
template <int LANES>
__device__ __forceinline__ float row_allreduce(float x) {
    x = dpp_add<0xB1>(x);    // quad_perm [1,0,3,2]
    x = dpp_add<0x4E>(x);    // quad_perm [2,3,0,1]
    x = dpp_add<0x141>(x);   // row_half_mirror: the other quad of the 8
    if (LANES == 16) x = dpp_add<0x140>(x);   // row_mirror: the other 8 of the 16
    return x;
}

// Division of an index x in [0, 2^31) by a fixed d in [1, 2^31) as one multiplication: with 2^(s-1) < d <= 2^s the
// quotient is (x * M) >> (31 + s), M = floor(2^(31 + s) / d) + 1 < 2^32 (Granlund and Montgomery: exact for x < 2^31,
// because M d exceeds 2^(31 + s) by at most d <= 2^s).
struct KsaDivisor {
    uint32_t mul, shift;
};
inline KsaDivisor ksa_divisor(int d) {
    const uint32_t s = d > 1 ? 32u - (uint32_t)__builtin_clz((unsigned)d - 1u) : 0u;
    return {(uint32_t)(((uint64_t)1 << (31 + s)) / (uint64_t)d + 1), s};
}
__device__ __forceinline__ int ksa_div(int x, const KsaDivisor &d) {
    return (int)(__umulhi((unsigned)x * 2u, d.mul) >> d.shift);
}

// Backward pass: where the log-sum-exp of row statistics slot x is kept; KSA_STAT_ROWS further the same row's delta.  32 rows of
// the one, then of the other: what a 32-row query tile needs is 256 consecutive bytes.
#define KSA_STAT_ROWS 32
template <class T>
__device__ __forceinline__ T ksa_stat_at(T x) { return x + (x & ~(T)(KSA_STAT_ROWS - 1)); }

// An LDS tile of row-major bf16 rows that is read both ways (rows as one product's operand, columns as another's): the 16-byte
// piece index is XORed with this function of the row, which spreads the 16 rows of a plain 16-byte read and the 4 rows of a
// transposing read over different banks.  At head_dim 64 two rows share the 256 bytes of all banks, so the rows of one parity
// have to differ.
template <int D>
__device__ __forceinline__ int ksa_swz(int row) { return ((D == 64 ? (row & 2) << 1 : (row & 3) << 2) | ((row >> 2) & 3)) & (D / 8 - 1); }

inline int log2_exact(int x) {
    if (x <= 0 || (x & (x - 1))) return -1;
    int s = 0;
    while ((1 << s) < x) ++s;
    return s;
}

}  // namespace

#endif

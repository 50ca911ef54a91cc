// Operand types of the matrix-core kernels, and sign planes -> bf16 weights in registers, by table.
//
// Within a scale group a row has only 2^q different weights, in pairs of opposite sign, so the 2^(q - 1) <= 8
// positive-last-plane values fit the eight bytes that v_perm_b32 selects from (low bytes and high bytes apart).  Selectors for
// four columns at a time are bits s, s + 8, s + 16, s + 24 of the planes, XNORed with the last plane, whose complement is the
// sign.  2.6 (q = 3) to 3.2 (q = 4) vector operations per weight instead of about 3 q + 0.5 for signed sums.  The table is the
// same chain of fp32 sums and one rounding as a signed sum, and negation commutes with both: the same weights bit for bit (but
// for the sign of a zero, which no sum of products keeps).
#pragma once
#include "bcq_internal.h"

namespace bcq {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;

// two fp32 -> two bf16 (round to nearest even) in one v_cvt_pk_bf16_f32; `lo` lands in the low half
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// Consecutive workgroup ids go round-robin over the 8 XCDs, each with its own L2: of `total` items every XCD takes an eighth
// in a row.
__device__ __forceinline__ bool xcd_item(uint32_t total, uint32_t& item) {
    const uint32_t xcd = blockIdx.x & 7;
    item = (uint32_t)((uint64_t)total * xcd >> 3) + (blockIdx.x >> 3);
    return item < (uint32_t)((uint64_t)total * (xcd + 1) >> 3);  // the eighths differ by one item
}
static inline unsigned xcd_grid(int64_t total) { return (unsigned)(8 * ((total + 7) / 8)); }

// The positive-last-plane weights of one row and scale group: bit i of the index = plane i is +1, i < Q - 1.
template <int Q>
struct LevelTable {
    uint32_t lo[2], hi[2];  // low and high bytes of the bf16 values, four to a word
    __device__ __forceinline__ void build(const float (&a)[Q]) {
        constexpr int E = 1 << (Q - 1);
        float v[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int cc = c < E ? c : 0;
            float s = 0.f;
#pragma unroll
            for (int i = 0; i < Q; ++i) s += (i == Q - 1 || ((cc >> i) & 1)) ? a[i] : -a[i];
            v[c] = s;
        }
        uint32_t p[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) p[c] = pack_bf16x2(v[2 * c], v[2 * c + 1]);
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            lo[w] = __builtin_amdgcn_perm(p[2 * w + 1], p[2 * w], 0x06040200u);
            hi[w] = __builtin_amdgcn_perm(p[2 * w + 1], p[2 * w], 0x07050301u);
        }
    }
};

// 32 signs of each plane -> 32 bf16 weights: frag[2 j + sub] = columns 16 j + 8 sub .. + 7 of the 32
template <int Q>
__device__ __forceinline__ void expand32(const uint32_t (&w)[Q], const LevelTable<Q>& t, u32x4 (&frag)[4]) {
    const uint32_t neg = ~w[Q - 1];
    uint32_t c[Q > 1 ? Q - 1 : 1];
#pragma unroll
    for (int i = 0; i + 1 < Q; ++i) c[i] = w[i] ^ neg;
    uint32_t even = 0u, odd = 0u;  // two-bit codes of the even and the odd columns
    if constexpr (Q >= 3) {
        even = (c[0] & 0x55555555u) | ((c[1] & 0x55555555u) << 1);
        odd = ((c[0] >> 1) & 0x55555555u) | (c[1] & 0xAAAAAAAAu);
    }
    uint32_t ab[8], cd[8];  // columns (s, s + 8) and (s + 16, s + 24)
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        uint32_t sel = 0u;
        if constexpr (Q == 2) sel = (c[0] >> s) & 0x01010101u;
        if constexpr (Q >= 3) sel = (((s & 1) ? odd : even) >> (s & 6)) & 0x03030303u;
        if constexpr (Q == 4) sel |= (s >= 2 ? c[2] >> (s - 2) : c[2] << (2 - s)) & 0x04040404u;
        const uint32_t l = __builtin_amdgcn_perm(t.lo[1], t.lo[0], sel);
        const uint32_t h = __builtin_amdgcn_perm(t.hi[1], t.hi[0], sel) ^ ((neg << (7 - s)) & 0x80808080u);
        ab[s] = __builtin_amdgcn_perm(h, l, 0x05010400u);
        cd[s] = __builtin_amdgcn_perm(h, l, 0x07030602u);
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        frag[0][p] = __builtin_amdgcn_perm(ab[2 * p + 1], ab[2 * p], 0x05040100u);
        frag[1][p] = __builtin_amdgcn_perm(ab[2 * p + 1], ab[2 * p], 0x07060302u);
        frag[2][p] = __builtin_amdgcn_perm(cd[2 * p + 1], cd[2 * p], 0x05040100u);
        frag[3][p] = __builtin_amdgcn_perm(cd[2 * p + 1], cd[2 * p], 0x07060302u);
    }
}

}  // namespace bcq

// Bit-plane pack / unpack and the transposed twin (gfx950, wave64).
// Layout: AlphaTuning Table 1 gives B the index order (q, h_out, h_in); one uint32 holds 32 consecutive
// columns, bit j = column 32w + j, 1 <=> +1.  All three kernels are pure data movement, HBM bound.
#include "bcq_internal.h"

namespace bcq {

// 4 sign bits of 4 packed int8 (bit = 1 where the byte is >= 0), byte 0 -> bit 0
__device__ __forceinline__ uint32_t nonneg_bits4(uint32_t u) {
    uint32_t m = ((~u) >> 7) & 0x01010101u;
    return (m | (m >> 7) | (m >> 14) | (m >> 21)) & 0xFu;
}

// One thread reads 16 int8 (one 16-byte load) and forms 16 bits; an even/odd lane pair forms one word.
__global__ __launch_bounds__(256) void pack_kernel(const int8_t* __restrict__ planes, int64_t total_words,
                                                   uint32_t* __restrict__ packed) {
    int64_t tid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    bool live = tid < 2 * total_words;
    uint32_t bits = 0;
    if (live) {
        uint4 v = *reinterpret_cast<const uint4*>(planes + 16 * tid);
        bits = nonneg_bits4(v.x) | (nonneg_bits4(v.y) << 4) | (nonneg_bits4(v.z) << 8) | (nonneg_bits4(v.w) << 12);
    }
    uint32_t hi = __shfl_down(bits, 1);
    if (live && !(threadIdx.x & 1)) packed[tid >> 1] = bits | (hi << 16);
}

__device__ __forceinline__ uint32_t expand4(uint32_t b) {  // 4 bits -> 4 int8 of +1 / -1
    uint32_t r = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) r |= (((b >> j) & 1u) ? 0x01u : 0xFFu) << (8 * j);
    return r;
}

__global__ __launch_bounds__(256) void unpack_kernel(const uint32_t* __restrict__ packed, int64_t total_words,
                                                     int8_t* __restrict__ planes) {
    int64_t tid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (tid >= 2 * total_words) return;
    uint32_t b = (packed[tid >> 1] >> ((tid & 1) * 16)) & 0xFFFFu;
    uint4 v;
    v.x = expand4(b);
    v.y = expand4(b >> 4);
    v.z = expand4(b >> 8);
    v.w = expand4(b >> 12);
    *reinterpret_cast<uint4*>(planes + 16 * tid) = v;
}

// In-register transpose of a 32 x 32 bit block, row r = a[r], column c = bit c (LSB = column 0):
// five rounds of swapping the off-diagonal sub-blocks of size s = 16, 8, 4, 2, 1.
__device__ __forceinline__ void transpose32(uint32_t (&a)[32]) {
#pragma unroll
    for (int s = 16; s >= 1; s >>= 1) {
        uint32_t m = 0xFFFFFFFFu / ((1u << s) + 1u);  // columns c with (c & s) == 0
#pragma unroll
        for (int r = 0; r < 32; ++r) {
            if (r & s) continue;
            uint32_t t = ((a[r] >> s) ^ a[r + s]) & m;
            a[r + s] ^= t;
            a[r] ^= t << s;
        }
    }
}

// Tile: 16 row blocks of 32 rows of W x 16 words of 32 columns.  Thread (vb, wb) transposes one 32 x 32 block read with
// lanes running along the words of a row (64-byte pieces); results pass through LDS so that the writes run along the words
// of a packed_t row.  Bound by latency: one memory trip in, some 500 ALU instructions, one trip out.  The LDS pitches (20
// words per wb, 336 per row of a block) put the 64 lanes of a write, and the 16 lanes of a 16-byte read, on 64 different
// banks; a tile of [512][17] had 16 lanes on one bank (10240 x 2560, q = 4: 12.3 us; 9.3 without the conflicts, 7.8 with
// 16-byte reads and stores as well; a copy of its 26 MB takes 4.9).  Tiles of 8 x 8 and 16 x 8 words were up to 0.3 us faster
// (1024 x 1024, q = 3: 3.3 / 3.1) or up to 5 us slower, 32 x 16 from 0.2 us faster to 0.9 slower.
// QUAD: rows of packed_t of whole 16-byte units (N % 128 == 0), four words per lane on the way out.
constexpr int TR_B = 16, TR_P2 = TR_B + 4, TR_P1 = TR_B * TR_P2 + 16;

template <bool QUAD>
__global__ __launch_bounds__(TR_B * TR_B) void transpose_kernel(const uint32_t* __restrict__ packed, int64_t N, int64_t K,
                                                                uint32_t* __restrict__ packed_t) {
    __shared__ __attribute__((aligned(16))) uint32_t tile[32 * TR_P1];
    const int64_t Kw = K / 32, Nw = N / 32;
    const int plane = blockIdx.z;
    const int wb = threadIdx.x % TR_B, vb = threadIdx.x / TR_B;
    const int64_t w = (int64_t)blockIdx.x * TR_B + wb, v = (int64_t)blockIdx.y * TR_B + vb;
    uint32_t a[32];
    const bool live = (w < Kw) && (v < Nw);
    const uint32_t* src = packed + ((int64_t)plane * N + 32 * v) * Kw + w;
#pragma unroll
    for (int r = 0; r < 32; ++r) a[r] = 0u;
    if (live) {
#pragma unroll
        for (int r = 0; r < 32; ++r) a[r] = src[(uint32_t)r * (uint32_t)Kw];
    }
    transpose32(a);
#pragma unroll
    for (int r = 0; r < 32; ++r) tile[r * TR_P1 + wb * TR_P2 + vb] = a[r];
    __syncthreads();
    // 512 output rows (columns k of W) x 16 words each, E words to a lane
    constexpr int E = QUAD ? 4 : 1, LANES = TR_B / E, ROWS = TR_B * TR_B / LANES;
    uint32_t* dst = packed_t + (int64_t)plane * K * Nw;
    const int ov = threadIdx.x % LANES * E;
    const int64_t gv = (int64_t)blockIdx.y * TR_B + ov;
#pragma unroll
    for (int pass = 0; pass < 32 * TR_B / ROWS; ++pass) {
        const int row = threadIdx.x / LANES + ROWS * pass;
        const int64_t k = (int64_t)blockIdx.x * (32 * TR_B) + row;
        if (k < K && gv < Nw) {
            const uint32_t* t = tile + row % 32 * TR_P1 + row / 32 * TR_P2 + ov;
            if (QUAD)
                *reinterpret_cast<uint4*>(dst + k * Nw + gv) = *reinterpret_cast<const uint4*>(t);
            else
                dst[k * Nw + gv] = *t;
        }
    }
}

hipError_t launch_pack(const int8_t* planes, int64_t total_words, uint32_t* packed, hipStream_t st) {
    int64_t threads = 2 * total_words;
    unsigned blocks = (unsigned)((threads + 255) / 256);
    BCQ_LAUNCH(pack_kernel, dim3(blocks), dim3(256), 0, st, planes, total_words, packed);
    return hipGetLastError();
}

hipError_t launch_unpack(const uint32_t* packed, int64_t total_words, int8_t* planes, hipStream_t st) {
    int64_t threads = 2 * total_words;
    unsigned blocks = (unsigned)((threads + 255) / 256);
    BCQ_LAUNCH(unpack_kernel, dim3(blocks), dim3(256), 0, st, packed, total_words, planes);
    return hipGetLastError();
}

hipError_t launch_pack_transposed(const uint32_t* packed, int64_t N, int64_t K, int q, uint32_t* packed_t,
                                  hipStream_t st) {
    const int64_t Kw = K / 32, Nw = N / 32;
    const dim3 grid((unsigned)((Kw + TR_B - 1) / TR_B), (unsigned)((Nw + TR_B - 1) / TR_B), (unsigned)q);
    if (Nw % 4 == 0)
        BCQ_LAUNCH((transpose_kernel<true>), grid, dim3(TR_B * TR_B), 0, st, packed, N, K, packed_t);
    else
        BCQ_LAUNCH((transpose_kernel<false>), grid, dim3(TR_B * TR_B), 0, st, packed, N, K, packed_t);
    return hipGetLastError();
}

}  // namespace bcq

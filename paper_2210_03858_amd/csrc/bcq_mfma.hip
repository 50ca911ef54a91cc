// Large-token path of the BCQ linear layer on the gfx950 matrix cores (bf16 in, fp32 accumulate).
//
// AlphaTuning Eq. 2 / Eq. 3 are one dense contraction each once the q planes of a weight are summed:
//     y  = X  * What^T   (contraction over K),      dX = dY * What   (contraction over N),
// with What[n][k] = sum_i alpha_i[n] B_i[n][k] (Eq. 1).  Summing the planes BEFORE the contraction executes
// 2 T N K matrix-core flops instead of the 2 q T N K of a plane-by-plane product.
//
// Two kernels per call:
//   1. expand_*: reads the packed sign planes and alpha and writes What (or What^T) as bf16 into the caller's
//      workspace, already in the register order of the MFMA B operand ("fragment order"): for every tile of
//      32 output columns and every 16-long slice of the contraction, 64 lanes x 8 bf16 = 1 KiB contiguous.
//      This scratch is transient per call; persistent storage stays q bits per weight.
//   2. gemm_kernel: 64 x 64 to 256 x 256 output tile per workgroup, 4 or 8 waves, v_mfma_f32_16x16x32_bf16.  Both operand
//      tiles go global -> LDS directly (buffer_load ... lds), several K-steps in flight; the activations' 16-byte chunks are
//      XOR-swizzled by row so that the fragment reads are bank-conflict free, the weights lie in LDS as in the workspace.
#include "bcq_internal.h"
#include <math.h>

#include <type_traits>

namespace bcq {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;


typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;

// two fp32 -> two bf16 (round to nearest even) in one v_cvt_pk_bf16_f32; `lo` lands in the low half
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// ---------------------------------------------------------------------------------------------------------
// Workgroup -> tile mapping.  Consecutive workgroup ids go round-robin over the 8 XCDs, each with its own L2.  The tiles
// (of all copies of the tile grid: token slices, parts of a contraction) are numbered in bands of `a` tile rows, down the
// rows first, and every XCD takes an eighth of that sequence: what it runs at one time is a block of a x (32 / a) tiles,
// so that its L2 fetches only those rows of the first operand and columns of the second, and the XCDs' shares differ
// by one tile at most (super-blocks of whole rectangles left 252 tiles in two rounds: 7000 tokens of 1696 x 1696 62 -> 34 us).
struct TileMap {
    int tiles_m, tiles_n, a, total;
};

__device__ __forceinline__ bool map_tile(const TileMap& tm, int bid, int& copy, int& tile_m, int& tile_n) {
    const int xcd = bid & 7, slot = bid >> 3;
    const int first = (int)((int64_t)tm.total * xcd >> 3), end = (int)((int64_t)tm.total * (xcd + 1) >> 3);
    if (first + slot >= end) return false;
    const int tiles = tm.tiles_m * tm.tiles_n;
    copy = (first + slot) / tiles;
    const int idx = (first + slot) % tiles;
    const int band = idx / (tm.a * tm.tiles_n), within = idx % (tm.a * tm.tiles_n);
    const int height = min(tm.a, tm.tiles_m - band * tm.a);
    tile_m = band * tm.a + within % height;
    tile_n = within / height;
    return true;
}

// The band height that brings in the fewest operand bytes for the tiles that an XCD runs at one time; cost_m and cost_n:
// bytes of a tile row and a tile column.  Returns the number of workgroups to launch.
static inline unsigned make_tile_map(int tiles_m, int tiles_n, int copies, double cost_m, double cost_n, TileMap* out) {
    const int64_t total = (int64_t)tiles_m * tiles_n * copies, share = (total + 7) / 8;
    const int cap = (int)(share < 32 ? share : 32);
    int best = 1;
    double least = 1e300;
    for (int a = 1; a <= tiles_m && a <= cap; ++a) {
        int b = (cap + a - 1) / a;
        if (b > tiles_n) b = tiles_n;
        const double cost = a * cost_m + b * cost_n;
        if (a * b * 8 >= cap * 7 && cost < least) {  // (a block that is too small to be a share says nothing)
            least = cost;
            best = a;
        }
    }
    *out = TileMap{tiles_m, tiles_n, best, (int)total};
    return (unsigned)(8 * share);
}

// ---------------------------------------------------------------------------------------------------------
// 32 fp32 sums -> 16 bf16 pairs -> four 16-byte fragment slots of 8 contraction indices each
__device__ __forceinline__ void store_word_frags(const float (&s)[32], u32x4* __restrict__ frag, int64_t block0, int c) {
#pragma unroll
    for (int gg = 0; gg < 4; ++gg) {
        u32x4 v;
#pragma unroll
        for (int p = 0; p < 4; ++p) v[p] = pack_bf16x2(s[8 * gg + 2 * p], s[8 * gg + 2 * p + 1]);
        frag[(block0 + (gg >> 1)) * 64 + c + 32 * (gg & 1)] = v;
    }
}

// expand for the forward: columns of the GEMM = rows n of W, contraction = k.
// thread = (c = n % 32, one packed word = 32 columns k) -> four 16-byte fragment slots.
__global__ __launch_bounds__(256) void expand_fwd_kernel(const uint32_t* __restrict__ packed,
                                                         const float* __restrict__ alpha, int64_t N, int64_t K,
                                                         int64_t g, int q, int64_t R16 /* padded K / 16 */,
                                                         u32x4* __restrict__ frag) {
    const int c = threadIdx.x & 31;
    const int64_t ct = blockIdx.x;
    const int64_t n = ct * 32 + c;
    const int64_t Kw = K / 32;
    const int64_t w = (int64_t)blockIdx.y * 8 + (threadIdx.x >> 5);
    if (w * 2 >= R16) return;
    const bool live = (n < N) && (w < Kw);
    const int64_t G = K / g, grp = live ? (w * 32) / g : 0;  // a packed word lies in one scale group (g % 32 == 0)
    float s[32];
#pragma unroll
    for (int e = 0; e < 32; ++e) s[e] = 0.f;
    // every plane's word and scale is requested before the first is used: one memory latency instead of one per plane
    float a[8];
    uint32_t bits[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (i < q) {
            a[i] = live ? alpha[((int64_t)i * N + n) * G + grp] : 0.f;
            bits[i] = live ? packed[((int64_t)i * N + n) * Kw + w] : 0u;
        }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (i < q) {
#pragma unroll
            for (int e = 0; e < 32; ++e) s[e] += ((bits[i] >> e) & 1u) ? a[i] : -a[i];
        }
    }
    store_word_frags(s, frag, ct * R16 + 2 * w, c);
}

// expand for the input gradient: columns of the GEMM = columns k of W, contraction = n.  Reads the transposed
// twin when the caller has one (one word = 32 consecutive n of this thread's column), else the canonical words
// (the 32 lanes of a column tile share a word and each takes its own bit).  The scales of the block's 256 rows
// pass through LDS.
// SPLIT (never with a twin): What is written as three bf16 terms hi + mid + lo (24 significant bits, all of the fp32 sum), one after the
// other along the contraction, smallest first; an Inf or NaN is its first term alone.
template <bool TWIN, bool SPLIT>
__global__ __launch_bounds__(256) void expand_bwd_kernel(const uint32_t* __restrict__ planes,
                                                         const float* __restrict__ alpha, int64_t N, int64_t K,
                                                         int64_t g, int q, int64_t R16 /* padded N / 16 */,
                                                         u32x4* __restrict__ frag) {
    __shared__ float sa[8][256];
    const int c = threadIdx.x & 31, vl = threadIdx.x >> 5;
    const int64_t ct = blockIdx.x;  // K / 32 column tiles, exactly one packed word wide
    const int64_t Kw = K / 32, Nw = N / 32;
    const int64_t n_blk = (int64_t)blockIdx.y * 256;
    const int64_t G = K / g, grp = (ct * 32) / g;  // the 32 columns of this block share one scale group
    const int64_t v = (int64_t)blockIdx.y * 8 + vl;  // word index along n
    const int64_t k = ct * 32 + c;
    // all planes' scales and, with a twin, all words of this thread are requested before the first is used
    uint32_t twin[8];
    float mine[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (i < q) {
            const int64_t n = n_blk + threadIdx.x;
            mine[i] = (n < N) ? alpha[((int64_t)i * N + n) * G + grp] : 0.f;  // rows beyond N expand to zero
            if (TWIN) twin[i] = (v < Nw) ? planes[((int64_t)i * K + k) * Nw + v] : 0u;
        }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if (i < q) sa[i][threadIdx.x] = mine[i];
    __syncthreads();
    if (v * 2 >= R16) return;
    float s[32];
#pragma unroll
    for (int e = 0; e < 32; ++e) s[e] = 0.f;
    auto add_plane = [&](int i, uint32_t bits) {
#pragma unroll
        for (int e = 0; e < 32; ++e) {
            const float a = sa[i][vl * 32 + e];
            s[e] += ((bits >> e) & 1u) ? a : -a;
        }
    };
    if (TWIN) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (i < q) add_plane(i, twin[i]);
    } else {
        for (int i = 0; i < q; ++i) {
            uint32_t bits = 0u;
#pragma unroll
            for (int e = 0; e < 32; ++e) {
                const int64_t n = v * 32 + e;
                const uint32_t wv = (n < N) ? planes[((int64_t)i * N + n) * Kw + ct] : 0u;
                bits |= ((wv >> c) & 1u) << e;
            }
            add_plane(i, bits);
        }
    }
    if (!SPLIT) {
        store_word_frags(s, frag, ct * R16 + 2 * v, c);
        return;
    }
    // A finite sum that would round beyond the largest bf16 value stops there and leaves the rest to the next terms.  Lanes
    // without any (their largest magnitude says so) take two operations per value and term.
    constexpr uint32_t BF16_LARGEST = 0x7F7F0000u;
    uint32_t top = 0u;
#pragma unroll
    for (int e = 0; e < 32; ++e) {
        const uint32_t m = __float_as_uint(s[e]) & 0x7FFFFFFFu;
        top = m > top ? m : top;
    }
    const bool ordinary = top <= BF16_LARGEST;
#pragma unroll
    for (int term = 2; term >= 0; --term) {
        float t[32];
#pragma unroll
        for (int p = 0; p < 16; ++p) {
            const uint32_t r = pack_bf16x2(s[2 * p], s[2 * p + 1]);
            t[2 * p] = __uint_as_float(r << 16);
            t[2 * p + 1] = __uint_as_float(r & 0xFFFF0000u);
        }
        if (!ordinary) {
            const float largest = __uint_as_float(BF16_LARGEST);
#pragma unroll
            for (int e = 0; e < 32; ++e) {
                const bool finite = (__float_as_uint(s[e]) & 0x7FFFFFFFu) < 0x7F800000u;
                t[e] = finite ? fminf(fmaxf(t[e], -largest), largest) : s[e];
            }
        }
        store_word_frags(t, frag, (ct * 3 + term) * R16 + 2 * v, c);
#pragma unroll
        for (int e = 0; e < 32; ++e) s[e] -= t[e];  // exact
        if (!ordinary) {
#pragma unroll
            for (int e = 0; e < 32; ++e) s[e] = (__float_as_uint(t[e]) & 0x7FFFFFFFu) < 0x7F800000u ? s[e] : 0.f;
        }
    }
}

// act[T][C] (any C) -> out[T][REP][P] with rows padded by zeros to P >= C (a multiple of 8): what the kernels below need
// of an operand whose rows are not 16-byte aligned.  REP = 3 goes with the three weight terms: non-finite values stand
// in the last copy only, the one that meets the leading term, so that an Inf meets every weight once.
template <int REP>
__global__ __launch_bounds__(256) void pad_act_kernel(const bf16_t* __restrict__ act, int64_t T, int64_t C, int64_t P,
                                                      u32x4* __restrict__ out) {
    const int64_t chunks = P / 8, idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= T * chunks) return;
    const int64_t t = idx / chunks, c = idx % chunks;
    const bf16_t* row = act + t * C;
    uint32_t h[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = 8 * c + e < C ? row[8 * c + e] : 0u;
    u32x4 v;
#pragma unroll
    for (int p = 0; p < 4; ++p) v[p] = h[2 * p] | (h[2 * p + 1] << 16);
    out[(t * REP + REP - 1) * chunks + c] = v;
    if (REP == 1) return;
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = (h[e] & 0x7F80u) == 0x7F80u ? 0u : h[e];
#pragma unroll
    for (int p = 0; p < 4; ++p) v[p] = h[2 * p] | (h[2 * p + 1] << 16);
#pragma unroll
    for (int r = 0; r < REP - 1; ++r) out[(t * REP + r) * chunks + c] = v;
}

// ---------------------------------------------------------------------------------------------------------
// C[M][NC] = A[M][R] * Bfrag, A row-major bf16 with leading dimension lda, Bfrag in fragment order with R16
// slices per column tile (R16 * 16 >= R, a multiple of 128), C row-major bf16 with leading dimension ldc.
//
// Both operand tiles go global -> LDS directly (buffer_load ... lds, 16 B per lane, no register round trip), several
// K-steps ahead, and come back as v_mfma_f32_16x16x32_bf16 operands, one 32-column slice ahead of their use.  Against weight
// fragments loaded straight into registers (one K-step ahead, twice per workgroup) this takes a third of the vector-memory
// traffic away and covers the latency of HBM; against v_mfma_f32_32x32x16_bf16 the 16 x 16 x 32 form reads and writes half
// the accumulator bits per product.  With all compute units busy the chip is at its power limit (1.7 GHz instead of 2.4),
// so that what a product costs in energy is what bounds the kernel: 6144 x 2048 at 16384 tokens 393 -> 312 us, 2048 x 8192
// 432 -> 372 us (1.32 and 1.48 PFLOP/s; weights expanded beforehand).
//
// Eight or four waves in a WM x WN grid, each TM x TN tiles of 16 x 16: two waves per vector unit hide each other's waits,
// and a wave keeps within 256 registers (accumulators in the other half of the file would be moved back and forth).  Per
// K-step one barrier: behind it every wave has the step's last fragments in registers, so the step's LDS is requested
// anew at once, and the first fragments of the next step are read under the MFMAs of the last slice.
// Nothing branches on the ragged edges: activation rows beyond M and column tiles beyond NC come back as zeros from the
// buffer range check, contraction indices beyond R meet zero weights.
//
// Tile shapes: 256 x 256 has the fewest operand bytes per product; the smaller ones fill the chip where it would leave
// compute units idle (launch_gemm).  NA, NB: stages of A and B, as many as 160 KiB hold.  KC: 64-column chunks per K-step, two
// for the smallest tiles, whose steps would otherwise be mostly barrier (about 360 cycles a step, beside BM BN / 32 of MFMA).
template <int BM, int BN> struct GemmShape;
template <> struct GemmShape<256, 256> { static constexpr int WM = 2, WN = 4, NA = 3, NB = 2, KC = 1; };
template <> struct GemmShape<256, 192> { static constexpr int WM = 2, WN = 4, NA = 3, NB = 2, KC = 1; };
template <> struct GemmShape<256, 160> { static constexpr int WM = 4, WN = 2, NA = 3, NB = 3, KC = 1; };
template <> struct GemmShape<256, 128> { static constexpr int WM = 4, WN = 2, NA = 3, NB = 3, KC = 1; };
template <> struct GemmShape<128, 160> { static constexpr int WM = 2, WN = 2, NA = 4, NB = 4, KC = 1; };
template <> struct GemmShape<128, 128> { static constexpr int WM = 2, WN = 2, NA = 5, NB = 5, KC = 1; };
template <> struct GemmShape<64, 128> { static constexpr int WM = 2, WN = 2, NA = 3, NB = 3, KC = 2; };
template <> struct GemmShape<64, 64> { static constexpr int WM = 2, WN = 2, NA = 5, NB = 5, KC = 2; };

template <int BM, int BN>
struct GemmCfg : GemmShape<BM, BN> {
    using S = GemmShape<BM, BN>;
    static constexpr int NW = S::WM * S::WN;
    static constexpr int TM = BM / S::WM / 16, TN = BN / S::WN / 16;
    static constexpr int CA = BM * 128, CB = BN * 128;             // bytes of a 64-column chunk of either operand
    static constexpr int A_B = CA * S::KC, B_B = CB * S::KC;       // bytes of a stage
    static constexpr int LDS_B = S::NA * A_B + S::NB * B_B;
    static constexpr int JA = BM / 8 / NW, JB = (BN / 8 + NW - 1) / NW;  // 1 KiB requests per wave and chunk
    static constexpr int DA = JA * S::KC, DB = JB * S::KC;               // and stage
    static_assert(BM % (16 * S::WM) == 0 && BN % (16 * S::WN) == 0 && BN % 32 == 0, "whole tiles");
    static_assert(BM % (8 * NW) == 0 && JA % 2 == 0, "the swizzle term of a row group depends on the request's index only");
    static_assert(S::NA >= S::NB && S::NA - S::NB <= 1, "the waits count on this order of requests");
    static_assert((S::NA - 1) * DA + (S::NB - 1) * DB < 64, "vmcnt");
    static_assert(LDS_B <= 160 * 1024, "LDS of a compute unit");
};

// gfx9 s_waitcnt immediate: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[5:4] at [15:14]; vmcnt alone
constexpr int wait_vm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

// sums != nullptr: the contraction is cut into parts of `per` K-steps (the tile map's copies), each workgroup stores its
// fp32 tile to sums[part][M][NC rounded up to 4].
template <int BM, int BN>
__global__ __launch_bounds__((64 * GemmCfg<BM, BN>::NW), 2) void gemm_kernel(
    const bf16_t* __restrict__ A, int64_t lda, const u32x4* __restrict__ Bfrag, bf16_t* __restrict__ C, int64_t ldc,
    int64_t M, int64_t NC, int64_t R, int64_t R16, TileMap tmap, int per, float* __restrict__ sums) {
#if defined(__HIP_DEVICE_COMPILE__)  // the buffer-resource builtins exist in the device pass only
    using Cfg = GemmCfg<BM, BN>;
    constexpr int WN = Cfg::WN, TM = Cfg::TM, TN = Cfg::TN, NA = Cfg::NA, NB = Cfg::NB, KC = Cfg::KC, SL = 2 * KC;
    constexpr int A_B = Cfg::A_B, B_B = Cfg::B_B, JA = Cfg::JA, JB = Cfg::JB, DA = Cfg::DA, DB = Cfg::DB;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: keeps descriptors and LDS bases scalar
    const int wm = wave / WN, wn = wave % WN;

    int tile_m, tile_n, part;
    if (!map_tile(tmap, blockIdx.x, part, tile_m, tile_n)) return;  // the eighths differ by one tile
    const int64_t m0 = (int64_t)tile_m * BM, n0 = (int64_t)tile_n * BN;
    const int total = (int)((R + 64 * KC - 1) / (64 * KC));  // K-steps of the whole contraction
    const int first = part * per, last = min(total, first + per) - 1;

    f32x4 acc[TN][TM];  // [weight tile][token tile]
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};

    // A: one wave instruction fills 1 KiB of LDS = 8 tile rows of 128 bytes; lane l lands in row l / 8, 16-byte slot l % 8
    // and fetches the chunk that the swizzle assigns to that slot, slot = chunk ^ (r & 7) ^ ((r >> 3) & 1), so that the
    // fragment reads (one chunk index of 16 consecutive rows) are bank-conflict free without padding.  Each wave has one
    // buffer descriptor, based at the first of its rows and ending at the end of A; rows advance through the lane offset
    // (below 2^31: lda < 2^24 and at most 64 rows), K-steps through the scalar offset.
    const int64_t wrow0 = m0 + wave * JA * 8;
    const int64_t left = (M - wrow0) * lda * 2;  // bytes from this wave's first row to the end of A (lda >= R)
    __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(A + (left > 0 ? wrow0 * lda : 0)), 0, (int)(left > 0 ? (left < 0x7fffffffll ? left : 0x7fffffffll) : 0),
        0x00020000);
    const int drow = lane >> 3, dslot = lane & 7;
    const bool ragged = (int64_t)total * 64 * KC > R;
    uint32_t avoff[JA], atail[KC][2];  // lane offsets; what the last step, which may reach beyond R, adds to them
#pragma unroll
    for (int j = 0; j < JA; ++j) avoff[j] = (uint32_t)((j * 8 + drow) * lda * 2 + (dslot ^ drow ^ (j & 1)) * 16);
#pragma unroll
    for (int c = 0; c < KC; ++c)
#pragma unroll
        for (int v = 0; v < 2; ++v) {  // chunks beyond R are clamped into the row (they meet zero weights)
            const int64_t k = (int64_t)(total - 1) * 64 * KC + c * 64 + (dslot ^ drow ^ v) * 8;
            atail[c][v] = k < R - 8 ? 0u : (uint32_t)((R - 8 - k) * 2);
        }
    auto dma_a = [&](int step, int slot, int d) {  // request d of a stage; steps beyond the last repeat it
        step = step < last ? step : last;
        const uint32_t tail = ragged && step == total - 1 ? ~0u : 0u;
        const int c = d / JA, j = d % JA;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            ra, (void __attribute__((address_space(3)))*)(smem + slot * A_B + c * Cfg::CA + (wave * JA + j) * 1024), 16,
            avoff[j] + (atail[c][j & 1] & tail), (step * KC + c) * 128, 0, 0);
    };
    // B: per column tile of 32 the four 16-slices of a chunk are 4 KiB in a row, and LDS holds them as they come.  Where a
    // wave's share is no whole number of requests the last ones are repeated.
    const int64_t ct0 = n0 / 32, ct_count = (NC + 31) / 32;
    const int64_t bleft = (ct_count - ct0) * R16 * 1024;
    __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(Bfrag + ct0 * R16 * 64), 0, (int)(bleft < 0x7fffffffll ? bleft : 0x7fffffffll), 0x00020000);
    uint32_t bvoff[JB];
    int bblk[JB];
#pragma unroll
    for (int j = 0; j < JB; ++j) {
        const int blk = wave * JB + j;
        bblk[j] = (BN / 8) % Cfg::NW == 0 ? blk : min(blk, BN / 8 - 1);
        bvoff[j] = (uint32_t)((bblk[j] >> 2) * (int)(R16 * 1024) + (bblk[j] & 3) * 1024 + lane * 16);
    }
    auto dma_b = [&](int step, int slot, int d) {
        step = step < last ? step : last;
        const int c = d / JB, j = d % JB;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rb, (void __attribute__((address_space(3)))*)(smem + NA * A_B + slot * B_B + c * Cfg::CB + bblk[j] * 1024), 16,
            bvoff[j], (step * KC + c) * 4096, 0, 0);
    };

    // Fragment reads are inline assembly: the compiler guards every LDS read it sees that may alias a direct-to-LDS
    // load with a wait for ALL outstanding loads.  `arrived` ties the fragment registers to an explicit s_waitcnt, so no
    // consumer can be scheduled above the wait.  Lane (r = lane % 16, h = lane / 16) takes columns 8 h .. + 7 of the slice.
    u32x4 xf[2][TM], wf[2][TN];  // fragments of two consecutive slices
    const int xrow = wm * 16 * TM + (lane & 15);
    const int xswz = (xrow & 7) ^ ((xrow >> 3) & 1);  // the same for rows 16 i further on
    uint32_t xoff[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) xoff[kk] = (uint32_t)(xrow * 128 + (((4 * kk + (lane >> 4)) ^ xswz) * 16));
    // column tile of 16 number c16 = half c16 & 1 of column tile c16 >> 1; with an odd TN every other wave starts at an odd one
    const int c16 = wn * TN;
    const uint32_t wlane = (uint32_t)(NA * A_B + (c16 >> 1) * 4096 + (lane >> 5) * 1024 + ((lane >> 4) & 1) * 512 + (lane & 15) * 16);
    const bool odd = (TN & 1) && (c16 & 1);
    const uint32_t woff[2] = {wlane + (odd ? 256u : 0u), wlane + (odd ? 4096u : 256u)};  // even and odd tiles of the wave
    auto read_x = [&](uint32_t stage, int kk, int i) {
        const uint32_t addr = xoff[kk & 1] + stage;
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(xf[kk & 1][i]) : "v"(addr), "n"((kk >> 1) * Cfg::CA + i * 2048));
    };
    auto read_w = [&](uint32_t stage, int kk, int j) {
        const uint32_t addr = woff[j & 1] + stage;
        asm volatile("ds_read_b128 %0, %1 offset:%2"
                     : "=v"(wf[kk & 1][j]) : "v"(addr), "n"((kk >> 1) * Cfg::CB + (j >> 1) * 4096 + (kk & 1) * 2048));
    };
    auto arrived = [&](int p) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(xf[p][i]));
#pragma unroll
        for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(wf[p][j]));
        __builtin_amdgcn_sched_barrier(0);
    };
    // The MFMAs of slice kk in boustrophedon order (neighbours share an operand), with the reads of the next slice and
    // `also` (the requests) spread between them.
    auto slice = [&](auto KK, uint32_t astage, uint32_t bstage, auto&& also) {
        constexpr int kk = decltype(KK)::value, next = (kk + 1) % SL, NM = TM * TN, NR = TM + TN;
        constexpr int GAP = NM * 3 / 4 / NR > 0 ? NM * 3 / 4 / NR : 1, PER = (NR + NM - 1) / NM;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const int j = m / TM, i = (j & 1) ? TM - 1 - m % TM : m % TM;
            acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(wf[kk & 1][j]), as_bf16x8(xf[kk & 1][i]), acc[j][i], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (m % GAP == 0) {
#pragma unroll
                for (int r = m / GAP * PER; r < m / GAP * PER + PER; ++r) {
                    if (r < TN) read_w(bstage, next, r);
                    else if (r < NR) read_x(astage, next, r - TN);
                }
            }
            also(m);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // Prologue: all stages requested in the order in which they are needed; the first one waited for.
#pragma unroll
    for (int p = 0; p < NA; ++p) {
#pragma unroll
        for (int d = 0; d < DA; ++d) dma_a(first + p, p, d);
        if (p < NB) {
#pragma unroll
            for (int d = 0; d < DB; ++d) dma_b(first + p, p, d);
        }
    }
    asm volatile("s_waitcnt %0" ::"n"(wait_vm((NA - 1) * DA + (NB - 1) * DB)) : "memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < TN; ++j) read_w(0, 0, j);
#pragma unroll
    for (int i = 0; i < TM; ++i) read_x(0, 0, i);
    __builtin_amdgcn_sched_barrier(0);

    int sa = 0, sb = 0;  // stages of step s
    for (int s = first; s <= last; ++s) {
        const int sa_next = sa + 1 == NA ? 0 : sa + 1, sb_next = sb + 1 == NB ? 0 : sb + 1;
        const uint32_t ab = (uint32_t)(sa * A_B), bb = (uint32_t)(sb * B_B);
        auto nothing = [](int) {};
        arrived(0);
        slice(std::integral_constant<int, 0>{}, ab, bb, nothing);
        if constexpr (KC == 2) {
            arrived(1);
            slice(std::integral_constant<int, 1>{}, ab, bb, nothing);
            arrived(0);
            slice(std::integral_constant<int, 2>{}, ab, bb, nothing);
        }
        arrived(1);
        // Hand-over: this wave's part of the next stage has landed (loads complete in order, only those of later stages
        // may remain), and behind the barrier everybody's has, and nobody reads this step's stage any more.
        asm volatile("s_waitcnt %0" ::"n"(wait_vm((NA - 2) * DA + (NB - 2) * DB)) : "memory");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        slice(std::integral_constant<int, SL - 1>{}, (uint32_t)(sa_next * A_B), (uint32_t)(sb_next * B_B), [&](int m) {
            constexpr int NM = TM * TN, ND = DA + DB, GAP = NM / ND > 0 ? NM / ND : 1, PER = (ND + NM - 1) / NM;
            if (m % GAP != GAP - 1) return;
#pragma unroll
            for (int d = m / GAP * PER; d < m / GAP * PER + PER; ++d) {
                if (d < DB) dma_b(s + NB, sb, d);
                else if (d < ND) dma_a(s + NA, sa, d - DB);
            }
        });
        sa = sa_next;
        sb = sb_next;
    }
    // the repeated requests of the last steps are still writing LDS, and the last fragment reads are in flight
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    arrived(0);

    // Epilogue: lane (t = lane % 16, h = lane / 16) holds columns 4 h .. + 3 of token t in every 16 x 16 tile.  Exchanging
    // odd against even rows of lanes between two neighbouring tiles leaves 8 consecutive columns in a lane, and 64
    // consecutive bytes of a token in the four lanes that share it: 16-byte stores without a trip through LDS (which
    // took 3.6 us instead of 1.9 per 256 x 256 tile).
    const int h = lane >> 4;
    if (sums) {
        const int64_t lds_ = (NC + 3) / 4 * 4;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int64_t t = m0 + (wm * TM + i) * 16 + (lane & 15);
            float* row = sums + ((int64_t)part * M + t) * lds_;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int64_t n = n0 + (wn * TN + j) * 16 + 4 * h;
                if (t < M && n < NC) *reinterpret_cast<f32x4*>(row + n) = acc[j][i];
            }
        }
        return;
    }
    const bool vec_ok = (ldc % 8 == 0);
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int64_t t = m0 + (wm * TM + i) * 16 + (lane & 15);
        bf16_t* crow = C + t * ldc;
        const int64_t nw = n0 + wn * TN * 16;
        if (vec_ok) {
#pragma unroll
            for (int j = 0; j + 1 < TN; j += 2) {
                const uint32_t a0 = pack_bf16x2(acc[j][i][0], acc[j][i][1]), a1 = pack_bf16x2(acc[j][i][2], acc[j][i][3]);
                const uint32_t b0 = pack_bf16x2(acc[j + 1][i][0], acc[j + 1][i][1]);
                const uint32_t b1 = pack_bf16x2(acc[j + 1][i][2], acc[j + 1][i][3]);
                const auto s0 = __builtin_amdgcn_permlane16_swap(a0, b0, false, false);
                const auto s1 = __builtin_amdgcn_permlane16_swap(a1, b1, false, false);
                const u32x4 v = {s0[0], s1[0], s0[1], s1[1]};
                const int64_t n = nw + (j + (h & 1)) * 16 + (h >> 1) * 8;
                if (t < M && n < NC) *reinterpret_cast<u32x4*>(crow + n) = v;  // NC % 8 == 0 where ldc is (ldc = NC)
            }
            if (TN & 1) {
                const int64_t n = nw + (TN - 1) * 16 + 4 * h;
                const f32x4 a = acc[TN - 1][i];
                if (t < M && n < NC) *reinterpret_cast<uint2*>(crow + n) = make_uint2(pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]));
            }
        } else if (t < M) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int64_t n = nw + j * 16 + 4 * h + e;
                    if (n < NC) crow[n] = f32_to_bf16(acc[j][i][e]);
                }
        }
    }
#endif
}

static inline int64_t round_up(int64_t a, int64_t b) { return (a + b - 1) / b * b; }

constexpr int RPAD = 128;  // contraction padding of the expanded operand: the longest K-step of any tile configuration
size_t mfma_fwd_workspace(int64_t N, int64_t K) { return (size_t)(round_up(N, 32) * round_up(K, RPAD) * 2); }
size_t mfma_bwd_input_workspace(int64_t N, int64_t K) { return (size_t)(round_up(K, 32) * round_up(N, RPAD) * 2); }

template <int BM, int BN>
static hipError_t launch_gemm_cfg(const bf16_t* A, int64_t lda, const u32x4* frag, bf16_t* C, int64_t ldc, int64_t M,
                                  int64_t NC, int64_t R, int64_t R16, hipStream_t st) {
    using Cfg = GemmCfg<BM, BN>;
    static LdsLimit limit;
    hipError_t e = limit.ensure((const void*)gemm_kernel<BM, BN>, Cfg::LDS_B);
    if (e != hipSuccess) return e;
    TileMap tmap;
    const unsigned wgs = make_tile_map((int)((M + BM - 1) / BM), (int)((NC + BN - 1) / BN), 1, (double)BM, (double)BN, &tmap);
    const int steps = (int)((R + 64 * Cfg::KC - 1) / (64 * Cfg::KC));
    BCQ_LAUNCH((gemm_kernel<BM, BN>), dim3(wgs), dim3(64 * Cfg::NW), Cfg::LDS_B, st, A, lda, frag, C, ldc, M, NC, R, R16,
                       tmap, steps, (float*)nullptr);
    return hipGetLastError();
}

// Tile choice: the least estimated time over the rounds of workgroups on 256 compute units (one resident on each).  A K-step
// of 64 takes 0.0115 ns per product and 1.11 ns per row and column of the tile (a little less when fewer compute units
// share power and caches: the share of them that works to the power 0.22), at least the 362 ns of its barrier and waits; a
// round costs another 2.6 us to start and 5 us per 256 x 256 outputs to store.  Fitted to 333 products of 64 to 16384 tokens
// with 768 to 10240 rows and columns, every shape timed: the pick is the fastest or within 3 % of it for 328 of them,
// within 7 % for all (256 x 256 tiles against the pick: 1280 x 5120 at 4096 tokens 87 / 47 us, 3072 x 1024 29 / 27).
static double gemm_estimate(int bm, int bn, int kc, int64_t M, int64_t NC, int64_t R) {
    const double tiles = (double)((M + bm - 1) / bm) * (double)((NC + bn - 1) / bn), steps = (double)((R + 63) / 64);
    const double full = 0.01153 * bm * bn + 1.112 * (bm + bn), least = 362.0 / kc;
    const double fixed = 2600.0 + 4955.0 * bm * bn / 65536.0;
    const double rounds = (double)(int64_t)(tiles / 256), busy = (tiles - 256 * rounds) / 256;
    double t = rounds * (steps * (full > least ? full : least) + fixed);
    if (busy > 0) {
        const double part = full * pow(busy, 0.22);
        t += steps * (part > least ? part : least) + fixed;
    }
    return t;
}

static hipError_t launch_gemm(const bf16_t* A, int64_t lda, const u32x4* frag, bf16_t* C, int64_t ldc, int64_t M,
                              int64_t NC, int64_t R, int64_t R16, hipStream_t st) {
    static constexpr int shapes[][3] = {{256, 256, 1}, {256, 192, 1}, {256, 160, 1}, {256, 128, 1},
                                        {128, 160, 1}, {128, 128, 1}, {64, 128, 2}, {64, 64, 2}};
    int best = 0;
    double least = 1e300;
    for (int i = 0; i < 8; ++i) {
        const double t = gemm_estimate(shapes[i][0], shapes[i][1], shapes[i][2], M, NC, R);
        if (t < least) {
            least = t;
            best = i;
        }
    }
    switch (best) {
        case 0: return launch_gemm_cfg<256, 256>(A, lda, frag, C, ldc, M, NC, R, R16, st);
        case 1: return launch_gemm_cfg<256, 192>(A, lda, frag, C, ldc, M, NC, R, R16, st);
        case 2: return launch_gemm_cfg<256, 160>(A, lda, frag, C, ldc, M, NC, R, R16, st);
        case 3: return launch_gemm_cfg<256, 128>(A, lda, frag, C, ldc, M, NC, R, R16, st);
        case 4: return launch_gemm_cfg<128, 160>(A, lda, frag, C, ldc, M, NC, R, R16, st);
        case 5: return launch_gemm_cfg<128, 128>(A, lda, frag, C, ldc, M, NC, R, R16, st);
        case 6: return launch_gemm_cfg<64, 128>(A, lda, frag, C, ldc, M, NC, R, R16, st);
        default: return launch_gemm_cfg<64, 64>(A, lda, frag, C, ldc, M, NC, R, R16, st);
    }
}

hipError_t launch_fwd_mfma(const uint32_t* packed, const float* alpha, const void* x, int64_t T, int64_t N,
                           int64_t K, int64_t g, int q, void* y, void* workspace, hipStream_t st) {
    const int64_t R16 = round_up(K, RPAD) / 16;
    const int64_t ct = (N + 31) / 32;
    dim3 grid((unsigned)ct, (unsigned)((R16 / 2 + 7) / 8));
    BCQ_LAUNCH(expand_fwd_kernel, grid, dim3(256), 0, st, packed, alpha, N, K, g, q, R16, (u32x4*)workspace);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_gemm((const bf16_t*)x, K, (const u32x4*)workspace, (bf16_t*)y, N, T, N, K, R16, st);
}

static dim3 expand_bwd_grid(int64_t K, int64_t R16) { return dim3((unsigned)(K / 32), (unsigned)((R16 / 2 + 7) / 8)); }

hipError_t launch_bwd_input_mfma(const uint32_t* packed, const uint32_t* packed_t, const float* alpha, const void* dy,
                                 int64_t T, int64_t N, int64_t K, int64_t g, int q, void* dx, void* workspace,
                                 hipStream_t st) {
    const int64_t R16 = round_up(N, RPAD) / 16;
    u32x4* frag = (u32x4*)workspace;
    if (packed_t && N % 32 == 0)
        BCQ_LAUNCH((expand_bwd_kernel<true, false>), expand_bwd_grid(K, R16), dim3(256), 0, st, packed_t, alpha, N, K, g, q,
                           R16, frag);
    else
        BCQ_LAUNCH((expand_bwd_kernel<false, false>), expand_bwd_grid(K, R16), dim3(256), 0, st, packed, alpha, N, K, g, q,
                           R16, frag);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_gemm((const bf16_t*)dy, N, frag, (bf16_t*)dx, K, T, K, N, R16, st);
}

// Input gradient with fp32 weights for row counts that launch_bwd_input_mfma does not take and that have no twin (N % 32 != 0):
// dX = [dY dY dY] [lo; mid; hi], the same contraction three times as long, on the same kernel.  Tokens are taken SPLIT_TOKENS
// at a time, which bounds the copies (50257 rows: 1.2 GB) and still fills the chip.
constexpr int64_t SPLIT_TOKENS = 4096;
size_t mfma_bwd_input_split_workspace(int64_t T, int64_t N, int64_t K) {
    return (size_t)(3 * round_up(N, RPAD) * 2 * ((T < SPLIT_TOKENS ? T : SPLIT_TOKENS) + round_up(K, 32)));
}

hipError_t launch_bwd_input_mfma_split(const uint32_t* packed, const float* alpha, const void* dy, int64_t T, int64_t N, int64_t K, int64_t g, int q, void* dx,
                                       void* workspace, hipStream_t st) {
    const int64_t P = round_up(N, RPAD), R16 = P / 16;
    u32x4* frag = (u32x4*)workspace;
    u32x4* rows = frag + round_up(K, 32) * 3 * P / 8;
    BCQ_LAUNCH((expand_bwd_kernel<false, true>), expand_bwd_grid(K, R16), dim3(256), 0, st, packed, alpha, N, K, g, q, R16, frag);
    hipError_t e = hipGetLastError();
    for (int64_t t0 = 0; t0 < T && e == hipSuccess; t0 += SPLIT_TOKENS) {
        const int64_t M = T - t0 < SPLIT_TOKENS ? T - t0 : SPLIT_TOKENS;
        BCQ_LAUNCH((pad_act_kernel<3>), dim3((unsigned)((M * (P / 8) + 255) / 256)), dim3(256), 0, st,
                           (const bf16_t*)dy + t0 * N, M, N, P, rows);
        e = hipGetLastError();
        if (e == hipSuccess)
            e = launch_gemm((const bf16_t*)rows, 3 * P, frag, (bf16_t*)dx + t0 * K, K, M, K, 3 * P, 3 * R16, st);
    }
    return e;
}


// =========================================================================================================
// Scale gradient on the matrix cores.  AlphaTuning Eq. 4, read as the gradient of Eq. 2, is
//     dalpha_i[n] = s * sum_t dY[t][n] * (X B_i^T)[t][n] = s * sum_k B_i[n][k] * G[n][k],   G = dY^T X.
// G is one dense contraction over the tokens (2 T N K matrix-core flops for ALL planes together, instead of
// 2 q T N K for q plane products); the sign planes only enter a signed row sum of the accumulators.
//
// Both MFMA operands need the token index innermost, which neither activation has in memory.  LDS fragment
// reads are the scarce resource of a compute unit (a 16-byte-per-lane read instruction takes ~16 clocks), so
// only ONE operand may pass through LDS:
//   1. transpose_frag_kernel rewrites the smaller activation (x if K <= N, else dy) into MFMA fragment order
//      with the token index innermost (8 x 8 register transposes); its fragments are then loaded straight
//      from global memory, 1 KiB coalesced per wave load, exactly like the expanded weights of the forward.
//   2. dalpha_kernel: 256 (k) x 256 (n) tile of G^T for one slice of the tokens; 4 waves in a 2 x 2 grid, each
//      128 x 128 = 4 x 4 tiles of v_mfma_f32_32x32x16_bf16 with X^T as first and dY^T as second operand, so a
//      lane holds one n and 16 k of every tile.  The other activation goes global -> registers -> 8 x 8
//      transpose (32 v_perm) -> XOR-swizzled LDS tile [column][64 tokens]; writes and fragment reads are
//      bank-conflict free.  The epilogue forms the signed sums over k for every trained plane.
//   3. dalpha_reduce_kernel adds the partial sums of all (token slice, k tile) pairs in a fixed order (no
//      floating-point atomics, bit-reproducible).
constexpr int DA_TILE = 256;               // k and n extent of a workgroup tile
constexpr int DA_STAGE = DA_TILE * 128;    // bytes per LDS stage: 256 columns x 64 tokens x 2 B

__device__ __forceinline__ int da_swz(int col, int chunk) { return col * 128 + ((chunk ^ (col & 7) ^ ((col >> 3) & 7)) << 4); }

// 8 x 8 transpose of 16-bit elements: in[r] holds row r (8 elements), out[c] holds column c.
__device__ __forceinline__ void transpose8x8(const u32x4 (&in)[8], u32x4 (&out)[8]) {
#pragma unroll
    for (int c = 0; c < 8; ++c)
#pragma unroll
        for (int w = 0; w < 4; ++w)
            out[c][w] = __builtin_amdgcn_perm(in[2 * w + 1][c >> 1], in[2 * w][c >> 1], (c & 1) ? 0x07060302u : 0x05040100u);
}

// act[T][C] (row-major bf16) -> fragments with the token index innermost: for column tile ct (32 columns) and
// token slice ks (16 tokens) one 1 KiB block; lane (c % 32) + 32 g holds tokens 16 ks + 8 g .. + 7 of column c.
// Tokens >= T (up to T16 * 16) and columns >= C are written as zeros.
__global__ __launch_bounds__(256) void transpose_frag_kernel(const bf16_t* __restrict__ act, int64_t T, int64_t C,
                                                             int64_t T16, u32x4* __restrict__ frag) {
    const int cb = threadIdx.x & 15, tbl = threadIdx.x >> 4;       // 16 column blocks x 16 token blocks per group
    const int64_t c0 = ((int64_t)blockIdx.x * 16 + cb) * 8;       // first of 8 columns
    const int64_t tb = (int64_t)blockIdx.y * 16 + tbl;            // block of 8 tokens
    if (tb * 8 >= T16 * 16) return;
    u32x4 in[8], out[8];
    const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int64_t t = tb * 8 + r;
        in[r] = (t < T && c0 < C) ? *reinterpret_cast<const u32x4*>(act + t * C + c0) : zero;
    }
    transpose8x8(in, out);
    const int64_t ct = c0 / 32, ks = tb >> 1;
    const int g = (int)(tb & 1);
    if (ct * 32 >= ((C + 31) / 32) * 32) return;
#pragma unroll
    for (int c = 0; c < 8; ++c) frag[(ct * T16 + ks) * 64 + (c0 % 32) + c + 32 * g] = out[c];
}

// XG: x comes as fragments from global memory and dy through LDS; otherwise the reverse.
// QT: planes summed in the epilogue (q_train rounded up to 1, 2, 3, 4 or 8; extra planes are computed, not stored).
// FINE: partial sums are kept per 32 columns k (for scale groups that are not whole 256-column tiles) instead of
//       per tile; they go to part[split][plane][n][8 tiles_k] and dalpha_reduce_fine_kernel adds each group's run.
template <bool XG, int QT, bool FINE>
__global__ __launch_bounds__(256, 1) void dalpha_kernel(const bf16_t* __restrict__ L /* activation through LDS */,
                                                        int64_t ldl, int64_t lcols,
                                                        const u32x4* __restrict__ Gfrag, int64_t T16,
                                                        const uint32_t* __restrict__ packed,
                                                        float* __restrict__ part, int64_t T, int64_t N, int64_t K,
                                                        int q_train, TileMap tmap, int splits,
                                                        int64_t tokens_per_split) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;  // wm: k half, wn: n half
    const int tiles_k = tmap.tiles_m;
    int split, tile_k, tile_n;
    if (!map_tile(tmap, blockIdx.x, split, tile_k, tile_n)) return;
    const int64_t k0 = (int64_t)tile_k * DA_TILE, n0 = (int64_t)tile_n * DA_TILE;
    const int64_t t_begin = (int64_t)split * tokens_per_split;  // a multiple of 64
    const int64_t t_end = (t_begin + tokens_per_split < T) ? t_begin + tokens_per_split : T;
    const int64_t steps = (t_end - t_begin + 63) / 64;
    const int64_t step0 = t_begin / 64;

    f32x16 acc[4][4];  // [k tile][n tile]
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // LDS-side activation: thread = (cb = column block of 8, tb = token block of 8)
    const int cb = tid & 31, tb = tid >> 5;
    int64_t lcol = (XG ? n0 : k0) + cb * 8;
    lcol = lcol < lcols - 8 ? lcol : lcols - 8;  // clamped columns only feed outputs that are never stored
    u32x4 lr[8];
    // rows of one step: uniform base (advances by 64 rows per step) + 32-bit lane offset + r rows
    const uint32_t row_b = (uint32_t)(ldl * 2);
    const uint32_t voff0 = (uint32_t)(tb * 8) * row_b + (uint32_t)(lcol * 2);
    auto load_blocks = [&](int64_t step) {
        const int64_t t0 = (step0 + step) * 64;
        const unsigned char* base = reinterpret_cast<const unsigned char*>(L + t0 * ldl);
        if (t0 + 64 <= T) {
#pragma unroll
            for (int r = 0; r < 8; ++r) lr[r] = *reinterpret_cast<const u32x4*>(base + (voff0 + (uint32_t)r * row_b));
        } else {  // last, ragged step: rows beyond T are clamped (they meet zero fragments of the other operand)
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                int64_t t = t0 + tb * 8 + r;
                t = t < T ? t : T - 1;
                lr[r] = *reinterpret_cast<const u32x4*>(L + t * ldl + lcol);
            }
        }
    };
    // column c of this thread's 8 x 8 block: 8 tokens of one column = one 16-byte LDS chunk (4 v_perm + 1 write)
    auto store_col = [&](int buf, int c) {
        u32x4 o;
#pragma unroll
        for (int w = 0; w < 4; ++w)
            o[w] = __builtin_amdgcn_perm(lr[2 * w + 1][c >> 1], lr[2 * w][c >> 1], (c & 1) ? 0x07060302u : 0x05040100u);
        *reinterpret_cast<u32x4*>(smem + buf * DA_STAGE + da_swz(cb * 8 + c, tb)) = o;
    };
    auto store_blocks = [&](int buf) {
#pragma unroll
        for (int c = 0; c < 8; ++c) store_col(buf, c);
    };
    bf16x8 lf[2][4];
    const int lbase = (XG ? wn : wm) * 128 + (lane & 31);
    auto read_frags = [&](int buf, int kk) {
        const unsigned char* sl = smem + buf * DA_STAGE;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            lf[kk & 1][i] = *reinterpret_cast<const bf16x8*>(sl + da_swz(lbase + i * 32, kk * 2 + (lane >> 5)));
    };
    // global-side fragments of this wave: 4 column tiles
    const int64_t gct_count = ((XG ? K : N) + 31) / 32;
    const int64_t gct0 = ((XG ? k0 + wm * 128 : n0 + wn * 128)) / 32;
    const u32x4* gptr[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        int64_t ct = gct0 + j;
        ct = ct < gct_count ? ct : gct_count - 1;
        gptr[j] = Gfrag + (ct * T16 + step0 * 4) * 64 + lane;
    }
    u32x4 g[4][4];  // [kk][tile]
    auto load_g = [&](int kk, int64_t step) {
#pragma unroll
        for (int j = 0; j < 4; ++j) g[kk][j] = gptr[j][(step * 4 + kk) * 64];
    };
    auto mfma_one = [&](int kk, int i, int j) {
        if (XG)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(g[kk][i]), lf[kk & 1][j], acc[i][j], 0, 0, 0);
        else
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lf[kk & 1][i], as_bf16x8(g[kk][j]), acc[i][j], 0, 0, 0);
    };
    auto mfma_slice = [&](int kk) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) mfma_one(kk, i, j);
    };

    // Three LDS stages.  The blocks of step s + 1 are requested during step s - 1, transposed and written into
    // their stage during the FIRST slice of step s, interleaved with its MFMAs (a stage is free from the barrier
    // that ends the step after its last read), and read from the barrier that ends step s: the global latency
    // has a whole step of cover and neither the transposes nor the LDS writes wait in front of a barrier.
    const int64_t last = steps - 1;
    load_blocks(0);
    load_g(0, 0);
    store_blocks(0);
    load_blocks(last < 1 ? last : 1);  // followed by three slices of fragment loads, as in every step of the loop
#pragma unroll
    for (int kk = 1; kk < 4; ++kk) load_g(kk, 0);
    __syncthreads();
    read_frags(0, 0);
    int stg = 0;  // stage of step s
    for (int64_t s = 0; s < steps; ++s) {
        const int64_t nx = s < last ? s + 1 : last;
        const int64_t nx2 = s + 2 < steps ? s + 2 : last;
        const int stg_next = (stg == 2) ? 0 : stg + 1;
        read_frags(stg, 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < 8; ++c) {  // two MFMAs (64 clocks of the matrix pipe) cover one column's perms and write
            mfma_one(0, c >> 1, 2 * (c & 1));
            mfma_one(0, c >> 1, 2 * (c & 1) + 1);
            store_col(stg_next, c);
            __builtin_amdgcn_sched_barrier(0);
        }
        load_g(0, nx);
        load_blocks(nx2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kk = 1; kk < 3; ++kk) {
            read_frags(stg, kk + 1);
            mfma_slice(kk);
            load_g(kk, nx);
            __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 16, 0);
            __builtin_amdgcn_sched_group_barrier(0x020, 4, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        read_frags(stg_next, 0);
        __builtin_amdgcn_sched_barrier(0);
        mfma_slice(3);
        load_g(3, nx);
        __builtin_amdgcn_sched_group_barrier(0x008, 16, 0);
        __builtin_amdgcn_sched_group_barrier(0x020, 4, 0);
        __builtin_amdgcn_sched_barrier(0);
        stg = stg_next;
    }
    __syncthreads();

    // epilogue: signed sums over this wave's 128 k for each plane; lane owns n = n_base + j*32 + lane%32.
    // All packed words of all trained planes are requested first (one memory latency instead of one per plane);
    // a sign is applied as a factor +-1.0 built from the (inverted) plane bit: shift, and-or, fused multiply-add
    // per value (the product with +-1.0 is exact, so this equals adding the signed value).
    float* red = reinterpret_cast<float*>(smem);  // [plane][wm][256 n]
    const int64_t Kw = K / 32;
    uint32_t words[QT][4][4];  // [plane][k tile][n tile], already inverted and shifted to this lane's rows
    const int64_t kt0 = (k0 + wm * 128) / 32;                      // first of this wave's four k tiles
    const bool quad = (kt0 + 3 < Kw) && ((Kw & 3) == 0);           // one aligned 16-byte load per row and plane
#pragma unroll
    for (int p = 0; p < QT; ++p) {
        const int pc = p < q_train ? p : q_train - 1;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int64_t n = n0 + wn * 128 + j * 32 + (lane & 31);
            const int64_t nc = n < N ? n : N - 1;
            const uint32_t* prow = packed + ((int64_t)pc * N + nc) * Kw;
            u32x4 w4;
            if (quad) {
                w4 = *reinterpret_cast<const u32x4*>(prow + kt0);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int64_t kt = kt0 + i < Kw ? kt0 + i : Kw - 1;  // tiles beyond K hold zero accumulators
                    w4[i] = prow[kt];
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) words[p][i][j] = ~(w4[i] >> (4 * (lane >> 5)));
        }
    }
    if (FINE) {
        // one signed sum per (plane, 32-column k tile, n): red[plane][chunk = 4 wm + i][256 n]
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float fs[QT][4];
#pragma unroll
            for (int p = 0; p < QT; ++p)
#pragma unroll
                for (int j = 0; j < 4; ++j) fs[p][j] = 0.f;
            if ((k0 + wm * 128 + i * 32) < K) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int bit = 8 * (v >> 2) + (v & 3);
                        const float a = acc[i][j][v];
#pragma unroll
                        for (int p = 0; p < QT; ++p)
                            fs[p][j] = __builtin_fmaf(a, __uint_as_float(((words[p][i][j] << (31 - bit)) & 0x80000000u) | 0x3f800000u), fs[p][j]);
                    }
            }
#pragma unroll
            for (int p = 0; p < QT; ++p)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    float s = fs[p][j];
                    s += __shfl_xor(s, 32);
                    if (lane < 32) red[(p * 8 + wm * 4 + i) * 256 + wn * 128 + j * 32 + lane] = s;
                }
        }
        __syncthreads();
        const int64_t n = n0 + tid;
        const int64_t Kc = (int64_t)tiles_k * 8;
        if (n < N) {
            for (int p = 0; p < q_train; ++p) {
                float* dst = part + (((int64_t)split * q_train + p) * N + n) * Kc + (int64_t)tile_k * 8;
                u32x4 lo, hi;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    lo[c] = __float_as_uint(red[(p * 8 + c) * 256 + tid]);
                    hi[c] = __float_as_uint(red[(p * 8 + 4 + c) * 256 + tid]);
                }
                *reinterpret_cast<u32x4*>(dst) = lo;
                *reinterpret_cast<u32x4*>(dst + 4) = hi;
            }
        }
        return;
    }
    // every accumulator is read once and added, with its sign, into the sums of all planes
    float sums[QT][4];  // [plane][n tile]
#pragma unroll
    for (int p = 0; p < QT; ++p)
#pragma unroll
        for (int j = 0; j < 4; ++j) sums[p][j] = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if ((k0 + wm * 128 + i * 32) < K) {  // uniform: tiles beyond K hold nothing
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int bit = 8 * (v >> 2) + (v & 3);
                    const float a = acc[i][j][v];
#pragma unroll
                    for (int p = 0; p < QT; ++p)  // sign bit set where the plane bit is 0 (-1): words are inverted
                        sums[p][j] = __builtin_fmaf(a, __uint_as_float(((words[p][i][j] << (31 - bit)) & 0x80000000u) | 0x3f800000u), sums[p][j]);
                }
        }
    }
#pragma unroll
    for (int p = 0; p < QT; ++p)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float s = sums[p][j];
            s += __shfl_xor(s, 32);
            if (lane < 32) red[(p * 2 + wm) * 256 + wn * 128 + j * 32 + lane] = s;
        }
    __syncthreads();
    const int64_t part_id = (int64_t)split * tiles_k + tile_k;
    for (int p = 0; p < q_train; ++p) {
        const int64_t n = n0 + tid;
        if (n < N) part[(part_id * q_train + p) * N + n] = red[(p * 2 + 0) * 256 + tid] + red[(p * 2 + 1) * 256 + tid];
    }
}

// dalpha[pn][grp] = scale * sum over token slices and over the k tiles of group grp of part[slice][tile][pn],
// pn = plane * N + n; `tpg` consecutive k tiles form one scale group (row-wise: all of them, G = 1).
// A workgroup owns 64 consecutive outputs; its four waves each add a quarter of the partial sums (every fourth one,
// eight loads in flight) and wave 0 adds the four quarters in wave order: a fixed order, bit-reproducible.
__global__ __launch_bounds__(256) void dalpha_reduce_kernel(const float* __restrict__ part, float* __restrict__ dalpha,
                                                            int64_t rows /* q_train * N */, int64_t G, int splits,
                                                            int tiles_k, int tpg, float scale, AdamWArgs opt) {
    __shared__ float quarter[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t idx = (int64_t)blockIdx.x * 64 + lane;
    const bool live = idx < rows * G;
    const int64_t pn = live ? idx / G : 0, grp = live ? idx % G : 0;
    const int items = splits * tpg;  // item it = (slice it / tpg, tile it % tpg of the group)
    float s = 0.f;
    int it = wave;
    for (; it + 28 < items; it += 32) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int iu = it + 4 * u;
            v[u] = part[((int64_t)(iu / tpg) * tiles_k + grp * tpg + iu % tpg) * rows + pn];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; it < items; it += 4) s += part[((int64_t)(it / tpg) * tiles_k + grp * tpg + it % tpg) * rows + pn];
    quarter[wave][lane] = s;
    __syncthreads();
    if (wave != 0 || !live) return;
    const float total = scale * ((quarter[0][lane] + quarter[1][lane]) + (quarter[2][lane] + quarter[3][lane]));
    dalpha[idx] = total;
    if (opt.alpha) adamw_apply(opt, idx, total);
}

// Fine partials part[slice][pn][Kc] (one value per 32 columns): a group is a run of cpg consecutive values.
// Same split of the work as above: item it = (slice it / cpg, value it % cpg of the run).
__global__ __launch_bounds__(256) void dalpha_reduce_fine_kernel(const float* __restrict__ part,
                                                                 float* __restrict__ dalpha, int64_t rows, int64_t G,
                                                                 int splits, int64_t Kc, int cpg, float scale,
                                                                 AdamWArgs opt) {
    __shared__ float quarter[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t idx = (int64_t)blockIdx.x * 64 + lane;
    const bool live = idx < rows * G;
    const int64_t pn = live ? idx / G : 0, grp = live ? idx % G : 0;
    const int items = splits * cpg;
    float s = 0.f;
    for (int it = wave; it < items; it += 4)
        s += part[((int64_t)(it / cpg) * rows + pn) * Kc + grp * cpg + it % cpg];
    quarter[wave][lane] = s;
    __syncthreads();
    if (wave != 0 || !live) return;
    const float total = scale * ((quarter[0][lane] + quarter[1][lane]) + (quarter[2][lane] + quarter[3][lane]));
    dalpha[idx] = total;
    if (opt.alpha) adamw_apply(opt, idx, total);
}

struct DalphaPlan {
    int tiles_k, tiles_n, splits;
    int64_t per_split, T16;
    bool xg, fine;
    size_t frag_bytes, part_bytes;
};

static DalphaPlan dalpha_plan(int64_t T, int64_t N, int64_t K, int64_t g, int q) {
    DalphaPlan pl;
    pl.tiles_k = (int)((K + DA_TILE - 1) / DA_TILE);
    pl.tiles_n = (int)((N + DA_TILE - 1) / DA_TILE);
    const int64_t tiles = (int64_t)pl.tiles_k * pl.tiles_n;
    int64_t s = tiles >= 256 ? 1 : 256 / tiles;       // one round of workgroups on the 256 compute units
    const int64_t max_s = (T + 255) / 256;            // at least 256 tokens (4 steps) per slice
    if (s > max_s) s = max_s;
    if (s < 1) s = 1;
    pl.per_split = ((T + s - 1) / s + 63) / 64 * 64;
    pl.splits = (int)((T + pl.per_split - 1) / pl.per_split);
    pl.T16 = (T + 63) / 64 * 4;
    pl.xg = (K <= N);
    const int64_t gcols = pl.xg ? K : N;
    pl.frag_bytes = (size_t)(((gcols + 31) / 32) * pl.T16 * 1024);
    pl.fine = (g != K) && (g % DA_TILE != 0);  // groups that are not whole k tiles need per-32-column partials
    pl.part_bytes = (size_t)pl.splits * pl.tiles_k * q * N * sizeof(float) * (pl.fine ? 8 : 1);
    return pl;
}

// Rows of dy that are not 16-byte aligned are copied into padded ones, this many tokens at a time (a multiple of 64): the
// copy stays below 512 MiB (50257 rows: 5312 tokens), and the partial sums of all pieces are added at the end.
static int64_t dalpha_piece(int64_t T, int64_t N) {
    if (N % 8 == 0) return T;
    int64_t piece = ((int64_t)1 << 29) / (2 * round_up(N, 8)) / 64 * 64;
    if (piece > ((int64_t)1 << 20)) piece = (int64_t)1 << 20;
    return T < piece ? T : piece;
}

struct DalphaScratch {
    size_t frag, part, pad;  // bytes: fragments of a piece, partial sums of all pieces, padded copy of a piece
    int splits;              // token slices of all pieces
};
static DalphaScratch dalpha_scratch(int64_t T, int64_t N, int64_t K, int64_t g, int q) {
    const int64_t piece = dalpha_piece(T, N), whole = T / piece, rest = T % piece;
    const DalphaPlan a = dalpha_plan(piece, N, K, g, q);
    DalphaScratch s = {a.frag_bytes, (size_t)whole * a.part_bytes, 0, (int)whole * a.splits};
    if (rest) {
        const DalphaPlan b = dalpha_plan(rest, N, K, g, q);
        s.part += b.part_bytes;
        s.splits += b.splits;
    }
    if (N % 8) {
        s.part = (s.part + 15) / 16 * 16;
        s.pad = (size_t)(piece * round_up(N, 8) * 2);
    }
    return s;
}

size_t mfma_bwd_alpha_workspace(int64_t T, int64_t N, int64_t K, int64_t g, int q) {
    const DalphaScratch s = dalpha_scratch(T, N, K, g, q);
    return s.frag + s.part + s.pad;
}

// Partial sums of T tokens into `part`: transposition of one activation, then the product
static hipError_t launch_dalpha_piece(const uint32_t* packed, const bf16_t* x, const bf16_t* dy, int64_t dcols, int64_t T,
                                      int64_t N, int64_t K, int q_train, const DalphaPlan& pl, u32x4* frag, float* part,
                                      hipStream_t st) {
    const int lds = 3 * DA_STAGE;
    const bf16_t* gact = pl.xg ? x : dy;
    const bf16_t* lact = pl.xg ? dy : x;
    const int64_t gcols = pl.xg ? K : dcols, lcols = pl.xg ? dcols : K;
    {
        dim3 grid((unsigned)((gcols + 127) / 128), (unsigned)((pl.T16 * 2 + 15) / 16));
        BCQ_LAUNCH(transpose_frag_kernel, grid, dim3(256), 0, st, gact, T, gcols, pl.T16, frag);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    TileMap tmap;
    const unsigned wgs = make_tile_map(pl.tiles_k, pl.tiles_n, pl.splits, 1.0, 1.0, &tmap);
    dim3 grid(wgs);
    const int qt = q_train <= 4 ? q_train : 8;
#define BCQ_DA_LAUNCH(XGV, QTV, FV)                                                                                   \
    {                                                                                                                 \
        static LdsLimit limit;                                                                                        \
        hipError_t ea = limit.ensure((const void*)dalpha_kernel<XGV, QTV, FV>, (size_t)lds);                           \
        if (ea != hipSuccess) return ea;                                                                              \
        BCQ_LAUNCH((dalpha_kernel<XGV, QTV, FV>), grid, dim3(256), lds, st, lact, lcols, lcols, frag, pl.T16,  \
                           packed, part, T, N, K, q_train, tmap, pl.splits, pl.per_split);                            \
    }
#define BCQ_DA_Q(XGV, FV)                                  \
    switch (qt) {                                          \
        case 1: BCQ_DA_LAUNCH(XGV, 1, FV) break;           \
        case 2: BCQ_DA_LAUNCH(XGV, 2, FV) break;           \
        case 3: BCQ_DA_LAUNCH(XGV, 3, FV) break;           \
        case 4: BCQ_DA_LAUNCH(XGV, 4, FV) break;           \
        default: BCQ_DA_LAUNCH(XGV, 8, FV) break;          \
    }
    if (pl.fine) {
        if (pl.xg) {
            BCQ_DA_Q(true, true)
        } else {
            BCQ_DA_Q(false, true)
        }
    } else {
        if (pl.xg) {
            BCQ_DA_Q(true, false)
        } else {
            BCQ_DA_Q(false, false)
        }
    }
#undef BCQ_DA_Q
#undef BCQ_DA_LAUNCH
    return hipGetLastError();
}

hipError_t launch_bwd_alpha_mfma(const uint32_t* packed, const void* x, const void* dy, int64_t T, int64_t N,
                                 int64_t K, int64_t g, int q, int q_train, float grad_scale, float* dalpha,
                                 void* workspace, const AdamWArgs* opt, hipStream_t st) {
    const DalphaScratch sc = dalpha_scratch(T, N, K, g, q);
    const int64_t piece = dalpha_piece(T, N), dcols = sc.pad ? round_up(N, 8) : N;
    unsigned char* ws = static_cast<unsigned char*>(workspace);
    u32x4* frag = reinterpret_cast<u32x4*>(ws);
    float* part = reinterpret_cast<float*>(ws + sc.frag);
    float* next = part;
    DalphaPlan pl;
    for (int64_t t0 = 0; t0 < T; t0 += piece) {
        const int64_t M = T - t0 < piece ? T - t0 : piece;
        pl = dalpha_plan(M, N, K, g, q);
        const bf16_t* rows = (const bf16_t*)dy + t0 * N;
        if (sc.pad) {
            u32x4* padded = reinterpret_cast<u32x4*>(ws + sc.frag + sc.part);
            BCQ_LAUNCH((pad_act_kernel<1>), dim3((unsigned)((M * (dcols / 8) + 255) / 256)), dim3(256), 0, st, rows, M, N,
                               dcols, padded);
            hipError_t ep = hipGetLastError();
            if (ep != hipSuccess) return ep;
            rows = reinterpret_cast<const bf16_t*>(padded);
        }
        hipError_t ep = launch_dalpha_piece(packed, (const bf16_t*)x + t0 * K, rows, dcols, M, N, K, q_train, pl, frag, next, st);
        if (ep != hipSuccess) return ep;
        next += (int64_t)pl.splits * pl.tiles_k * q_train * N * (pl.fine ? 8 : 1);
    }
    const int64_t rows = (int64_t)q_train * N, G = K / g;
    const dim3 rgrid((unsigned)((rows * G + 63) / 64));
    AdamWArgs oa = {};
    if (opt) oa = *opt;
    if (pl.fine)
        BCQ_LAUNCH(dalpha_reduce_fine_kernel, rgrid, dim3(256), 0, st, (const float*)part, dalpha, rows, G,
                           sc.splits, (int64_t)pl.tiles_k * 8, (int)(g / 32), grad_scale, oa);
    else
        BCQ_LAUNCH(dalpha_reduce_kernel, rgrid, dim3(256), 0, st, (const float*)part, dalpha, rows, G,
                           sc.splits, pl.tiles_k, (int)(g == K ? pl.tiles_k : g / DA_TILE), grad_scale, oa);
    return hipGetLastError();
}

}  // namespace bcq

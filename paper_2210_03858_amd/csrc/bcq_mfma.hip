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
#include <math.h>

#include <type_traits>

#include "bcq_expand.h"

namespace bcq {

// ---------------------------------------------------------------------------------------------------------
// Workgroup -> tile mapping.  The tiles (of all copies of the tile grid, one per token slice) are numbered in
// bands of `a` tile rows, down the rows first, and every XCD takes an eighth of that sequence: what it runs at one time is a
// block of a x (32 / a) tiles, so that its L2 fetches only those rows of the first operand and columns of the second, and the
// XCDs' shares differ by one tile at most (super-blocks of whole rectangles left 252 tiles in two rounds: 7000 tokens of 1696 x 1696 62 -> 34 us).
struct TileMap {
    int tiles_m, tiles_n, a, total;
};

__device__ __forceinline__ bool map_tile(const TileMap& tm, int& copy, int& tile_m, int& tile_n) {
    uint32_t item;
    if (!xcd_item((uint32_t)tm.total, item)) return false;
    const int tiles = tm.tiles_m * tm.tiles_n;
    copy = (int)item / tiles;
    const int idx = (int)item % tiles;
    const int band = idx / (tm.a * tm.tiles_n), within = idx % (tm.a * tm.tiles_n);
    const int height = min(tm.a, tm.tiles_m - band * tm.a);
    tile_m = band * tm.a + within % height;
    tile_n = within / height;
    return true;
}

// The band height that brings in the fewest operand bytes for the tiles that an XCD runs at one time; cost_m and cost_n:
// bytes of a tile row and a tile column.  Up to `whole` times those bytes the band is all rows: an XCD then has an eighth of
// the columns to itself.  Returns the number of workgroups to launch.
static inline unsigned make_tile_map(int tiles_m, int tiles_n, int copies, double cost_m, double cost_n, double whole, TileMap* out) {
    const int64_t total = (int64_t)tiles_m * tiles_n * copies, share = (total + 7) / 8;
    const int cap = (int)(share < 32 ? share : 32);
    int best = 1;
    double least = 1e300;
    for (int a = 1; a <= tiles_m && a <= cap; ++a) {
        int b = (cap + a - 1) / a;
        if (b > tiles_n) b = tiles_n;
        const double cost = a * cost_m + b * cost_n;
        if (a * b * 8 >= cap * 7 && (cost < least || (a == tiles_m && cost <= whole * least))) {  // (a block that is too small to be a share says nothing)
            least = cost;
            best = a;
        }
    }
    *out = TileMap{tiles_m, tiles_n, best, (int)total};
    return xcd_grid(total);
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

// `columns`: in the product an XCD has an eighth of the column tiles to itself (make_tile_map), and the expansion's blocks on
// that XCD write them: a fragment that another XCD holds in its L2 from the call before costs its next writer a trip there.
// With one workspace kept from call to call (expansion and product, us, plain order / this one): 3072 x 1024, 550 tokens,
// q = 1 17 / 12, input gradient of 2048 x 8192 at 65 tokens 33 / 18, of 6144 x 2048 at 86 40 / 29; workspaces in turn, where no
// XCD holds them, 12.2 / 12.1, 18 / 18, 28 / 29.

// The scales of a layer in training lie in two tensors (ScaleParts), and its backward pass wants them in one: blocks beyond those of
// the forward's expansion write that (a concatenation before the expansion was a launch of 4 to 6 us).
__device__ __forceinline__ void join_scales(const ScaleParts& a, int64_t per_plane, int q, uint32_t chunk) {
    const int64_t split = a.q_first * per_plane, total = q * per_plane;
    const int64_t idx0 = (int64_t)chunk * 2048 + threadIdx.x;
    float v[8];  // all requested before the first is stored: one trip to memory
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int64_t idx = idx0 + e * 256;
        if (idx < total) v[e] = idx < split ? a.first[idx] : a.rest[idx - split];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (idx0 + e * 256 < total) a.joined[idx0 + e * 256] = v[e];
}

__global__ __launch_bounds__(256) void join_scales_kernel(ScaleParts a, int64_t per_plane, int q) {
    join_scales(a, per_plane, q, blockIdx.x);
}

hipError_t launch_join_scales(const ScaleParts& a, int64_t per_plane, int q, hipStream_t st) {
    BCQ_LAUNCH(join_scales_kernel, dim3((unsigned)((q * per_plane + 2047) / 2048)), dim3(256), 0, st, a, per_plane, q);
    return hipGetLastError();
}

// expand for the forward: columns of the GEMM = rows n of W, contraction = k.
// thread = (one row n, one packed word = 32 columns k) -> four 16-byte fragment slots; block = 8 rows x 32 words, so that it
// reads whole 128-byte lines and stores whole 128-byte pieces (32 rows x 8 words, the lines shared by four blocks: 13.4 us
// instead of 12.1).  Q planes by table up to four, else (Q = 0) q of them as signed sums.  What bounds it is the 16 bits per
// weight that it writes (5.4 TB/s with its reads); by signed sums four planes were bound by vector operations.  Measured:
// 10240 x 2560, q = 4 17.7 -> 12.5 us, 2560 x 10240 17.5 -> 11.8, 8192 x 2048, q = 3 10.8 -> 8.4, 4096 x 1024 5.6 -> 5.2.
template <int Q>
__global__ __launch_bounds__(256) void expand_fwd_kernel(const uint32_t* __restrict__ packed, ScaleParts alpha, uint32_t blocks,
                                                         int64_t N, int64_t K, int64_t g, int q,
                                                         int64_t R16 /* padded K / 16 */, int columns,
                                                         u32x4* __restrict__ frag) {
    if (blockIdx.x >= blocks) {
        join_scales(alpha, N * (K / g), q, (blockIdx.x - blocks) * gridDim.y + blockIdx.y);
        return;
    }
    uint32_t block = blockIdx.x, run = blockIdx.y;  // plain: 8 rows x a run of 32 words (the divisions cost 0.4 us of 5)
    if (columns) {
        const uint32_t runs = (uint32_t)((R16 / 2 + 31) / 32);
        uint32_t item;
        if (!xcd_item((uint32_t)((N + 31) / 32) * runs * 4, item)) return;
        run = (item >> 2) % runs;
        block = (item >> 2) / runs * 4 + (item & 3);
    }
    const int c = (threadIdx.x & 7) + 8 * (block & 3);
    const int64_t ct = block >> 2;
    const int64_t n = ct * 32 + c;
    const int64_t Kw = K / 32;
    const int64_t w = (int64_t)run * 32 + (threadIdx.x >> 3);
    if (w * 2 >= R16) return;
    const bool live = (n < N) && (w < Kw);
    const int64_t G = K / g, grp = live ? (w * 32) / g : 0;  // a packed word lies in one scale group (g % 32 == 0)
    // every plane's word and scale is requested before the first is used: one memory latency instead of one per plane
    constexpr int P = Q ? Q : 8;
    float a[P];
    uint32_t bits[P];
#pragma unroll
    for (int i = 0; i < P; ++i) {
        if (Q || i < q) {
            const float* scales = i < alpha.q_first ? alpha.first + i * N * G : alpha.rest + (i - alpha.q_first) * N * G;
            a[i] = live ? scales[n * G + grp] : 0.f;
            bits[i] = live ? packed[((int64_t)i * N + n) * Kw + w] : 0u;
        }
    }
    if constexpr (Q > 0) {
        LevelTable<Q> table;
        table.build(a);
        u32x4 out[4];
        expand32<Q>(bits, table, out);
#pragma unroll
        for (int gg = 0; gg < 4; ++gg) frag[(ct * R16 + 2 * w + (gg >> 1)) * 64 + c + 32 * (gg & 1)] = out[gg];
    } else {
        float s[32];
#pragma unroll
        for (int e = 0; e < 32; ++e) s[e] = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i < q) {
#pragma unroll
                for (int e = 0; e < 32; ++e) s[e] += ((bits[i] >> e) & 1u) ? a[i] : -a[i];
            }
        }
        store_word_frags(s, frag, ct * R16 + 2 * w, c);
    }
}

// dalpha[pn][grp] = scale * sum over token slices and over the k tiles of group grp of part[slice][tile][pn],
// pn = plane * N + n; `run` consecutive k tiles form one scale group (row-wise: all of them, G = 1).  Fine: partials
// part[slice][pn][per_slice] (one value per 32 columns), a group is a run of `run` consecutive values.
// A workgroup owns 64 consecutive outputs; its four waves each add a quarter of the partial sums (every fourth one,
// eight loads in flight) and wave 0 adds the four quarters in wave order: a fixed order, bit-reproducible.
struct DalphaSums {
    const float* part;
    float* dalpha;
    int64_t rows /* q_train * N */, G, per_slice /* k tiles, or 32-column values */;
    int splits, run;
    float scale;
    bool fine;
    AdamWArgs opt;
};
__device__ __forceinline__ void dalpha_reduce(const DalphaSums& a, uint32_t block, float (*quarter)[64]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, run = a.run;
    const int64_t idx = (int64_t)block * 64 + lane;
    const bool live = idx < a.rows * a.G;
    const int64_t pn = live ? idx / a.G : 0, grp = live ? idx % a.G : 0;
    const int items = a.splits * run;  // item it = (slice it / run, value it % run of the group)
    float s = 0.f;
    int it = wave;
    if (a.fine) {
        for (; it < items; it += 4) s += a.part[((int64_t)(it / run) * a.rows + pn) * a.per_slice + grp * run + it % run];
    } else {
        for (; it + 28 < items; it += 32) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int iu = it + 4 * u;
                v[u] = a.part[((int64_t)(iu / run) * a.per_slice + grp * run + iu % run) * a.rows + pn];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; it < items; it += 4) s += a.part[((int64_t)(it / run) * a.per_slice + grp * run + it % run) * a.rows + pn];
    }
    quarter[wave][lane] = s;
    __syncthreads();
    if (wave != 0 || !live) return;
    const float total = a.scale * ((quarter[0][lane] + quarter[1][lane]) + (quarter[2][lane] + quarter[3][lane]));
    a.dalpha[idx] = total;
    if (a.opt.alpha) adamw_apply(a.opt, idx, total);
}

__global__ __launch_bounds__(256) void dalpha_reduce_kernel(DalphaSums a) {
    __shared__ float quarter[4][64];
    dalpha_reduce(a, blockIdx.x, quarter);
}
static unsigned dalpha_reduce_blocks(const DalphaSums& a) { return (unsigned)((a.rows * a.G + 63) / 64); }

// The same for the input gradient (columns of the GEMM = columns k, contraction = n), up to four planes: a thread expands 32
// columns of one row n with that row's table, the tile of 32 rows x 256 columns goes through LDS, and ds_read_b64_tr_b16
// returns it with the rows innermost.  (With the bits running along n, as in the twin, every weight of a word has scales of
// its own: signed sums, 12.5 operations per weight.  10240 x 2560, q = 4: 18.1 -> 11.8 us, 8192 x 2048, q = 3 11.2 -> 8.0,
// 4096 x 1024 6.8 -> 6.4.)
// Blocks from `blocks` on reduce the scale gradient of the same backward pass, whose partial sums the launch before left:
// that is 4 to 5 us of two dependent trips to memory by a few workgroups, in a launch of its own or hidden in this one.
template <int Q>
__global__ __launch_bounds__(256) void expand_bwd_rows_kernel(const uint32_t* __restrict__ packed,
                                                              const float* __restrict__ alpha, int64_t N, int64_t K,
                                                              int64_t g, int64_t R16 /* padded N / 16 */, int columns,
                                                              u32x4* __restrict__ frag, uint32_t blocks, DalphaSums sums) {
    __shared__ __attribute__((aligned(16))) unsigned char tile[32 * 512];  // rows of 256 columns, in 32-byte pieces c ^ swz(row)
    if (blockIdx.x >= blocks) {
        dalpha_reduce(sums, blockIdx.x - blocks, reinterpret_cast<float(*)[64]>(tile));
        return;
    }
    const int r = threadIdx.x >> 3, wl = threadIdx.x & 7;
    const int64_t Kw = K / 32, G = K / g;
    const uint32_t row_tiles = (uint32_t)(R16 / 2);
    uint32_t item = blockIdx.x;
    const uint32_t items = row_tiles * (uint32_t)((Kw + 7) / 8);
    if (columns ? !xcd_item(items, item) : item >= items) return;
    const int64_t rt = item % row_tiles, wg = item / row_tiles;
    const int64_t n = rt * 32 + r, w = wg * 8 + wl;
    const bool live = n < N && w < Kw;
    float a[Q];
    uint32_t bits[Q];
    const int64_t grp = live ? (w * 32) / g : 0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        a[i] = live ? alpha[((int64_t)i * N + n) * G + grp] : 0.f;  // rows beyond N expand to zero
        bits[i] = live ? packed[((int64_t)i * N + n) * Kw + w] : 0u;
    }
    LevelTable<Q> table;
    table.build(a);
    u32x4 out[4];
    expand32<Q>(bits, table, out);
    auto swz = [](int row) { return (row & 3) | (((row >> 3) & 1) << 2); };
#pragma unroll
    for (int f = 0; f < 4; ++f)
        *reinterpret_cast<u32x4*>(tile + r * 512 + (((2 * wl + (f >> 1)) ^ swz(r)) * 32) + (f & 1) * 16) = out[f];
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int piece = (lane >> 4) & 1, grow = 8 * (lane >> 5) + ((lane >> 2) & 3);
#pragma unroll
    for (int j = 0; j < 4; ++j) {  // column tile 2 wave + (j >> 1) of 32, slice j & 1 of 16 rows
        const int ctl = 2 * wave + (j >> 1), row = 16 * (j & 1) + grow;
        const uint32_t addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)tile +
                              (uint32_t)(row * 512 + (((2 * ctl + piece) ^ swz(row)) * 32) + (lane & 3) * 8);
        u32x2 lo, hi;
        asm volatile("ds_read_b64_tr_b16 %0, %2\n\tds_read_b64_tr_b16 %1, %2 offset:2048\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(lo), "=&v"(hi) : "v"(addr) : "memory");
        const int64_t ct = wg * 8 + ctl, ks = rt * 2 + (j & 1);
        if (ct < Kw && ks < R16) frag[(ct * R16 + ks) * 64 + lane] = u32x4{lo[0], lo[1], hi[0], hi[1]};
    }
}

// expand for the input gradient by signed sums, from five planes on and for three terms.  Reads the transposed twin when the
// caller has one (one word = 32 consecutive n of this thread's column), else the canonical words (the 32 lanes of a column
// tile share a word and each takes its own bit).  The scales of the block's 256 rows pass through LDS.
// SPLIT (never with a twin): What is written as three bf16 terms hi + mid + lo (24 significant bits, all of the fp32 sum), one after the
// other along the contraction, smallest first; an Inf or NaN is its first term alone.
template <bool TWIN, bool SPLIT>
__global__ __launch_bounds__(256) void expand_bwd_kernel(const uint32_t* __restrict__ planes,
                                                         const float* __restrict__ alpha, int64_t N, int64_t K,
                                                         int64_t g, int q, int64_t R16 /* padded N / 16 */, int columns,
                                                         u32x4* __restrict__ frag) {
    __shared__ float sa[8][256];
    const int c = threadIdx.x & 31, vl = threadIdx.x >> 5;
    // the K / 32 column tiles (exactly one packed word wide), or the XCD's eighth of them, side by side: neighbours share the
    // lines of scales and canonical words (one tile after the other 7680 x 2560, q = 8, g = 64 105 -> 190 us)
    const int64_t Kw = K / 32, Nw = N / 32;
    const uint32_t first = columns ? (uint32_t)(Kw * (blockIdx.x & 7) >> 3) : 0u;
    const uint32_t width = columns ? (uint32_t)(Kw * ((blockIdx.x & 7) + 1) >> 3) - first : (uint32_t)Kw;
    const uint32_t slot = columns ? blockIdx.x >> 3 : blockIdx.x;
    if (width == 0 || slot >= width * (uint32_t)((R16 / 2 + 7) / 8)) return;
    const int64_t ct = first + slot % width;
    const int64_t n_blk = (int64_t)(slot / width) * 256;
    const int64_t G = K / g, grp = (ct * 32) / g;  // the 32 columns of this block share one scale group
    const int64_t v = n_blk / 32 + vl;  // word index along n
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
// the accumulator bits per product.  With all compute units busy the clock falls (1.9 GHz on average at 16384 tokens, 2.5 to
// 2.7 where tiles are few), so that what a product costs in energy counts as much as its cycles: 6144 x 2048 at 16384 tokens
// 393 -> 312 us, 2048 x 8192 432 -> 372 us (1.32 and 1.48 PFLOP/s; weights expanded beforehand).  The matrix cores work in 75 %
// of the busy cycles there; of the LDS cycles 40 % are bank conflicts.
//
// Eight or four waves in a WM x WN grid, each TM x TN tiles of 16 x 16: with eight, two waves per vector unit hide each other's
// waits (the four-wave shapes' LDS admits one workgroup too, so that there one wave stands alone), and a wave keeps within 256
// registers (accumulators in the other half of the file would be moved back and forth).  Per
// K-step one barrier: behind it every wave has the step's last fragments in registers, so the step's LDS is requested
// anew at once, and the first fragments of the next step are read under the MFMAs of the last slice.
// Nothing branches on the ragged edges: activation rows beyond M, their columns beyond R and column tiles beyond NC come back
// as zeros from the buffer range check (zeros and no other finite or infinite value: an Inf times the zero weights there is NaN).
//
// Tile shapes: 256 x 256 has the fewest operand bytes per product; the smaller ones fill the chip where it would leave
// compute units idle (gemm_plan).  NA, NB: stages of A and B, as many as 160 KiB hold, but three of 64 x 64 (two
// more only hold up the first step, whose data the prologue's requests share the way with: 1024 x 1024 at 1024 tokens, expansion and product 10.4 -> 9.6 us, input
// gradient of 4096 x 1024 at 309 21.0 -> 20.4, forward of 384 x 2688 at 1232 14.7 -> 14.0).  KC: 64-column chunks per K-step, two
// for the smallest tiles, whose steps would otherwise be mostly barrier (about 360 cycles a step, beside BM BN / 32 of MFMA).
template <int BM, int BN> struct GemmShape;
template <> struct GemmShape<256, 256> { static constexpr int WM = 2, WN = 4, NA = 3, NB = 2, KC = 1; };
template <> struct GemmShape<256, 192> { static constexpr int WM = 2, WN = 4, NA = 3, NB = 2, KC = 1; };
template <> struct GemmShape<256, 160> { static constexpr int WM = 4, WN = 2, NA = 3, NB = 3, KC = 1; };
template <> struct GemmShape<256, 128> { static constexpr int WM = 4, WN = 2, NA = 3, NB = 3, KC = 1; };
template <> struct GemmShape<128, 160> { static constexpr int WM = 2, WN = 2, NA = 4, NB = 4, KC = 1; };
template <> struct GemmShape<128, 128> { static constexpr int WM = 2, WN = 2, NA = 5, NB = 5, KC = 1; };
template <> struct GemmShape<64, 128> { static constexpr int WM = 2, WN = 2, NA = 3, NB = 3, KC = 2; };
template <> struct GemmShape<64, 64> { static constexpr int WM = 2, WN = 2, NA = 3, NB = 3, KC = 2; };

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

template <int BM, int BN>
__global__ __launch_bounds__((64 * GemmCfg<BM, BN>::NW), 2) void gemm_kernel(
    const bf16_t* __restrict__ A, int64_t lda, const u32x4* __restrict__ Bfrag, bf16_t* __restrict__ C, int64_t ldc,
    int64_t M, int64_t NC, int64_t R, int64_t R16, TileMap tmap) {
#if defined(__HIP_DEVICE_COMPILE__)  // the buffer-resource builtins exist in the device pass only
    using Cfg = GemmCfg<BM, BN>;
    constexpr int WN = Cfg::WN, TM = Cfg::TM, TN = Cfg::TN, NA = Cfg::NA, NB = Cfg::NB, KC = Cfg::KC, SL = 2 * KC;
    constexpr int A_B = Cfg::A_B, B_B = Cfg::B_B, JA = Cfg::JA, JB = Cfg::JB, DA = Cfg::DA, DB = Cfg::DB;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: keeps descriptors and LDS bases scalar
    const int wm = wave / WN, wn = wave % WN;

    int tile_m, tile_n, only;
    if (!map_tile(tmap, only, tile_m, tile_n)) return;
    const int64_t m0 = (int64_t)tile_m * BM, n0 = (int64_t)tile_n * BN;
    const int last = (int)((R + 64 * KC - 1) / (64 * KC)) - 1;  // K-step

    f32x4 acc[TN][TM];  // [weight tile][token tile]
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};

    // A: one wave instruction fills 1 KiB of LDS = 8 tile rows of 128 bytes; lane l lands in row l / 8, 16-byte slot l % 8
    // and fetches the chunk that the swizzle assigns to that slot, slot = chunk ^ (r & 7) ^ ((r >> 3) & 1), so that one
    // chunk index of 16 consecutive rows touches every bank once without padding.  Each wave has one
    // buffer descriptor, based at the first of its rows and ending at the end of A; rows advance through the lane offset
    // (below 2^31: lda < 2^24 and at most 64 rows), K-steps through the scalar offset.
    const int64_t wrow0 = m0 + wave * JA * 8;
    const int64_t left = (M - wrow0) * lda * 2;  // bytes from this wave's first row to the end of A (lda >= R)
    __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(A + (left > 0 ? wrow0 * lda : 0)), 0, (int)(left > 0 ? (left < 0x7fffffffll ? left : 0x7fffffffll) : 0),
        0x00020000);
    const int drow = lane >> 3, dslot = lane & 7;
    const bool ragged = (int64_t)(last + 1) * 64 * KC > R;
    uint32_t avoff[JA], atail[KC][2];  // lane offsets; what the last step, which may reach beyond R, adds to them
#pragma unroll
    for (int j = 0; j < JA; ++j) avoff[j] = (uint32_t)((j * 8 + drow) * lda * 2 + (dslot ^ drow ^ (j & 1)) * 16);
#pragma unroll
    for (int c = 0; c < KC; ++c)
#pragma unroll
        for (int v = 0; v < 2; ++v) {  // chunks beyond R are sent beyond every descriptor: zeros, as the weights they meet
            const int64_t k = (int64_t)last * 64 * KC + c * 64 + (dslot ^ drow ^ v) * 8;
            atail[c][v] = k < R ? 0u : 0x80000000u;
        }
    auto dma_a = [&](int step, int slot, int d) {  // request d of a stage; steps beyond the last repeat it
        step = step < last ? step : last;
        const uint32_t tail = ragged && step == last ? ~0u : 0u;
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
        for (int d = 0; d < DA; ++d) dma_a(p, p, d);
        if (p < NB) {
#pragma unroll
            for (int d = 0; d < DB; ++d) dma_b(p, p, d);
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
    for (int s = 0; s <= last; ++s) {
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

struct GemmPlan {
    int shape;
    unsigned wgs;
    TileMap map;
    bool columns() const { return map.a == map.tiles_m; }  // an XCD has an eighth of the column tiles to itself
};

template <int BM, int BN>
static hipError_t launch_gemm_cfg(const GemmPlan& pl, const bf16_t* A, int64_t lda, const u32x4* frag, bf16_t* C, int64_t ldc, int64_t M,
                                  int64_t NC, int64_t R, int64_t R16, hipStream_t st) {
    using Cfg = GemmCfg<BM, BN>;
    static LdsLimit limit;
    hipError_t e = limit.ensure((const void*)gemm_kernel<BM, BN>, Cfg::LDS_B);
    if (e != hipSuccess) return e;
    BCQ_LAUNCH((gemm_kernel<BM, BN>), dim3(pl.wgs), dim3(64 * Cfg::NW), Cfg::LDS_B, st, A, lda, frag, C, ldc, M, NC, R, R16,
                       pl.map);
    return hipGetLastError();
}

// Tile choice: the least estimated time over the rounds of workgroups on 256 compute units (one resident on each).  A K-step
// of 64 takes 0.0115 ns per product and 1.11 ns per row and column of the tile (a little less when fewer compute units
// share power and caches: the share of them that works to the power 0.22), at least the 362 ns of its barrier and waits; a
// round costs another 2.6 us to start and 5 us per 256 x 256 outputs to store.  Fitted to 333 products of 64 to 16384 tokens
// with 768 to 10240 rows and columns, every shape timed: the pick is the fastest or within 3 % of it for 328 of them,
// within 7 % for all (256 x 256 tiles against the pick: 1280 x 5120 at 4096 tokens 87 / 47 us, 3072 x 1024 29 / 27).
struct ShareTable {  // (k / 256) ^ e
    double v[256];
    explicit ShareTable(double e) {
        for (int k = 0; k < 256; ++k) v[k] = pow(k / 256.0, e);
    }
};
static double round_estimate(double full, double least, const ShareTable& share, int64_t tiles, int64_t steps, double fixed) {
    double t = (double)(tiles / 256) * ((double)steps * (full > least ? full : least) + fixed);
    if (tiles % 256) {
        const double part = full * share.v[tiles % 256];
        t += (double)steps * (part > least ? part : least) + fixed;
    }
    return t;
}
static double gemm_estimate(int bm, int bn, int kc, int64_t M, int64_t NC, int64_t R) {
    static const ShareTable share(0.22);
    return round_estimate(0.01153 * bm * bn + 1.112 * (bm + bn), 362.0 / kc, share, ((M + bm - 1) / bm) * ((NC + bn - 1) / bn),
                          (R + 63) / 64, 2600.0 + 4955.0 * bm * bn / 65536.0);
}

static GemmPlan gemm_plan(int64_t M, int64_t NC, int64_t R, double* estimate = nullptr) {
    static constexpr int shapes[][3] = {{256, 256, 1}, {256, 192, 1}, {256, 160, 1}, {256, 128, 1},
                                        {128, 160, 1}, {128, 128, 1}, {64, 128, 2}, {64, 64, 2}};
    GemmPlan pl = {};
    double least = 1e300;
    for (int i = 0; i < 8; ++i) {
        const double t = gemm_estimate(shapes[i][0], shapes[i][1], shapes[i][2], M, NC, R);
        if (t < least) {
            least = t;
            pl.shape = i;
        }
    }
    if (estimate) *estimate = least;
    const int bm = shapes[pl.shape][0], bn = shapes[pl.shape][1];
    // Bands of all rows: up to 2048 tokens always that an XCD's share has room for them (1024 x 1024, 786 tokens, with 1.36 times
    // the operand bytes, kept workspace 11.1 -> 9.2 us, in turn 9.4 / 9.3), up to 3072 for up to 3.5 million weights with more
    // columns than contraction (forward of 3072 x 1024, 2600 tokens, 1.54 times, kept 28.6 -> 25.0, in turn 24.5 / 24.3).  Beyond that
    // they still save 1 to 4 us with a kept workspace, but cost as much with workspaces in turn, as in training (input gradient of
    // 2016 x 2016, 2477 tokens, kept 33.9 -> 31.1, in turn 29.8 -> 31.1; forward of 1024 x 3072, 2600 tokens, 30.4 -> 29.3, 27.2 ->
    // 29.1; input gradient of 7680 x 2560, 2300 tokens, 92.9 -> 96.3, 92.3 -> 93.7; 3840 x 1280, 4096 tokens, 44.3 -> 41.4, 39.3 -> 40.1).
    const double whole = M <= 2048 || (M <= 3072 && NC * R <= 3500000 && NC > R) ? 2.5 : 1.4;
    pl.wgs = make_tile_map((int)((M + bm - 1) / bm), (int)((NC + bn - 1) / bn), 1, (double)bm, (double)bn, whole, &pl.map);
    return pl;
}

// us of expansion and product together (230 forwards of 33 to 830 tokens: mean error 4 %, 18 % at worst)
double two_kernel_estimate(int64_t T, int64_t N, int64_t K, int q) {
    double product = 0.0;
    gemm_plan(T, N, K, &product);
    return 3.3 + 1.045e-3 * product + (0.315e-6 + 0.026e-6 * q) * (double)(N * K);
}

static hipError_t launch_gemm(const GemmPlan& pl, const bf16_t* A, int64_t lda, const u32x4* frag, bf16_t* C, int64_t ldc, int64_t M,
                              int64_t NC, int64_t R, int64_t R16, hipStream_t st) {
    switch (pl.shape) {
        case 0: return launch_gemm_cfg<256, 256>(pl, A, lda, frag, C, ldc, M, NC, R, R16, st);
        case 1: return launch_gemm_cfg<256, 192>(pl, A, lda, frag, C, ldc, M, NC, R, R16, st);
        case 2: return launch_gemm_cfg<256, 160>(pl, A, lda, frag, C, ldc, M, NC, R, R16, st);
        case 3: return launch_gemm_cfg<256, 128>(pl, A, lda, frag, C, ldc, M, NC, R, R16, st);
        case 4: return launch_gemm_cfg<128, 160>(pl, A, lda, frag, C, ldc, M, NC, R, R16, st);
        case 5: return launch_gemm_cfg<128, 128>(pl, A, lda, frag, C, ldc, M, NC, R, R16, st);
        case 6: return launch_gemm_cfg<64, 128>(pl, A, lda, frag, C, ldc, M, NC, R, R16, st);
        default: return launch_gemm_cfg<64, 64>(pl, A, lda, frag, C, ldc, M, NC, R, R16, st);
    }
}

hipError_t launch_fwd_mfma(const uint32_t* packed, const ScaleParts& alpha, const void* x, int64_t T, int64_t N,
                           int64_t K, int64_t g, int q, void* y, void* workspace, hipStream_t st) {
    const int64_t R16 = round_up(K, RPAD) / 16;
    const GemmPlan pl = gemm_plan(T, N, K);
    const int64_t blocks = (N + 31) / 32 * 4, runs = (R16 / 2 + 31) / 32;
    dim3 grid = pl.columns() ? dim3(xcd_grid(blocks * runs)) : dim3((unsigned)blocks, (unsigned)runs);
    const unsigned expand_blocks = grid.x;
    if (alpha.joined) grid.x += (unsigned)(((int64_t)q * N * (K / g) + 2048 * grid.y - 1) / (2048 * grid.y));
#define BCQ_EXPAND(Q) \
    BCQ_LAUNCH(expand_fwd_kernel<Q>, grid, dim3(256), 0, st, packed, alpha, expand_blocks, N, K, g, q, R16, (int)pl.columns(), (u32x4*)workspace)
    switch (q) {
        case 1: BCQ_EXPAND(1); break;
        case 2: BCQ_EXPAND(2); break;
        case 3: BCQ_EXPAND(3); break;
        case 4: BCQ_EXPAND(4); break;
        default: BCQ_EXPAND(0); break;
    }
#undef BCQ_EXPAND
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_gemm(pl, (const bf16_t*)x, K, (const u32x4*)workspace, (bf16_t*)y, N, T, N, K, R16, st);
}

static dim3 expand_bwd_grid(int64_t K, int64_t R16) { return dim3(xcd_grid(K / 32) * (unsigned)((R16 / 2 + 7) / 8)); }
// The XCD order of expand_bwd_kernel gives whole column tiles to an XCD: only where the eighths are equal within 7 % (18 tiles,
// q = 5, 10002 rows: 20.5 us in plain order, 26 with eighths of two and three).
static bool even_eighths(int64_t K) { return (K / 32 + 7) / 8 * 8 * 15 <= K / 32 * 16; }

// sums != nullptr (up to four planes): the expansion's launch also reduces a scale gradient
static hipError_t launch_input_product(const uint32_t* packed, const uint32_t* packed_t, const float* alpha, const void* dy,
                                       int64_t T, int64_t N, int64_t K, int64_t g, int q, void* dx, void* workspace,
                                       const DalphaSums* sums, hipStream_t st) {
    const int64_t R16 = round_up(N, RPAD) / 16;
    u32x4* frag = (u32x4*)workspace;
    const GemmPlan pl = gemm_plan(T, K, N);
    const int columns = pl.columns();
    const unsigned rows_blocks = xcd_grid(R16 / 2 * ((K / 32 + 7) / 8));
    const DalphaSums reduce = sums ? *sums : DalphaSums{};
    const dim3 rows_grid(rows_blocks + (sums ? dalpha_reduce_blocks(reduce) : 0u));
#define BCQ_EXPAND(Q)                                                                                                      \
    BCQ_LAUNCH(expand_bwd_rows_kernel<Q>, rows_grid, dim3(256), 0, st, packed, alpha, N, K, g, R16, columns, frag, rows_blocks, \
               reduce)
    switch (q) {
        case 1: BCQ_EXPAND(1); break;
        case 2: BCQ_EXPAND(2); break;
        case 3: BCQ_EXPAND(3); break;
        case 4: BCQ_EXPAND(4); break;
        default:
            if (packed_t && N % 32 == 0)
                BCQ_LAUNCH((expand_bwd_kernel<true, false>), expand_bwd_grid(K, R16), dim3(256), 0, st, packed_t, alpha, N, K, g, q,
                           R16, columns && even_eighths(K), frag);
            else
                BCQ_LAUNCH((expand_bwd_kernel<false, false>), expand_bwd_grid(K, R16), dim3(256), 0, st, packed, alpha, N, K, g, q,
                           R16, columns && even_eighths(K), frag);
    }
#undef BCQ_EXPAND
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_gemm(pl, (const bf16_t*)dy, N, frag, (bf16_t*)dx, K, T, K, N, R16, st);
}

hipError_t launch_bwd_input_mfma(const uint32_t* packed, const uint32_t* packed_t, const float* alpha, const void* dy,
                                 int64_t T, int64_t N, int64_t K, int64_t g, int q, void* dx, void* workspace,
                                 hipStream_t st) {
    return launch_input_product(packed, packed_t, alpha, dy, T, N, K, g, q, dx, workspace, nullptr, st);
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
    const int columns = gemm_plan(T < SPLIT_TOKENS ? T : SPLIT_TOKENS, K, 3 * P).columns() && even_eighths(K);
    BCQ_LAUNCH((expand_bwd_kernel<false, true>), expand_bwd_grid(K, R16), dim3(256), 0, st, packed, alpha, N, K, g, q, R16, columns,
                       frag);
    hipError_t e = hipGetLastError();
    for (int64_t t0 = 0; t0 < T && e == hipSuccess; t0 += SPLIT_TOKENS) {
        const int64_t M = T - t0 < SPLIT_TOKENS ? T - t0 : SPLIT_TOKENS;
        BCQ_LAUNCH((pad_act_kernel<3>), dim3((unsigned)((M * (P / 8) + 255) / 256)), dim3(256), 0, st,
                           (const bf16_t*)dy + t0 * N, M, N, P, rows);
        e = hipGetLastError();
        if (e == hipSuccess)
            e = launch_gemm(gemm_plan(M, K, 3 * P), (const bf16_t*)rows, 3 * P, frag, (bf16_t*)dx + t0 * K, K, M, K, 3 * P, 3 * R16, st);
    }
    return e;
}


// =========================================================================================================
// Scale gradient on the matrix cores.  AlphaTuning Eq. 4, read as the gradient of Eq. 2, is
//     dalpha_i[n] = s * sum_t dY[t][n] * (X B_i^T)[t][n] = s * sum_k B_i[n][k] * G[n][k],   G = dY^T X.
// G is one dense contraction over the tokens (2 T N K matrix-core flops for ALL planes together, instead of
// 2 q T N K for q plane products); the sign planes only enter a signed row sum of the accumulators.
//
// Both MFMA operands need the token index innermost, which neither activation has in memory:
//   1. dalpha_kernel: a tile of G^T (k x n) for one slice of the tokens.  Both activations go global -> LDS directly as
//      they lie in memory (rows of tokens) and are transposed on the way out by ds_read_b64_tr_b16: no transposed copy
//      (34 us and 64 MB each way for 2048 columns at 16384 tokens), no transposition in registers.  Loop, waits and barrier are
//      those of gemm_kernel, and so is what bounds it: power with all compute units busy (8192 x 2048 at 16384 tokens,
//      q = 3, the whole call 490 -> 404 us, 6144 x 2048 463 -> 322, 3072 x 1024 at 4096 tokens 41 -> 33).  The epilogue forms the signed sums
//      over k for every trained plane.
//   2. dalpha_reduce adds the partial sums of all (token slice, k tile) pairs in a fixed order (no
//      floating-point atomics, bit-reproducible).

// Rows of 64 tokens, BK or BN columns wide, in 32-byte pieces (16 columns) with piece c of token t at c ^ da_swizzle(t): the
// transposing read takes 4 tokens x 32 bytes per 16 lanes, and the eight tokens that 32 lanes touch then lie in different banks.
__device__ __forceinline__ int da_swizzle(int t) { return (t & 3) | (((t >> 3) & 1) << 2); }

template <int TILE> struct DalphaShape;  // TILE x TILE outputs; WK x WN waves; NX, NY: stages of x and dy
template <> struct DalphaShape<256> { static constexpr int WK = 2, WN = 4, NX = 3, NY = 2; };
template <> struct DalphaShape<128> { static constexpr int WK = 2, WN = 2, NX = 5, NY = 5; };
template <int TILE>
struct DalphaCfg : DalphaShape<TILE> {
    using S = DalphaShape<TILE>;
    static constexpr int NW = S::WK * S::WN;
    static constexpr int TK = TILE / S::WK / 16, TN = TILE / S::WN / 16;
    static constexpr int ROWB = TILE * 2, STAGE_B = 64 * ROWB;     // a stage: 64 tokens
    static constexpr int RPI = 1024 / ROWB;                        // tokens per 1 KiB request
    static constexpr int J = 64 / RPI / NW;                        // requests per wave and stage
    static constexpr int LDS_B = (S::NX + S::NY) * STAGE_B;
    static_assert(J * RPI * NW == 64 && LDS_B <= 160 * 1024 && S::NX >= S::NY && S::NX - S::NY <= 1, "as in gemm_kernel");
};

// QT: planes summed in the epilogue (q_train rounded up to 1, 2, 3, 4 or 8; extra planes are computed, not stored).
// FINE: partial sums are kept per 32 columns k (for scale groups that are not whole tiles) instead of per tile; they
//       go to part[split][plane][n][TILE / 32 tiles_k] and the reduction adds each group's run.
template <int TILE, int QT, bool FINE>
__global__ __launch_bounds__((64 * DalphaCfg<TILE>::NW), 2) void dalpha_kernel(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ dy, int64_t ldy, const uint32_t* __restrict__ packed,
    float* __restrict__ part, int64_t T, int64_t N, int64_t K, int q_train, TileMap tmap, int64_t tokens_per_split) {
#if defined(__HIP_DEVICE_COMPILE__)
    using Cfg = DalphaCfg<TILE>;
    constexpr int WN = Cfg::WN, TK = Cfg::TK, TN = Cfg::TN, NX = Cfg::NX, NY = Cfg::NY, J = Cfg::J, RPI = Cfg::RPI;
    constexpr int ROWB = Cfg::ROWB, STAGE_B = Cfg::STAGE_B;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave / WN, wn = wave % WN;
    const int tiles_k = tmap.tiles_m;
    int split, tile_k, tile_n;
    if (!map_tile(tmap, split, tile_k, tile_n)) return;
    const int64_t k0 = (int64_t)tile_k * TILE, n0 = (int64_t)tile_n * TILE;
    const int64_t t_begin = (int64_t)split * tokens_per_split;  // a multiple of 64
    const int64_t t_end = (t_begin + tokens_per_split < T) ? t_begin + tokens_per_split : T;
    const int last = (int)((t_end - t_begin + 63) / 64) - 1;

    f32x4 acc[TN][TK];  // [n tile][k tile]
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TK; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Requests: a lane's 16 bytes land at its place of the row and come from where the swizzle puts them.  The descriptor of a
    // step starts at its first token and ends with the activation, so tokens beyond T come back as zeros; columns beyond
    // K or N (of the next row) only feed outputs that are never stored.
    uint32_t xoff[J], yoff[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int t = (wave * J + j) * RPI + lane / (64 / RPI);
        const int col = ((lane % (64 / RPI)) ^ (da_swizzle(t) << 1)) * 16;
        xoff[j] = (uint32_t)(t * K * 2 + col);
        yoff[j] = (uint32_t)(t * ldy * 2 + col);
    }
    auto rows_from = [&](const bf16_t* act, int64_t ld, int64_t col, int step) {
        const int64_t t = t_begin + (int64_t)(step < last ? step : last) * 64;
        const int64_t left = ((T - t) * ld - col) * 2;
        return __builtin_amdgcn_make_buffer_rsrc((void*)(act + t * ld + col), 0, (int)(left < 0x7fffffffll ? left : 0x7fffffffll),
                                                 0x00020000);
    };
    auto dma = [&](__amdgpu_buffer_rsrc_t rows, int stage_byte, uint32_t off, int j) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rows, (void __attribute__((address_space(3)))*)(smem + stage_byte + (wave * J + j) * 1024), 16, off, 0, 0, 0);
    };

    // Fragments (16 columns x 32 tokens): two transposing reads, lanes 16 h .. + 15 give the addresses of tokens 8 h + 0 .. 3
    // and + 4 .. 7 (four lanes to a token's 32 bytes) and receive one column each.  As in gemm_kernel the reads are inline
    // assembly, tied to an explicit wait.
    u32x2 xf[2][TK][2], yf[2][TN][2];
    const int h = lane >> 4, tok = 8 * h + ((lane >> 2) & 3);
    const uint32_t lanebase = (uint32_t)(tok * ROWB + (lane & 3) * 8);
    uint32_t xaddr[TK], yaddr[TN];
#pragma unroll
    for (int i = 0; i < TK; ++i) xaddr[i] = lanebase + (uint32_t)(((wk * TK + i) ^ da_swizzle(tok)) * 32);
#pragma unroll
    for (int j = 0; j < TN; ++j) yaddr[j] = lanebase + (uint32_t)(((wn * TN + j) ^ da_swizzle(tok)) * 32 + NX * STAGE_B);
    auto read_t = [&](u32x2 (&f)[2], uint32_t addr, auto KK) {
        constexpr int kk = decltype(KK)::value;
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(f[0]) : "v"(addr), "n"(kk * 32 * ROWB));
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(f[1]) : "v"(addr), "n"(kk * 32 * ROWB + 4 * ROWB));
    };
    auto arrived = [&](int p) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < TK; ++i) asm volatile("" : "+v"(xf[p][i][0]), "+v"(xf[p][i][1]));
#pragma unroll
        for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(yf[p][j][0]), "+v"(yf[p][j][1]));
        __builtin_amdgcn_sched_barrier(0);
    };
    auto whole = [](const u32x2 (&f)[2]) { return as_bf16x8(u32x4{f[0][0], f[0][1], f[1][0], f[1][1]}); };
    auto slice = [&](auto KK, uint32_t xstage, uint32_t ystage, auto&& also) {
        constexpr int kk = decltype(KK)::value, NM = TK * TN, NR = TK + TN;
        constexpr int GAP = NM * 3 / 4 / NR > 0 ? NM * 3 / 4 / NR : 1;
        static_assert(NR <= NM, "one fragment per MFMA");
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const int j = m / TK, i = (j & 1) ? TK - 1 - m % TK : m % TK;
            acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(whole(xf[kk][i]), whole(yf[kk][j]), acc[j][i], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (m % GAP == 0) {
                const int r = m / GAP;
                if (r < TN) read_t(yf[1 - kk][r], yaddr[r] + ystage, std::integral_constant<int, 1 - kk>{});
                else if (r < NR) read_t(xf[1 - kk][r - TN], xaddr[r - TN] + xstage, std::integral_constant<int, 1 - kk>{});
            }
            also(m);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

#pragma unroll
    for (int p = 0; p < NX; ++p) {
        const auto xr = rows_from(x, K, k0, p), yr = rows_from(dy, ldy, n0, p);
#pragma unroll
        for (int j = 0; j < J; ++j) dma(xr, p * STAGE_B, xoff[j], j);
        if (p < NY) {
#pragma unroll
            for (int j = 0; j < J; ++j) dma(yr, (NX + p) * STAGE_B, yoff[j], j);
        }
    }
    asm volatile("s_waitcnt %0" ::"n"(wait_vm((NX + NY - 2) * J)) : "memory");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < TN; ++j) read_t(yf[0][j], yaddr[j], std::integral_constant<int, 0>{});
#pragma unroll
    for (int i = 0; i < TK; ++i) read_t(xf[0][i], xaddr[i], std::integral_constant<int, 0>{});
    __builtin_amdgcn_sched_barrier(0);

    int sx = 0, sy = 0;  // stages of step s
    for (int s = 0; s <= last; ++s) {
        const int sx_next = sx + 1 == NX ? 0 : sx + 1, sy_next = sy + 1 == NY ? 0 : sy + 1;
        arrived(0);
        slice(std::integral_constant<int, 0>{}, (uint32_t)(sx * STAGE_B), (uint32_t)(sy * STAGE_B), [](int) {});
        arrived(1);
        asm volatile("s_waitcnt %0" ::"n"(wait_vm((NX + NY - 4) * J)) : "memory");  // the hand-over, as in gemm_kernel
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        const auto xr = rows_from(x, K, k0, s + NX), yr = rows_from(dy, ldy, n0, s + NY);
        slice(std::integral_constant<int, 1>{}, (uint32_t)(sx_next * STAGE_B), (uint32_t)(sy_next * STAGE_B), [&](int m) {
            constexpr int GAP = TK * TN / (2 * J);
            static_assert(GAP > 0, "at most one request per MFMA");
            if (m % GAP != GAP - 1) return;
            const int d = m / GAP;
            if (d < J) dma(yr, (NX + sy) * STAGE_B, yoff[d], d);
            else if (d < 2 * J) dma(xr, sx * STAGE_B, xoff[d - J], d - J);
        });
        sx = sx_next;
        sy = sy_next;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    arrived(0);
    __syncthreads();

    // epilogue: signed sums over this wave's k for each plane; lane (c = lane % 16, h) owns n = 16 j + c and k = 16 i + 4 h + e.
    // The packed words of (up to four) planes are requested first (one memory latency instead of one per plane);
    // a sign is applied as a factor +-1.0 built from the (inverted) plane bit: shift, and-or, fused multiply-add
    // per value (the product with +-1.0 is exact, so this equals adding the signed value).
    constexpr int WORDS = TK / 2;  // packed words (32 columns) of this wave
    constexpr int SLOTS = FINE ? TILE / 32 : Cfg::WK;  // sums per (plane, n): per 32 columns, or per wave row
    constexpr int PB = QT > 4 ? 4 : QT;                // planes at a time
    float* red = reinterpret_cast<float*>(smem);       // [plane][slot][n]
    const int64_t Kw = K / 32, kt0 = (k0 + wk * 16 * TK) / 32;
    const bool quad = WORDS == 4 && (kt0 + 3 < Kw) && ((Kw & 3) == 0);  // one aligned 16-byte load per row and plane
#pragma unroll
    for (int pb = 0; pb < QT; pb += PB) {
        uint32_t words[PB][TN][WORDS];  // already inverted and shifted to this lane's columns
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            const int pc = pb + p < q_train ? pb + p : q_train - 1;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int64_t n = n0 + (wn * TN + j) * 16 + (lane & 15);
                const int64_t nc = n < N ? n : N - 1;
                const uint32_t* prow = packed + ((int64_t)pc * N + nc) * Kw;
                if (quad) {
                    const u32x4 w4 = *reinterpret_cast<const u32x4*>(prow + kt0);
#pragma unroll
                    for (int w = 0; w < WORDS; ++w) words[p][j][w] = ~(w4[w & 3] >> (4 * h));
                } else {
#pragma unroll
                    for (int w = 0; w < WORDS; ++w) words[p][j][w] = ~(prow[kt0 + w < Kw ? kt0 + w : Kw - 1] >> (4 * h));
                }
            }
        }
        // the four lanes that share an n, in a fixed order
        auto put = [&](const float (&sum)[PB][TN], int slot) {
#pragma unroll
            for (int p = 0; p < PB; ++p)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    float s = sum[p][j];
                    s += __shfl_xor(s, 16);
                    s += __shfl_xor(s, 32);
                    if (lane < 16) red[((pb + p) * SLOTS + slot) * TILE + (wn * TN + j) * 16 + lane] = s;
                }
        };
        float sum[PB][TN] = {};  // every accumulator is read once and added, with its sign, into the sums of the planes
#pragma unroll
        for (int w = 0; w < WORDS; ++w) {
            if (kt0 + w < Kw) {  // uniform: words beyond K hold nothing that counts
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int v = 0; v < 8; ++v) {
                        const int bit = 16 * (v >> 2) + (v & 3);
                        const float a = acc[j][2 * w + (v >> 2)][v & 3];
#pragma unroll
                        for (int p = 0; p < PB; ++p)  // sign bit set where the plane bit is 0 (-1): words are inverted
                            sum[p][j] = __builtin_fmaf(a, __uint_as_float(((words[p][j][w] << (31 - bit)) & 0x80000000u) | 0x3f800000u), sum[p][j]);
                    }
            }
            if (FINE) {
                put(sum, wk * WORDS + w);
#pragma unroll
                for (int p = 0; p < PB; ++p)
#pragma unroll
                    for (int j = 0; j < TN; ++j) sum[p][j] = 0.f;
            }
        }
        if (!FINE) put(sum, wk);
    }
    __syncthreads();
    const int64_t n = n0 + tid;
    if (tid >= TILE || n >= N) return;
    for (int p = 0; p < q_train; ++p) {
        const float* sums = red + p * SLOTS * TILE + tid;
        if (FINE) {
            float* dst = part + (((int64_t)split * q_train + p) * N + n) * ((int64_t)tiles_k * SLOTS) + (int64_t)tile_k * SLOTS;
#pragma unroll
            for (int c = 0; c < SLOTS; c += 4)
                *reinterpret_cast<f32x4*>(dst + c) = f32x4{sums[c * TILE], sums[(c + 1) * TILE], sums[(c + 2) * TILE], sums[(c + 3) * TILE]};
        } else {
            static_assert(FINE || SLOTS == 2, "two rows of waves");
            part[(((int64_t)split * tiles_k + tile_k) * q_train + p) * N + n] = sums[0] + sums[TILE];
        }
    }
#endif
}

// Bytes of scratch that a call may use for its partial sums: what callers have been told since the kernel also kept a
// transposed copy of the smaller activation there (which bounds the token slices only where T or both dimensions are small).
struct DalphaBudget {
    size_t copy, part;
};
static DalphaBudget dalpha_budget(int64_t T, int64_t N, int64_t K, int64_t g, int q) {
    const int64_t tiles_k = (K + 255) / 256, tiles = tiles_k * ((N + 255) / 256);
    int64_t s = tiles >= 256 ? 1 : 256 / tiles;
    const int64_t max_s = (T + 255) / 256;
    if (s > max_s) s = max_s;
    if (s < 1) s = 1;
    const int64_t per_split = ((T + s - 1) / s + 63) / 64 * 64, splits = (T + per_split - 1) / per_split;
    DalphaBudget b;
    b.copy = (size_t)((((K <= N ? K : N) + 31) / 32) * ((T + 63) / 64 * 4) * 1024);
    b.part = (size_t)splits * tiles_k * q * N * sizeof(float) * (g != K && g % 256 != 0 ? 8 : 1);
    return b;
}

struct DalphaPlan {
    int tile, tiles_k, tiles_n, splits;
    int64_t per_split;
    bool fine;  // groups that are not whole k tiles need per-32-column partials
};

// Tile and token slices by an estimate like that of gemm_plan: a step of 64 tokens 0.0117 ns per product and 1.25 ns per
// row and column, at least 490 ns; a round 6.4 us and 0.5 us per trained plane and 256 x 256 outputs; the partial sums,
// written and read by the reduction, 1 ns a KB.  `budget` bounds those.  Of 6870 calls of 17 to 8192 tokens, q = 1 .. 8, one or all
// planes trained, g = K, 32 .. 640, the pick is within 4 % of the fastest of up to ten tiles and slice counts for 96 %, within
// 10 % for 98 % (6144 x 2048 at 16384 tokens: 192 tiles in one slice leave a quarter of the chip idle, 430 us; four slices 322.
// With all planes counted, trained or not, and 2 ns a KB, which is dear where partial sums are kept per 32 columns, 128 x
// 128 tiles were taken for groups of 128 and many planes: 10240 x 2560, q = 8, 22 tokens 124 us, now 76).
static DalphaPlan dalpha_plan(int64_t T, int64_t N, int64_t K, int64_t g, int q_train, int smallest, size_t budget) {
    static const ShareTable share(0.112);
    DalphaPlan best = {};
    double least = 1e300;
    const int64_t steps = (T + 63) / 64;
    for (int tile = 256; tile >= smallest; tile -= 128) {
        DalphaPlan pl;
        pl.tile = tile;
        pl.tiles_k = (int)((K + tile - 1) / tile);
        pl.tiles_n = (int)((N + tile - 1) / tile);
        pl.fine = (g != K) && (g % tile != 0);
        const int64_t tiles = (int64_t)pl.tiles_k * pl.tiles_n;
        const size_t slice_bytes = (size_t)pl.tiles_k * q_train * N * sizeof(float) * (pl.fine ? tile / 32 : 1);
        int64_t before = 0;
        for (int64_t s = 1; s <= steps && s <= 64 && (s == 1 || s * tiles <= 2048); ++s) {
            const int64_t per = (steps + s - 1) / s, splits = (steps + per - 1) / per;
            if (splits == before) continue;
            before = splits;
            const size_t bytes = (size_t)splits * slice_bytes;
            if (bytes > budget) break;  // (256 x 256 tiles in one slice always fit)
            const double t = round_estimate(0.0117 * tile * tile + 2.5 * tile, 490.0, share, tiles * splits, per,
                                            6400.0 + 500.0 * q_train * tile * tile / 65536.0) + (double)bytes / 1000.0;
            if (t < least) {
                least = t;
                best = pl;
                best.splits = (int)splits;
                best.per_split = per * 64;
            }
        }
    }
    return best;
}

// Rows of dy that are not 16-byte aligned are copied into padded ones, this many tokens at a time (a multiple of 64): the
// copy stays below 512 MiB (50257 rows: 5312 tokens), and the partial sums of all pieces are added at the end.
static int64_t dalpha_piece(int64_t T, int64_t N) {
    if (N % 8 == 0) return T;
    int64_t piece = ((int64_t)1 << 29) / (2 * round_up(N, 8)) / 64 * 64;
    if (piece > ((int64_t)1 << 20)) piece = (int64_t)1 << 20;
    return T < piece ? T : piece;
}

// Workspace: [partial sums][padded copy of a piece]
struct DalphaScratch {
    size_t part, pad;
};
static DalphaScratch dalpha_scratch(int64_t T, int64_t N, int64_t K, int64_t g, int q) {
    const int64_t piece = dalpha_piece(T, N), whole = T / piece, rest = T % piece;
    const DalphaBudget a = dalpha_budget(piece, N, K, g, q);
    DalphaScratch s = {a.copy + (size_t)whole * a.part, 0};
    if (rest) s.part += dalpha_budget(rest, N, K, g, q).part;
    if (N % 8) {
        s.part = (s.part + 15) / 16 * 16;
        s.pad = (size_t)(piece * round_up(N, 8) * 2);
    }
    return s;
}
// One piece: any plan within the budget.  Several: 256 x 256 tiles for all, so that one reduction takes their partial sums.
static DalphaPlan dalpha_piece_plan(int64_t M, int64_t T, int64_t N, int64_t K, int64_t g, int q, int q_train) {
    const DalphaBudget b = dalpha_budget(M, N, K, g, q);
    return M == T ? dalpha_plan(M, N, K, g, q_train, 128, b.copy + b.part) : dalpha_plan(M, N, K, g, q_train, 256, b.part);
}

size_t mfma_bwd_alpha_workspace(int64_t T, int64_t N, int64_t K, int64_t g, int q) {
    const DalphaScratch s = dalpha_scratch(T, N, K, g, q);
    return s.part + s.pad;
}

// Partial sums of T tokens into `part`
template <int TILE>
static hipError_t launch_dalpha_tile(const uint32_t* packed, const bf16_t* x, const bf16_t* dy, int64_t dcols, int64_t T,
                                     int64_t N, int64_t K, int q_train, const DalphaPlan& pl, float* part, hipStream_t st) {
    TileMap tmap;
    const unsigned wgs = make_tile_map(pl.tiles_k, pl.tiles_n, pl.splits, 1.0, 1.0, 0.0, &tmap);
    using Cfg = DalphaCfg<TILE>;
#define BCQ_DA_LAUNCH(QTV, FV)                                                                                        \
    {                                                                                                                 \
        static LdsLimit limit;                                                                                        \
        hipError_t ea = limit.ensure((const void*)dalpha_kernel<TILE, QTV, FV>, (size_t)Cfg::LDS_B);                   \
        if (ea != hipSuccess) return ea;                                                                              \
        BCQ_LAUNCH((dalpha_kernel<TILE, QTV, FV>), dim3(wgs), dim3(64 * Cfg::NW), Cfg::LDS_B, st, x, dy, dcols, packed, \
                   part, T, N, K, q_train, tmap, pl.per_split);                                                       \
    }
#define BCQ_DA_Q(FV)                                \
    switch (q_train) {                              \
        case 1: BCQ_DA_LAUNCH(1, FV) break;         \
        case 2: BCQ_DA_LAUNCH(2, FV) break;         \
        case 3: BCQ_DA_LAUNCH(3, FV) break;         \
        case 4: BCQ_DA_LAUNCH(4, FV) break;         \
        default: BCQ_DA_LAUNCH(8, FV) break;        \
    }
    if (pl.fine) {
        BCQ_DA_Q(true)
    } else {
        BCQ_DA_Q(false)
    }
#undef BCQ_DA_Q
#undef BCQ_DA_LAUNCH
    return hipGetLastError();
}

// Partial sums of all tokens into the workspace; *out: what is left to reduce
static hipError_t launch_dalpha_sums(const uint32_t* packed, const void* x, const void* dy, int64_t T, int64_t N, int64_t K,
                                     int64_t g, int q, int q_train, float grad_scale, float* dalpha, void* workspace,
                                     DalphaSums* out, hipStream_t st) {
    const DalphaScratch sc = dalpha_scratch(T, N, K, g, q);
    const int64_t piece = dalpha_piece(T, N), dcols = sc.pad ? round_up(N, 8) : N;
    unsigned char* ws = static_cast<unsigned char*>(workspace);
    float* part = reinterpret_cast<float*>(ws);
    float* next = part;
    DalphaPlan pl = {};
    int splits = 0;
    for (int64_t t0 = 0; t0 < T; t0 += piece) {
        const int64_t M = T - t0 < piece ? T - t0 : piece;
        pl = dalpha_piece_plan(M, T, N, K, g, q, q_train);
        const bf16_t* rows = (const bf16_t*)dy + t0 * N;
        if (sc.pad) {
            u32x4* padded = reinterpret_cast<u32x4*>(ws + sc.part);
            BCQ_LAUNCH((pad_act_kernel<1>), dim3((unsigned)((M * (dcols / 8) + 255) / 256)), dim3(256), 0, st, rows, M, N,
                               dcols, padded);
            hipError_t ep = hipGetLastError();
            if (ep != hipSuccess) return ep;
            rows = reinterpret_cast<const bf16_t*>(padded);
        }
        const bf16_t* xrows = (const bf16_t*)x + t0 * K;
        hipError_t ep = pl.tile == 256 ? launch_dalpha_tile<256>(packed, xrows, rows, dcols, M, N, K, q_train, pl, next, st)
                                       : launch_dalpha_tile<128>(packed, xrows, rows, dcols, M, N, K, q_train, pl, next, st);
        if (ep != hipSuccess) return ep;
        next += (int64_t)pl.splits * pl.tiles_k * q_train * N * (pl.fine ? pl.tile / 32 : 1);
        splits += pl.splits;
    }
    *out = {};
    out->part = part;
    out->dalpha = dalpha;
    out->rows = (int64_t)q_train * N;
    out->G = K / g;
    out->splits = splits;
    out->scale = grad_scale;
    out->fine = pl.fine;
    out->per_slice = pl.fine ? (int64_t)pl.tiles_k * (pl.tile / 32) : pl.tiles_k;
    out->run = pl.fine ? (int)(g / 32) : (int)(g == K ? pl.tiles_k : g / pl.tile);
    return hipSuccess;
}

hipError_t launch_bwd_alpha_mfma(const uint32_t* packed, const void* x, const void* dy, int64_t T, int64_t N,
                                 int64_t K, int64_t g, int q, int q_train, float grad_scale, float* dalpha,
                                 void* workspace, const AdamWArgs* opt, hipStream_t st) {
    DalphaSums sums;
    hipError_t e = launch_dalpha_sums(packed, x, dy, T, N, K, g, q, q_train, grad_scale, dalpha, workspace, &sums, st);
    if (e != hipSuccess) return e;
    if (opt) sums.opt = *opt;
    BCQ_LAUNCH(dalpha_reduce_kernel, dim3(dalpha_reduce_blocks(sums)), dim3(256), 0, st, sums);
    return hipGetLastError();
}

hipError_t launch_bwd_mfma(const uint32_t* packed, const float* alpha, const void* x, const void* dy, int64_t T, int64_t N, int64_t K,
                           int64_t g, int q, int q_train, float grad_scale, void* dx, void* input_workspace, float* dalpha,
                           void* alpha_workspace, hipStream_t st) {
    DalphaSums sums;
    hipError_t e = launch_dalpha_sums(packed, x, dy, T, N, K, g, q, q_train, grad_scale, dalpha, alpha_workspace, &sums, st);
    if (e != hipSuccess) return e;
    return launch_input_product(packed, nullptr, alpha, dy, T, N, K, g, q, dx, input_workspace, &sums, st);
}

}  // namespace bcq

// Any-shape kernels for the BCQ linear layer in fp64: on the matrix cores (v_mfma_f64_16x16x4_f64) and, for few tokens or
// few rows, on the vector ALU; fp32 or bf16 I/O.
// They evaluate AlphaTuning Eq. 2 (forward), Eq. 3 (input gradient) and Eq. 4 (scale gradient, read as the
// gradient of Eq. 2) directly on the packed sign planes, never forming W in memory, and need no workspace.
// The library uses them for fp32 activations, for shapes the tiled bf16 matrix-core kernels do not take, and
// whenever the caller passes no workspace.
//
// Why fp64: its roundings, 2^-53 relative for every step of What = sum_i +-alpha_i and of the contraction, stay far below
// the one rounding of a bf16 or fp32 result, so that the order in which waves share the contraction is free.  One
// 16 x 16 x 4 instruction is 2048 flops, ~45 TFLOP/s measured over the chip: the 1024 x 1024 layer at 32 tokens needs 1.5 us
// per product, so the calls are bound by launch and load latency, and the split is chosen to put every compute unit to work:
// one workgroup per 16 output columns, its eight waves share the contraction and add their tiles in wave order through LDS
// (bit-reproducible).
// Measured against one wave per row / one thread per column on the vector ALU (which read every activation once per
// plane and ran the contraction over N serially), kernel times: 1024 x 1024 at 32 fp32 tokens forward 26 -> 9, input
// gradient 685 -> 10, scale gradient 42 -> 14 us; 1500 x 1056 at 333 bf16 tokens input gradient 1347 -> 52, scale
// gradient 527 -> 70 us (with a workspace the padded forms of bcq_mfma.hip take these from there on).
//
// Lane layout (checked by measurement): lane l holds A[row l % 16][k l / 16], B[k l / 16][col l % 16] and, in
// accumulator register r, D[row 4 r + l / 16][col l % 16].  The contraction index of a lane group may be any
// permutation as long as both operands agree: a group takes eight consecutive indices, one byte of a packed word.
#include "bcq_internal.h"

namespace bcq {

typedef __attribute__((ext_vector_type(4))) double f64x4;

constexpr int GEN_WAVES = 8;  // waves per workgroup, all on the same output tile

__device__ __forceinline__ f64x4 mfma_f64(double a, double b, f64x4 c) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
#else
    return c;
#endif
}

// eight consecutive activations; the pointer is only element-aligned when the row length is odd
template <typename XT>
struct Eight {
    XT v[8];
    __device__ __forceinline__ void load(const XT* p) { __builtin_memcpy(v, p, sizeof(v)); }
    __device__ __forceinline__ float at(int j) const { return Elem<XT>::load(&v[j]); }
};

// sign bit `s` of an inverted plane word, moved to the sign position and applied to an fp32 scale, widened to fp64
__device__ __forceinline__ double signed_scale(float a, uint32_t inverted, int s) {
    return (double)__uint_as_float(__float_as_uint(a) ^ ((inverted << (31 - s)) & 0x80000000u));
}

// Adds the eight waves' tiles in wave order and hands every sum to `put(tile, row, col, sum)`.
// part: [GEN_WAVES][TILES * 4][64] doubles
template <int TILES, typename Put>
__device__ __forceinline__ void reduce_tiles(double* part, const f64x4 (&acc)[TILES], Put put) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int t = 0; t < TILES; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[(wave * TILES * 4 + t * 4 + r) * 64 + lane] = acc[t][r];
    __syncthreads();
    for (int e = threadIdx.x; e < TILES * 256; e += GEN_WAVES * 64) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < GEN_WAVES; ++w) s += part[w * TILES * 256 + e];
        const int l = e & 63, r = (e >> 6) & 3;
        put(e >> 8, 4 * r + (l >> 4), l & 15, s);
    }
}

// Forward, Eq. 2: 16 rows n of W x 16 TT tokens per workgroup; the waves take the packed words in turn.
// Per word and lane: one byte (eight signs) of each plane, eight activations of TT tokens, 8 TT matrix instructions.
template <typename XT, int TT>
__global__ __launch_bounds__(GEN_WAVES * 64) void fwd_generic_kernel(const uint32_t* __restrict__ packed,
                                                                     const float* __restrict__ alpha,
                                                                     const XT* __restrict__ x, XT* __restrict__ y,
                                                                     int64_t T, int64_t N, int64_t K, int64_t g,
                                                                     int q) {
    __shared__ double part[GEN_WAVES * TT * 256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 15, h = lane >> 4;
    const int64_t n0 = (int64_t)blockIdx.y * 16, t0 = (int64_t)blockIdx.x * (16 * TT);
    const int64_t n = n0 + col < N ? n0 + col : N - 1;  // rows and tokens beyond the edge are computed, never stored
    const int64_t Kw = K / 32, G = K / g, gw = g / 32;
    const XT* xrow[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
        const int64_t t = t0 + tt * 16 + col;
        xrow[tt] = x + (t < T ? t : T - 1) * K + 8 * h;
    }
    f64x4 acc[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) acc[tt] = (f64x4){0.0, 0.0, 0.0, 0.0};

    uint32_t bits[8];
    float a[8];
    Eight<XT> xv[TT];
    auto load = [&](int64_t w) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i < q) {
                bits[i] = packed[((int64_t)i * N + n) * Kw + w];
                a[i] = alpha[((int64_t)i * N + n) * G + w / gw];  // a word never straddles groups: g % 32 == 0
            }
        }
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) xv[tt].load(xrow[tt] + 32 * w);
    };
    if (wave < Kw) load(wave);
    for (int64_t w = wave; w < Kw; w += GEN_WAVES) {
        double what[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) what[j] = 0.0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i < q) {
                const uint32_t inv = ~(bits[i] >> (8 * h));
#pragma unroll
                for (int j = 0; j < 8; ++j) what[j] += signed_scale(a[i], inv, j);
            }
        }
        double xd[TT][8];
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
            for (int j = 0; j < 8; ++j) xd[tt][j] = (double)xv[tt].at(j);
        if (w + GEN_WAVES < Kw) load(w + GEN_WAVES);  // in flight during the products
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) acc[tt] = mfma_f64(xd[tt][j], what[j], acc[tt]);
    }
    reduce_tiles<TT>(part, acc, [&](int tt, int row, int c, double s) {
        const int64_t t = t0 + tt * 16 + row;
        if (t < T && n0 + c < N) Elem<XT>::store(y + t * N + n0 + c, (float)s);
    });
}

// Input gradient, Eq. 3: 16 KB columns k (KB = 2: a whole packed word) x 16 TT tokens per workgroup; the waves take
// runs of 32 rows n in turn.  Lane l < 32 fetches row n0 + l's words, lane 32 + l its scales; both pass through a
// wave-private piece of LDS, from which every lane group reads the eight rows it contracts over.
template <typename XT, int TT, int KB>
__global__ __launch_bounds__(GEN_WAVES * 64) void bwd_input_generic_kernel(const uint32_t* __restrict__ packed,
                                                                           const float* __restrict__ alpha,
                                                                           const XT* __restrict__ dy,
                                                                           XT* __restrict__ dx, int64_t T, int64_t N,
                                                                           int64_t K, int64_t g, int q) {
    __shared__ double part[GEN_WAVES * TT * KB * 256];  // the staging area (2 KiB per wave) lies in its own wave's part
    static_assert(TT * KB * 256 * 8 >= 8 * 64 * 4, "staging of eight planes fits");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 15, h = lane >> 4;
    const int64_t k0 = (int64_t)blockIdx.y * (16 * KB), t0 = (int64_t)blockIdx.x * (16 * TT);
    const int64_t Kw = K / 32, G = K / g, grp = k0 / g, kw = k0 / 32;
    const int kbit = (int)(k0 & 31) + col;
    uint32_t* stage = reinterpret_cast<uint32_t*>(part + wave * TT * KB * 256);  // [plane][32 words, 32 scales]
    const XT* drow[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
        const int64_t t = t0 + tt * 16 + col;
        drow[tt] = dy + (t < T ? t : T - 1) * N;
    }
    f64x4 acc[TT * KB];
#pragma unroll
    for (int i = 0; i < TT * KB; ++i) acc[i] = (f64x4){0.0, 0.0, 0.0, 0.0};

    uint32_t mine[8];
    Eight<XT> dv[TT];
    const int64_t chunks = (N + 31) / 32;
    auto load = [&](int64_t c) {
        const int64_t n = c * 32 + (lane & 31);
        const bool live = n < N;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i < q) {
                const int64_t row = (int64_t)i * N + (live ? n : N - 1);
                const uint32_t v = lane < 32 ? packed[row * Kw + kw] : __float_as_uint(alpha[row * G + grp]);
                mine[i] = live ? v : 0u;  // rows beyond N have zero scales
            }
        }
        const int64_t nl = c * 32 + 8 * h;
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            if (nl + 8 <= N) {
                dv[tt].load(drow[tt] + nl);
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) dv[tt].v[j] = nl + j < N ? drow[tt][nl + j] : (XT)0;
            }
        }
    };
    if (wave < chunks) load(wave);
    for (int64_t c = wave; c < chunks; c += GEN_WAVES) {
        // LDS executes one wave's instructions in order: only the compiler has to keep writes and reads in order
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (i < q) stage[i * 64 + lane] = mine[i];
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        double what[KB][8];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int j = 0; j < 8; ++j) what[kb][j] = 0.0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i < q) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const uint32_t inv = ~stage[i * 64 + 8 * h + j];
                    const float a = __uint_as_float(stage[i * 64 + 32 + 8 * h + j]);
#pragma unroll
                    for (int kb = 0; kb < KB; ++kb) what[kb][j] += signed_scale(a, inv, kbit + 16 * kb);
                }
            }
        }
        double dd[TT][8];
#pragma unroll
        for (int tt = 0; tt < TT; ++tt)
#pragma unroll
            for (int j = 0; j < 8; ++j) dd[tt][j] = (double)dv[tt].at(j);
        if (c + GEN_WAVES < chunks) load(c + GEN_WAVES);
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt)
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
                    acc[tt * KB + kb] = mfma_f64(dd[tt][j], what[kb][j], acc[tt * KB + kb]);
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    reduce_tiles<TT * KB>(part, acc, [&](int tile, int row, int cc, double s) {
        const int64_t t = t0 + (tile / KB) * 16 + row, k = k0 + (tile % KB) * 16 + cc;
        if (t < T) Elem<XT>::store(dx + t * K + k, (float)s);
    });
}

// Scale gradient, Eq. 4 as the gradient of Eq. 2: dalpha_i[n] = s sum_k B_i[n][k] G[n][k], G = dY^T X.  16 rows n per
// workgroup; a wave forms G for its 32-column words (contraction over all tokens, four per instruction) and adds the
// signed row sums.  `per` waves (a power of two) share one scale group; when there are more groups than waves
// they are taken in rounds.
template <typename XT>
__global__ __launch_bounds__(GEN_WAVES * 64) void bwd_alpha_generic_kernel(const uint32_t* __restrict__ packed,
                                                                           const XT* __restrict__ x,
                                                                           const XT* __restrict__ dy,
                                                                           float* __restrict__ dalpha, int64_t T,
                                                                           int64_t N, int64_t K, int64_t g,
                                                                           int q_train, float grad_scale, int per) {
    __shared__ double red[GEN_WAVES][8][16];  // [wave][plane][n]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 15, h = lane >> 4;
    const int64_t n0 = (int64_t)blockIdx.x * 16;
    const int64_t Kw = K / 32, G = K / g, gw = g / 32;
    const int64_t nd = n0 + col < N ? n0 + col : N - 1;
    const int sub = wave % per, slot = wave / per, slots = GEN_WAVES / per;
    for (int64_t round = 0; round * slots < G; ++round) {
        const int64_t grp = round * slots + slot;
        double sum[8][4];  // [plane][row register]
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) sum[i][r] = 0.0;
        if (grp < G) {
            for (int64_t w = grp * gw + sub; w < (grp + 1) * gw; w += per) {
                f64x4 acc[2];
                acc[0] = acc[1] = (f64x4){0.0, 0.0, 0.0, 0.0};
                const XT* xp = x + 32 * w + 2 * col;
                int64_t t = 0;
                for (; t + 32 <= T; t += 32) {  // eight token quads in flight
                    XT xa[8][2], d[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int64_t tu = t + 4 * u + h;
                        __builtin_memcpy(xa[u], xp + tu * K, sizeof(xa[u]));
                        d[u] = dy[tu * N + nd];
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const double dd = (double)Elem<XT>::load(&d[u]);
                        acc[0] = mfma_f64(dd, (double)Elem<XT>::load(&xa[u][0]), acc[0]);
                        acc[1] = mfma_f64(dd, (double)Elem<XT>::load(&xa[u][1]), acc[1]);
                    }
                }
                for (; t < T; t += 4) {
                    const int64_t tu = t + h;
                    double dd = 0.0, x0 = 0.0, x1 = 0.0;
                    if (tu < T) {
                        dd = (double)Elem<XT>::load(dy + tu * N + nd);
                        x0 = (double)Elem<XT>::load(xp + tu * K);
                        x1 = (double)Elem<XT>::load(xp + tu * K + 1);
                    }
                    acc[0] = mfma_f64(dd, x0, acc[0]);
                    acc[1] = mfma_f64(dd, x1, acc[1]);
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    if (i < q_train) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int64_t n = n0 + 4 * r + h;
                            const uint32_t word = packed[((int64_t)i * N + (n < N ? n : N - 1)) * Kw + w] >> (2 * col);
                            sum[i][r] += (word & 1u) ? acc[0][r] : -acc[0][r];
                            sum[i][r] += (word & 2u) ? acc[1][r] : -acc[1][r];
                        }
                    }
                }
            }
        }
        if (round) __syncthreads();  // the previous round's sums have been read
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i < q_train) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    double s = sum[i][r];
#pragma unroll
                    for (int off = 8; off >= 1; off >>= 1) s += __shfl_xor(s, off);
                    if (col == 0) red[wave][i][4 * r + h] = s;
                }
            }
        }
        __syncthreads();
        for (int e = threadIdx.x; e < slots * q_train * 16; e += GEN_WAVES * 64) {
            const int row = e & 15, i = (e >> 4) % q_train, sl = (e >> 4) / q_train;
            const int64_t go = round * slots + sl;
            if (go < G && n0 + row < N) {
                double s = 0.0;
                for (int p = 0; p < per; ++p) s += red[sl * per + p][i][row];
                dalpha[((int64_t)i * N + n0 + row) * G + go] = (float)((double)grad_scale * s);
            }
        }
    }
}

// ---- few tokens or few rows: the vector ALU, also in fp64 ---------------------------------------------------------
// A 16 x 16 tile of the matrix instruction wastes most of its work on one or two tokens, or on a few rows; what remains
// are the planes, which these kernels read with whole waves, and What, which costs three operations per weight and plane.

// the value with the sign of an inverted plane bit, kept in fp64 from the start: shift, and-xor
__device__ __forceinline__ double signed_value(double a, uint32_t inverted, int s) {
    return __hiloint2double(__double2hiint(a) ^ (int)((inverted << (31 - s)) & 0x80000000u), __double2loint(a));
}

// Sums of the `share` (1 or 4) waves that work on one row, in wave order; all lanes of the first of them get the result.
template <int COUNT>
__device__ __forceinline__ void share_sums(double (&part)[4][COUNT], double (&s)[COUNT], int share) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < COUNT; ++i) s[i] = wave_sum(s[i]);
    if (share == 1) return;
    if (lane == 0)
#pragma unroll
        for (int i = 0; i < COUNT; ++i) part[wave][i] = s[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < COUNT; ++i) s[i] = (part[0][i] + part[1][i]) + (part[2][i] + part[3][i]);
}

// Forward: `share` waves per row n and ROW_TOKENS tokens, their lanes take the words of the row in turn.
constexpr int ROW_TOKENS = 4;
template <typename XT>
__global__ __launch_bounds__(256) void fwd_rows_kernel(const uint32_t* __restrict__ packed,
                                                       const float* __restrict__ alpha, const XT* __restrict__ x,
                                                       XT* __restrict__ y, int64_t T, int64_t N, int64_t K, int64_t g,
                                                       int q, int share) {
    __shared__ double part[4][ROW_TOKENS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, sub = share == 1 ? 0 : wave;
    const int64_t row = share == 1 ? (int64_t)blockIdx.y * 4 + wave : blockIdx.y, n = row < N ? row : N - 1;
    const int64_t t0 = (int64_t)blockIdx.x * ROW_TOKENS;
    const int Kw = (int)(K / 32), G = (int)(K / g), gw = (int)(g / 32);
    double acc[ROW_TOKENS];
#pragma unroll
    for (int t = 0; t < ROW_TOKENS; ++t) acc[t] = 0.0;
    uint32_t bits[8];
    float a[8];
    auto load = [&](int w) {
        const int grp = w / gw;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i < q) {
                bits[i] = packed[((int64_t)i * N + n) * Kw + w];
                a[i] = alpha[((int64_t)i * N + n) * G + grp];
            }
        }
    };
    const int first = sub * 64 + lane, step = 64 * share;
    if (first < Kw) load(first);
    for (int w = first; w < Kw; w += step) {
        Eight<XT> v[4];
        auto load_x = [&](int t) {
#pragma unroll
            for (int b = 0; b < 4; ++b) v[b].load(x + (t0 + t) * K + 32 * w + 8 * b);
        };
        load_x(0);  // in flight during the expansion
        double what[32];
#pragma unroll
        for (int j = 0; j < 32; ++j) what[j] = 0.0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i < q) {
                const double ad = (double)a[i];
                const uint32_t inv = ~bits[i];
#pragma unroll
                for (int j = 0; j < 32; ++j) what[j] += signed_value(ad, inv, j);
            }
        }
        if (w + step < Kw) load(w + step);  // in flight during the products
#pragma unroll
        for (int t = 0; t < ROW_TOKENS; ++t) {
            if (t0 + t < T) {
                if (t) load_x(t);
#pragma unroll
                for (int j = 0; j < 32; ++j) acc[t] = __builtin_fma((double)v[j >> 3].at(j & 7), what[j], acc[t]);
            }
        }
    }
    share_sums(part, acc, share);
    if (lane == 0 && sub == 0 && row < N)
#pragma unroll
        for (int t = 0; t < ROW_TOKENS; ++t)
            if (t0 + t < T) Elem<XT>::store(y + (t0 + t) * N + n, (float)acc[t]);
}

// Scale gradient: `share` waves per row n; a lane forms G[n][k] of its words over all tokens and adds it with the signs
// of every trained plane, one scale group after the other.
template <typename XT>
__global__ __launch_bounds__(256) void bwd_alpha_rows_kernel(const uint32_t* __restrict__ packed,
                                                             const XT* __restrict__ x, const XT* __restrict__ dy,
                                                             float* __restrict__ dalpha, int64_t T, int64_t N,
                                                             int64_t K, int64_t g, int q_train, float grad_scale,
                                                             int share) {
    __shared__ double part[4][8];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, sub = share == 1 ? 0 : wave;
    const int64_t row = share == 1 ? (int64_t)blockIdx.x * 4 + wave : blockIdx.x, n = row < N ? row : N - 1;
    const int Kw = (int)(K / 32), G = (int)(K / g), gw = (int)(g / 32);
    for (int grp = 0; grp < G; ++grp) {
        double s[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) s[i] = 0.0;
        for (int w = grp * gw + sub * 64 + lane; w < (grp + 1) * gw; w += 64 * share) {
            uint32_t inv[8];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (i < q_train) inv[i] = ~packed[((int64_t)i * N + n) * Kw + w];
            double gk[32];
#pragma unroll
            for (int j = 0; j < 32; ++j) gk[j] = 0.0;
            for (int64_t t = 0; t < T; ++t) {
                const double d = (double)Elem<XT>::load(dy + t * N + n);
                Eight<XT> v[4];
#pragma unroll
                for (int b = 0; b < 4; ++b) v[b].load(x + t * K + 32 * w + 8 * b);
#pragma unroll
                for (int j = 0; j < 32; ++j) gk[j] = __builtin_fma(d, (double)v[j >> 3].at(j & 7), gk[j]);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                if (i < q_train) {
#pragma unroll
                    for (int j = 0; j < 32; ++j) s[i] += signed_value(gk[j], inv[i], j);
                }
            }
        }
        if (grp && share > 1) __syncthreads();  // the previous group's sums have been read
        share_sums(part, s, share);
        if (lane == 0 && sub == 0 && row < N)
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (i < q_train) dalpha[((int64_t)i * N + n) * G + grp] = (float)((double)grad_scale * s[i]);
    }
}

// Input gradient for few rows n: a thread per column k and COL_TOKENS tokens, the rows in turn.
constexpr int COL_TOKENS = 8;
template <typename XT>
__global__ __launch_bounds__(256) void bwd_input_cols_kernel(const uint32_t* __restrict__ packed,
                                                             const float* __restrict__ alpha,
                                                             const XT* __restrict__ dy, XT* __restrict__ dx, int64_t T,
                                                             int64_t N, int64_t K, int64_t g, int q) {
    const int64_t k = (int64_t)blockIdx.y * 256 + threadIdx.x, t0 = (int64_t)blockIdx.x * COL_TOKENS;
    if (k >= K) return;
    const int64_t Kw = K / 32, G = K / g;
    const uint32_t* word = packed + (k >> 5);
    const float* scale = alpha + k / g;
    const int bit = (int)(k & 31);
    double acc[COL_TOKENS];
#pragma unroll
    for (int t = 0; t < COL_TOKENS; ++t) acc[t] = 0.0;
    for (int64_t n = 0; n < N; ++n) {
        double what = 0.0;
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (i < q) what += signed_scale(scale[((int64_t)i * N + n) * G], ~word[((int64_t)i * N + n) * Kw], bit);
#pragma unroll
        for (int t = 0; t < COL_TOKENS; ++t)
            if (t0 + t < T) acc[t] = __builtin_fma((double)Elem<XT>::load(dy + (t0 + t) * N + n), what, acc[t]);
    }
#pragma unroll
    for (int t = 0; t < COL_TOKENS; ++t)
        if (t0 + t < T) Elem<XT>::store(dx + (t0 + t) * K + k, (float)acc[t]);
}

// The lines, from 24 layers at 1 .. 6000 tokens with both sides timed (matrix instruction / vector ALU, us, fp32).
// Forward: 256 x 16384, q = 2, 1 token 74 / 6, 4 tokens 48 / 8; 10000 x 4096, q = 3, 1 token 57 / 28, 4 tokens 58 / 77;
// q = 8, 4 tokens 180 / 108; 1500 x 4096 at 4 tokens 18 / 15, at 8 19 / 23; 3 x 4096 at 2048 tokens 19 / 18.  bf16, whose
// activations are half the reads: 1500 x 4096, q = 1, 8 tokens 1.7 times as fast, 10000 x 4096, 8 tokens 0.85 times.
// Lanes hold whole words: below 24 of them most of a wave idles (400 x 256, 4 tokens, q = 4 4.2 / 8.5; 384 columns, 1 token
// 4.7 / 4.4, 4 tokens 4.8 / 5.7; 768 columns, 4 tokens 7.5 / 5.9; one plane, 8 tokens of 700 x 768 5.6 / 6.6).
static bool fwd_rows_ok(int64_t T, int64_t N, int64_t K, int q, bool fp32) {
    const int64_t jobs = N * T;
    if (K < 768) return K >= 384 && T <= (K >= 512 ? 2 : 1) && jobs <= 1500;
    if (T == 1 || jobs <= (K < 1408 ? 4096 : 6000)) return true;
    if (K < 1408) return false;
    if (T <= (fp32 && q <= 4 ? 2 : 4)) return true;
    return fp32 ? K >= 8192 && jobs <= 8200 : K >= 4096 && jobs <= 20000;
}
// Scale gradient, row-wise or long groups: 256 x 16384 at 8 tokens 65 / 18; 10000 x 4096, all of 8 planes, 2 tokens 133 / 78,
// one plane 4 tokens 41 / 72; 1500 x 4096, one plane, 3 tokens 16 / 15, 8 tokens 17 / 27.
// 400 x 256, one plane, 8 tokens 5.3 / 7.5; 384 columns, 4 tokens 5.3 / 5.1.
static bool bwd_alpha_rows_ok(int64_t T, int64_t N, int64_t K, int64_t g, int q_train) {
    if (K < 384 || (g != K && g < 2048)) return false;
    return T == 1 || (T <= (K >= 768 ? 8 : 4) && N * T <= 5000) || T <= (q_train > 4 ? 4 : q_train > 2 && K >= 1408 ? 2 : 1);
}
// Input gradient: the threads of few rows must fill the chip.  7 x 16384, q = 1, 4 tokens 3.8 / 4.5, 17 tokens 8.2 / 5.9,
// 6000 tokens 1237 / 198; 16 x 4096 at 64 tokens 5.6 / 11, at 333 22 / 12; 24 x 1024 at 333 tokens 6 / 10, at 2048 29 / 18;
// 33 x 4096, q = 3, 333 tokens 0.8 times as fast, 2048 tokens 1.1 times.  More planes move the line up (12 x 512, 1024 tokens,
// q = 1 1.05 times as fast, q = 8 0.76 times; 32 x 1024, 4096 tokens, q = 8 73 / 83), a second run of 32 rows for the
// matrix form moves it down (36 x 1024, 4096 tokens, q = 1 56 / 43).
static bool bwd_input_cols_ok(int64_t T, int64_t N, int64_t K, int q) {
    return N == 1 || (N <= (q > 4 ? 27 : 40) && T * K >= (3750 * (7 + q) * N + 50 * N * N * N) / (N > 32 ? 2 : 1));
}
// waves per row: all four of a workgroup while the rows alone leave compute units idle
static int row_share(int64_t jobs, int64_t words) { return jobs < 1024 && words >= 128 ? 4 : 1; }

// Token tiles per workgroup: one more halves the reads of the planes and the work of summing them, but also the
// number of workgroups; more than one only when at least one workgroup per compute unit is left.
static int token_tiles(int64_t T, int64_t column_tiles) {
    for (int tt = 4; tt > 1; tt /= 2)
        if (T > 8 * tt && ((T + 16 * tt - 1) / (16 * tt)) * column_tiles >= 256) return tt;
    return 1;
}

template <typename XT>
static hipError_t fwd_typed(const uint32_t* packed, const float* alpha, const XT* x, int64_t T, int64_t N, int64_t K,
                            int64_t g, int q, XT* y, hipStream_t st) {
    if (fwd_rows_ok(T, N, K, q, sizeof(XT) == 4)) {
        const int64_t tiles = (T + ROW_TOKENS - 1) / ROW_TOKENS;
        const int share = row_share(N * tiles, K / 32);
        BCQ_LAUNCH(fwd_rows_kernel<XT>, dim3((unsigned)tiles, (unsigned)((N * share + 3) / 4)), dim3(256), 0, st, packed,
                           alpha, x, y, T, N, K, g, q, share);
        return hipGetLastError();
    }
    const int64_t nb = (N + 15) / 16;
    const int tt = token_tiles(T, nb);
    dim3 grid((unsigned)((T + 16 * tt - 1) / (16 * tt)), (unsigned)nb), block(GEN_WAVES * 64);
    if (tt == 4)
        BCQ_LAUNCH((fwd_generic_kernel<XT, 4>), grid, block, 0, st, packed, alpha, x, y, T, N, K, g, q);
    else if (tt == 2)
        BCQ_LAUNCH((fwd_generic_kernel<XT, 2>), grid, block, 0, st, packed, alpha, x, y, T, N, K, g, q);
    else
        BCQ_LAUNCH((fwd_generic_kernel<XT, 1>), grid, block, 0, st, packed, alpha, x, y, T, N, K, g, q);
    return hipGetLastError();
}

template <typename XT>
static hipError_t bwd_input_typed(const uint32_t* packed, const float* alpha, const XT* dy, int64_t T, int64_t N,
                                  int64_t K, int64_t g, int q, XT* dx, hipStream_t st) {
    if (bwd_input_cols_ok(T, N, K, q)) {
        dim3 cols((unsigned)((T + COL_TOKENS - 1) / COL_TOKENS), (unsigned)((K + 255) / 256));
        BCQ_LAUNCH(bwd_input_cols_kernel<XT>, cols, dim3(256), 0, st, packed, alpha, dy, dx, T, N, K, g, q);
        return hipGetLastError();
    }
    const int64_t kb = K / 32;
    const int tt = token_tiles(T, kb);
    const int64_t tiles = (T + 16 * tt - 1) / (16 * tt);
    const bool half = tt == 1 && tiles * kb < 256;  // half a packed word per workgroup fills the chip sooner
    dim3 grid((unsigned)tiles, (unsigned)(half ? 2 * kb : kb)), block(GEN_WAVES * 64);
    if (half)
        BCQ_LAUNCH((bwd_input_generic_kernel<XT, 1, 1>), grid, block, 0, st, packed, alpha, dy, dx, T, N, K, g, q);
    else if (tt == 1)
        BCQ_LAUNCH((bwd_input_generic_kernel<XT, 1, 2>), grid, block, 0, st, packed, alpha, dy, dx, T, N, K, g, q);
    else  // two token tiles: four do not fit 64 KiB of tiles next to two column tiles
        BCQ_LAUNCH((bwd_input_generic_kernel<XT, 2, 2>), dim3((unsigned)((T + 31) / 32), (unsigned)kb), block, 0, st,
                           packed, alpha, dy, dx, T, N, K, g, q);
    return hipGetLastError();
}

template <typename XT>
static hipError_t bwd_alpha_typed(const uint32_t* packed, const XT* x, const XT* dy, int64_t T, int64_t N, int64_t K,
                                  int64_t g, int q_train, float grad_scale, float* dalpha, hipStream_t st) {
    if (bwd_alpha_rows_ok(T, N, K, g, q_train)) {
        const int share = row_share(N, g / 32);
        BCQ_LAUNCH(bwd_alpha_rows_kernel<XT>, dim3((unsigned)((N * share + 3) / 4)), dim3(256), 0, st, packed, x, dy,
                           dalpha, T, N, K, g, q_train, grad_scale, share);
        return hipGetLastError();
    }
    int per = GEN_WAVES;  // waves per scale group
    while (per > 1 && per * (K / g) > GEN_WAVES) per /= 2;
    BCQ_LAUNCH(bwd_alpha_generic_kernel<XT>, dim3((unsigned)((N + 15) / 16)), dim3(GEN_WAVES * 64), 0, st, packed, x,
                       dy, dalpha, T, N, K, g, q_train, grad_scale, per);
    return hipGetLastError();
}

hipError_t launch_fwd_generic(const uint32_t* packed, const float* alpha, const void* x, int dtype, int64_t T,
                              int64_t N, int64_t K, int64_t g, int q, void* y, hipStream_t st) {
    if (dtype == 0) return fwd_typed(packed, alpha, (const float*)x, T, N, K, g, q, (float*)y, st);
    return fwd_typed(packed, alpha, (const bf16_t*)x, T, N, K, g, q, (bf16_t*)y, st);
}

hipError_t launch_bwd_alpha_generic(const uint32_t* packed, const void* x, const void* dy, int dtype, int64_t T,
                                    int64_t N, int64_t K, int64_t g, int q, int q_train, float grad_scale,
                                    float* dalpha, hipStream_t st) {
    (void)q;
    if (dtype == 0)
        return bwd_alpha_typed(packed, (const float*)x, (const float*)dy, T, N, K, g, q_train, grad_scale, dalpha, st);
    return bwd_alpha_typed(packed, (const bf16_t*)x, (const bf16_t*)dy, T, N, K, g, q_train, grad_scale, dalpha, st);
}

hipError_t launch_bwd_input_generic(const uint32_t* packed, const float* alpha, const void* dy, int dtype,
                                    int64_t T, int64_t N, int64_t K, int64_t g, int q, void* dx, hipStream_t st) {
    if (dtype == 0) return bwd_input_typed(packed, alpha, (const float*)dy, T, N, K, g, q, (float*)dx, st);
    return bwd_input_typed(packed, alpha, (const bf16_t*)dy, T, N, K, g, q, (bf16_t*)dx, st);
}

}  // namespace bcq

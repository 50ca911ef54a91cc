// Forward of the BCQ linear layer for a few hundred tokens at most, in one kernel (bf16 in, fp32 accumulate, q <= 4).
//
// AlphaTuning Eq. 2 as one contraction with What = sum_i alpha_i B_i rounded once to bf16 (Eq. 1), like the two-kernel
// path of bcq_mfma.hip, but What never reaches memory: every wave expands the sign planes of its 32 rows straight into
// the registers of v_mfma_f32_32x32x16_bf16 and multiplies them with all the tokens of its tile.  At these token counts
// the two-kernel path is bound by writing and re-reading 16 bits per weight, here a weight costs q bits.
//
// Expansion by table (bcq_expand.h): from 64 tokens on the matrix instructions take longer than it.
//
// Split: a workgroup owns 32 rows x 32 TT tokens; its W waves take runs of 128 columns in turn and add their tiles
// through LDS in wave order (deterministic).  Up to 32 tokens are read from their rows; more are first rewritten in
// operand order, because a wave's 16-byte pieces of 32 rows would touch 32 cache lines per load (256 tokens of
// 10240 x 2560: 80 us from the rows, 41 us in order).  What bounds it: up to 32 tokens the planes' scattered rows and launch
// latency (6144 x 2048, groups of 128, 4 tokens: 26 -> 9 us against two kernels), above that the activation fragments,
// which every 32 rows read again from L2 through the vector memory path.
#include "bcq_expand.h"

namespace bcq {

typedef __attribute__((ext_vector_type(16))) float fu_f32x16;

// Activations -> the order the matrix instruction reads them in: for every 32-token tile, 32-column word and half slice
// one contiguous KiB, lane (t, h) holding columns 16 h + 8 sub .. + 7 of the word.  Tokens beyond T become zeros.
// A wave takes 8 tokens x 128 bytes: whole lines in, 128-byte runs out.
__global__ __launch_bounds__(256) void order_act_kernel(const bf16_t* __restrict__ x, int64_t T, int64_t K,
                                                        u32x4* __restrict__ xfrag) {
    const int lane = threadIdx.x & 63;
    const int64_t Kw = K / 32, pairs = (Kw + 1) / 2;
    const int64_t job = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);  // (eight tokens, two words)
    const int64_t t = (job / pairs) * 8 + (lane & 7), w = (job % pairs) * 2 + (lane >> 5);
    const int chunk = (lane >> 3) & 3;
    if (w >= Kw || t >= (T + 31) / 32 * 32) return;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (t < T) v = *reinterpret_cast<const u32x4*>(x + t * K + 32 * w + 8 * chunk);
    xfrag[(((t / 32) * Kw + w) * 2 + (chunk & 1)) * 64 + (t % 32) + 32 * (chunk >> 1)] = v;
}

// GROUPED: group-wise scales (the table follows the group); else one table per row.
// ORDERED: x is the output of order_act_kernel; else row-major.
template <int Q, int TT, int W, bool GROUPED, bool ORDERED>
__global__ __launch_bounds__(64 * W) void fused_fwd_kernel(const uint32_t* __restrict__ packed,
                                                           const float* __restrict__ alpha, const bf16_t* __restrict__ x,
                                                           bf16_t* __restrict__ y, int64_t T, int64_t N, int64_t K,
                                                           int64_t g, int per, float* __restrict__ sums) {
    __shared__ f32x4 part[2][W][4][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 31, h = lane >> 5;
    const int64_t n0 = (int64_t)blockIdx.x * 32, t0 = (int64_t)blockIdx.y * (32 * TT);
    const int64_t n = n0 + col < N ? n0 + col : N - 1;  // rows and tokens beyond the edge are computed, never stored
    const int Kw = (int)(K / 32), G = (int)(K / g), gw = (int)(g / 32);
    // this workgroup's units of 128 columns: part blockIdx.z of `per` each (all of them when the contraction is not split)
    const int first = (int)blockIdx.z * per + wave;
    const int units = min((Kw + 3) / 4, (int)(blockIdx.z + 1) * per);

    const uint32_t* prow[Q];
    const float* arow[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        prow[i] = packed + ((int64_t)i * N + n) * Kw;
        arow[i] = alpha + ((int64_t)i * N + n) * G;
    }
    // of a 32-column word, lane half h contracts over columns 16 h .. 16 h + 15
    const bf16_t* xrow[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
        if (ORDERED) {
            const int64_t tile = t0 / 32 + tt, tiles = (T + 31) / 32;
            xrow[tt] = x + (tile < tiles ? tile : tiles - 1) * K * 32 + lane * 8;
        } else {
            const int64_t t = t0 + tt * 32 + col;
            xrow[tt] = x + (t < T ? t : T - 1) * K + 16 * h;
        }
    }
    fu_f32x16 acc[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[tt][v] = 0.f;

    // In flight per wave: the planes (and scales of group-wise calls) D units ahead, the activations XW words ahead.
    // One token tile: one unit, so that four waves fit a SIMD (two units ahead: 8.7 -> 12 us for 6144 x 2048 at 4 tokens).
    constexpr int D = TT == 1 ? 1 : 2, XW = TT == 2 ? 4 : 2;
    uint32_t bits[D][Q][4];
    float a[D][2][Q];  // [unit][pair of words]
    auto load_bits = [&](int u, int buf) {
        if (4 * u + 4 <= Kw) {
#pragma unroll
            for (int i = 0; i < Q; ++i) __builtin_memcpy(bits[buf][i], prow[i] + 4 * u, 16);
        } else {
#pragma unroll
            for (int i = 0; i < Q; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) bits[buf][i][j] = 4 * u + j < Kw ? prow[i][4 * u + j] : 0u;
        }
    };
    auto load_alpha = [&](int w, float (&dst)[Q]) {
        const int grp = GROUPED ? (w < Kw ? w : Kw - 1) / gw : 0;
#pragma unroll
        for (int i = 0; i < Q; ++i) dst[i] = arow[i][grp];
    };
    auto load_unit = [&](int u, int buf) {
        load_bits(u, buf);
        if (GROUPED) {
            load_alpha(4 * u, a[buf][0]);
            load_alpha(4 * u + 2, a[buf][1]);
        }
    };
    u32x4 xf[XW][2][TT];  // [word][slice][token tile]
    const u32x4 zero = {0u, 0u, 0u, 0u};
    auto load_x = [&](int w, int slot) {  // words beyond K contribute nothing
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt)
                xf[slot][sub][tt] = w < Kw ? *reinterpret_cast<const u32x4*>(
                                                 xrow[tt] + (ORDERED ? (2 * w + sub) * 512 : 32 * w + 8 * sub)) : zero;
    };
    LevelTable<Q> table;
    // the two words of a pair may lie in two groups (g = 32): then the table is rebuilt between them
    const bool split = GROUPED && (gw & 1);
    const uint32_t half_sel = h ? 0x07060302u : 0x05040100u;

    auto clamp_unit = [&](int u) { return u < units ? u : units - 1; };
    load_unit(clamp_unit(first), 0);
    if (!GROUPED) load_alpha(0, a[0][0]);
#pragma unroll
    for (int j = 0; j < XW; ++j) load_x(4 * clamp_unit(first) + j, j);
    if (D == 2) load_unit(clamp_unit(first + W), D - 1);
    if (!GROUPED) table.build(a[0][0]);

    auto unit = [&](int u, int buf) {
        uint32_t own[2][Q];  // this lane half's 2 x 16 signs of each pair of words
        LevelTable<Q> tables[2];
#pragma unroll
        for (int pr = 0; pr < 2; ++pr) {
#pragma unroll
            for (int i = 0; i < Q; ++i)
                own[pr][i] = __builtin_amdgcn_perm(bits[buf][i][2 * pr + 1], bits[buf][i][2 * pr], half_sel);
            if (GROUPED) tables[pr].build(a[buf][pr]);
        }
        load_unit(clamp_unit(u + D * W), buf);
#pragma unroll
        for (int pr = 0; pr < 2; ++pr) {
            if (4 * u + 2 * pr < Kw) {
                u32x4 frag[4];
                expand32<Q>(own[pr], GROUPED ? tables[pr] : table, frag);
                if (split) {
                    u32x4 second[4];
                    float as[Q];
                    load_alpha(4 * u + 2 * pr + 1, as);
                    if (4 * u + 2 * pr + 1 >= Kw) {  // no such columns: zero weights, as Inf times a zero activation is NaN
#pragma unroll
                        for (int i = 0; i < Q; ++i) as[i] = 0.f;
                    }
                    table.build(as);
                    expand32<Q>(own[pr], table, second);
                    frag[2] = second[2];
                    frag[3] = second[3];
                }
                if (!GROUPED && 4 * u + 2 * pr + 1 >= Kw) {  // the same for row-wise scales
                    frag[2] = zero;
                    frag[3] = zero;
                }
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    constexpr int MASK = XW - 1;
                    const int slot = (2 * pr + j) & MASK;
#pragma unroll
                    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
                        for (int tt = 0; tt < TT; ++tt)
                            acc[tt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                __builtin_bit_cast(bf16x8, frag[2 * j + sub]),
                                __builtin_bit_cast(bf16x8, xf[slot][sub][tt]), acc[tt], 0, 0, 0);
                    if (XW == 2 && pr == 0)
                        load_x(4 * u + 2 + j, slot);
                    else
                        load_x(4 * clamp_unit(u + W) + 2 * pr + j - (XW == 2 ? 2 : 0), slot);
                }
            }
        }
    };
    for (int u = first; u < units; u += D * W) {
        unit(u, 0);
        if (D == 2 && u + W < units) unit(u + W, D - 1);
    }

    // accumulator register 4 gg + e of lane l: row n0 + 8 gg + 4 (l / 32) + e, token l % 32
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
#pragma unroll
        for (int gg = 0; gg < 4; ++gg)
            part[tt & 1][wave][gg][lane] = f32x4{acc[tt][4 * gg], acc[tt][4 * gg + 1], acc[tt][4 * gg + 2], acc[tt][4 * gg + 3]};
        __syncthreads();  // two buffers: the sums of tile tt are read while tile tt + 1 is written
        if (threadIdx.x < 256) {
            const int gg = threadIdx.x >> 6;
            f32x4 s = part[tt & 1][0][gg][lane];
#pragma unroll
            for (int w = 1; w < W; ++w) s += part[tt & 1][w][gg][lane];
            const int64_t t = t0 + tt * 32 + col, nn = n0 + 8 * gg + 4 * h;
            if (sums) {  // split contraction: sum_parts_kernel adds the parts
                if (t < T && nn < N)
                    *reinterpret_cast<f32x4*>(sums + ((int64_t)blockIdx.z * T + t) * ((N + 3) / 4 * 4) + nn) = s;
            } else if (t < T) {
                bf16_t* dst = y + t * N + nn;
                if (nn + 3 < N && (N & 3) == 0) {
                    *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16x2(s[0], s[1]), pack_bf16x2(s[2], s[3]));
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (nn + e < N) dst[e] = f32_to_bf16(s[e]);
                }
            }
        }
    }
}

// y[t][n] = sum of the parts, in order; a thread adds four rows n of one token
__global__ __launch_bounds__(256) void sum_parts_kernel(const float* __restrict__ sums, int parts, int64_t T, int64_t N,
                                                        bf16_t* __restrict__ y) {
    const int64_t quads = (N + 3) / 4, idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= T * quads) return;
    const f32x4* p = reinterpret_cast<const f32x4*>(sums) + idx;
    f32x4 s = p[0];
    for (int i = 1; i < parts; ++i) s += p[i * T * quads];
    const int64_t t = idx / quads, n = idx % quads * 4;
    bf16_t* dst = y + t * N + n;
    if ((N & 3) == 0) {
        *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16x2(s[0], s[1]), pack_bf16x2(s[2], s[3]));
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (n + e < N) dst[e] = f32_to_bf16(s[e]);
    }
}

static size_t order_bytes(int64_t T, int64_t K) { return T <= 32 ? 0 : (size_t)((T + 31) / 32 * 32 * K * 2); }
static size_t sums_bytes(int64_t T, int64_t N, int parts) { return (size_t)parts * T * ((N + 3) / 4 * 4) * 4; }

// 128 tokens per workgroup read and expand every plane half as often, 64 make twice as many workgroups: measured
// (256 tokens, q = 4) 7680 x 2560 27 against 31 us, 10240 x 2560 35 / 38, 2560 x 2560 17 / 17, 1024 x 1024 10 / 8, and
// with the contraction split 2560 x 10240 48 / 53.
static bool wide_tokens(int64_t T, int64_t N, int64_t K) {
    const int64_t tiles = (N + 31) / 32 * ((T + 127) / 128), units = (K + 127) / 128;
    return T > 64 && (tiles >= 256 || (tiles >= 64 && units >= 64));
}

template <int Q, bool GROUPED>
static hipError_t launch_q(const uint32_t* packed, const float* alpha, const bf16_t* x, int64_t T, int64_t N, int64_t K,
                           int64_t g, bf16_t* y, void* workspace, hipStream_t st) {
    const unsigned cols = (unsigned)((N + 31) / 32);
    const int units = (int)((K + 127) / 128);
    const bf16_t* xo = x;
    if (T > 32) {
        const int64_t jobs = (T + 31) / 32 * 4 * ((K / 32 + 1) / 2);
        BCQ_LAUNCH(order_act_kernel, dim3((unsigned)((jobs + 3) / 4)), dim3(256), 0, st, x, T, K, (u32x4*)workspace);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        xo = (const bf16_t*)workspace;
    }
    const bool wide = wide_tokens(T, N, K);
    const int W = T <= 32 ? 8 : 4, tile = T <= 32 ? 32 : wide ? 128 : 64;
    const unsigned tiles = (unsigned)((T + tile - 1) / tile);
    // Few rows and a long contraction: parts of it go to workgroups of their own while they still find an idle compute
    // unit and every wave keeps a unit (2048 x 8192, groups of 128, 4 tokens: 25.2 -> 12.5 us, 1024 x 4096 at 32 tokens
    // 16.5 -> 9.7; below 2048 columns the extra launch costs more, 1024 x 1024 at 96 tokens 8 -> 9).
    int parts = 1;
    while (units >= 16 && cols * tiles * parts * 2 <= (wide ? 512u : 256u) && units >= 2 * W * parts &&
           order_bytes(T, K) + sums_bytes(T, N, 2 * parts) <= mfma_fwd_workspace(N, K))
        parts *= 2;
    const int per = (units + parts - 1) / parts;
    parts = (units + per - 1) / per;
    float* sums = parts > 1 ? reinterpret_cast<float*>(static_cast<unsigned char*>(workspace) + order_bytes(T, K)) : nullptr;
    const dim3 grid(cols, tiles, (unsigned)parts), block(64 * W);
    if (T <= 32)
        BCQ_LAUNCH((fused_fwd_kernel<Q, 1, 8, GROUPED, false>), grid, block, 0, st, packed, alpha, xo, y, T, N, K, g, per,
                           sums);
    else if (wide)
        BCQ_LAUNCH((fused_fwd_kernel<Q, 4, 4, GROUPED, true>), grid, block, 0, st, packed, alpha, xo, y, T, N, K, g, per,
                           sums);
    else
        BCQ_LAUNCH((fused_fwd_kernel<Q, 2, 4, GROUPED, true>), grid, block, 0, st, packed, alpha, xo, y, T, N, K, g, per,
                           sums);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || parts == 1) return e;
    BCQ_LAUNCH(sum_parts_kernel, dim3((unsigned)((T * ((N + 3) / 4) + 255) / 256)), dim3(256), 0, st, sums, parts, T, N, y);
    return hipGetLastError();
}

// Row-wise scales, 129 to 384 tokens, large layers: whether the workgroups of the one-kernel forward run in one round and
// fill it (two of 128 tokens or one of 64 to a compute unit at a time).  A round that is half empty, or a second one, goes
// to two kernels; so do three tiles of 128 tokens.
static bool one_full_round(int64_t T, int64_t N, int64_t K, int q) {
    const int64_t cols = (N + 31) / 32;
    if (!wide_tokens(T, N, K)) return cols * ((T + 63) / 64) <= 256;
    const int64_t tiles = cols * ((T + 127) / 128);
    return T <= 256 && tiles <= 512 && tiles > (q == 4 ? 384 : 320);
}

// Where one kernel is faster than expanding What and multiplying.  Row-wise scales (65000 timings of both sides, 81 to 384 tokens,
// 0.05 to 100 million weights, q = 1 .. 4): up to 128 tokens one kernel.  Above that the planes are expanded again for
// every 128 tokens, which costs more than writing What once where the product alone fills the chip: above 40 million weights,
// and with four planes above 256 tokens from 8 million on, unless one_full_round (one kernel / two, us: 50257 x 1024 at 144
// tokens 64 / 53 (q = 1) and 76 / 57 (q = 4), 10240 x 2560, q = 4, 288 tokens 42 / 33; one full round 8191 x 7072, q = 2,
// 160 tokens 53 / 60, 1615 x 5120, q = 4, 320 tokens 25 / 28, and just beyond 1664 x 5120 29 / 25), and up to 100 million, from
// where What no longer fits the 256 MB cache in front of HBM (12288 x 12288, q = 3, 200 tokens 126 / 211, 16384 x 8192, q = 4,
// 256 tokens 119 / 161).  Of the 3574 timed calls beyond the first two sizes 22 go to the side that is more than 4 % slower
// (worst 1.17).  Below them one kernel is more than 4 %
// slower in 3 % of the calls up to 128 tokens, in 15 % up to 256 and in 48 % above (3072 x 1024, q = 4, 128 tokens 8.6 / 10.4,
// 256 12.0 / 10.5, 384 15.0 / 12.2).  Above 384 tokens two kernels.
// Group-wise scales: a unit of 128 columns also builds 2 tables of q loads and 2^(q - 1) sums, 4 when groups hold an odd
// number of words, for every 128 tokens (64 in small layers) again, so the line moves down with q and that parity (`level`),
// and less so where N K T is small and leaves the matrix product with few workgroups.  The line was set against an earlier,
// slower product: against the present one it takes the side that is more than 4 % slower in 26 % of 34440 calls and more than
// 10 % in 19 %, nearly always one kernel (10240 x 2560, g = 64, q = 2, 128 tokens 25 / 27, 256 37 / 31; q = 4, 128 tokens 36 / 29).
// The re-ordered activations of more than 32 tokens take the place of the expanded weights in the workspace.
bool fused_fwd_ok(int64_t T, int64_t N, int64_t K, int64_t g, int q) {
    if (q > 4 || T > 384 || order_bytes(T, K) > mfma_fwd_workspace(N, K)) return false;
    if (T <= 16) return true;
    if (g == K) {
        const bool large = (T > 128 && N * K > 40000000) || (T > 256 && q == 4 && N * K > 8000000);
        return !large || N * K > 100000000 || one_full_round(T, N, K, q);
    }
    const bool odd = (g / 32) % 2 != 0;
    const int level = q + (odd ? 1 : 0);
    const int64_t work = N * K * T;
    if (odd && q > 1 && T > 32 && N * K < 1200000) return false;  // 1024 x 1024, q = 4, 64 tokens: 14 / 11
    switch (level) {
        case 1: return true;
        case 2: return T <= 256 || (!odd && work <= 8000000000);
        case 5: return T <= 64 ? N <= 8192 : T <= 160 && N * T <= 320000;
        default: break;
    }
    if (T <= 128) return true;
    if (T <= 256) return odd ? N <= 4096 && work <= 1300000000 : work <= (level == 3 ? 4000000000 : 2500000000);
    return !odd && T <= 320 && work <= 800000000;
}

hipError_t launch_fwd_fused(const uint32_t* packed, const float* alpha, const void* x, int64_t T, int64_t N, int64_t K,
                            int64_t g, int q, void* y, void* workspace, hipStream_t st) {
    const bf16_t* xb = (const bf16_t*)x;
    bf16_t* yb = (bf16_t*)y;
#define BCQ_FUSED_GO(QQ)                                                                                 \
    if (g != K) return launch_q<QQ, true>(packed, alpha, xb, T, N, K, g, yb, workspace, st);             \
    return launch_q<QQ, false>(packed, alpha, xb, T, N, K, g, yb, workspace, st);
    switch (q) {
        case 1: BCQ_FUSED_GO(1)
        case 2: BCQ_FUSED_GO(2)
        case 3: BCQ_FUSED_GO(3)
        default: BCQ_FUSED_GO(4)
    }
#undef BCQ_FUSED_GO
}

}  // namespace bcq

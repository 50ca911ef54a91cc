// Forward of the BCQ linear layer for a few hundred tokens at most, in one kernel (bf16 in, fp32 accumulate, q <= 4).
//
// AlphaTuning Eq. 2 as one contraction with What = sum_i alpha_i B_i rounded once to bf16 (Eq. 1), like the two-kernel
// path of bcq_mfma.hip, but What never reaches memory: every wave expands the sign planes of its rows straight into
// the registers of the matrix instructions (by table, bcq_expand.h).  At these token counts the two-kernel path is bound by
// writing and re-reading 16 bits per weight, here a weight costs q bits.
//
// Two forms: group_fwd_kernel up to 32 tokens (16 rows to a workgroup, its waves share the contraction), tile_fwd_kernel above.
#include <type_traits>

#include "bcq_expand.h"

namespace bcq {

// Up to 32 tokens.  A workgroup owns 16 rows; a wave takes a segment of 128 WPL columns at a time, of which lane row h expands the WPL
// words 4 h WPL .. of its row (one group: WPL divides the words of a group), so that a plane costs one load and one scale per lane and
// segment, and adds into 16 rows x 16 TT tokens of v_mfma_f32_16x16x32_bf16.  The segment's activations go global -> LDS directly, a
// token's columns in a row, and stay with the wave; the waves' tiles meet in LDS and are added in wave order (deterministic).
// What bounds it: launch, one trip to memory and, in larger layers, the expansion's vector operations.  Groups of 128, q = 3, 4 tokens, us,
// against 32 rows to a workgroup and single words and scales per request (scattered requests bound that kernel): 6144 x 2048 10.4 -> 5.7,
// 2048 x 2048 7.2 and a sum of 2 -> 3.9, 8192 x 2048 10.5 -> 6.1, 2048 x 8192 10 and a sum of 3 -> 7.3; 16 tokens of 7680 x 2560 7.1, 32 8.8.
template <int Q, int WPL, int TT>
__global__ __launch_bounds__(1024) void group_fwd_kernel(const uint32_t* __restrict__ packed, const float* __restrict__ alpha,
                                                         const bf16_t* __restrict__ x, bf16_t* __restrict__ y, int T, int64_t N,
                                                         int K, int gw, uint32_t inverse, int segs, int per, int W, int stage,
                                                         float* __restrict__ sums) {
#if defined(__HIP_DEVICE_COMPILE__)  // the buffer-resource builtins exist in the device pass only
    constexpr int SLOTS = 16 * WPL, TPR = 4 / WPL;  // 16-byte pieces of a token's segment; tokens of a request
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int lane = threadIdx.x & 63, r = lane & 15, h = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t n0 = (int64_t)blockIdx.x * 16, left = N - 1 - n0;
    const int Kw = K / 32, G = Kw / gw;
    const int first = (int)blockIdx.y * per + wave, end = min(segs, (int)(blockIdx.y + 1) * per);

    // rows beyond the edge are computed, never stored; addresses are a uniform base and a 32-bit lane offset
    const uint32_t row = (uint32_t)(r < left ? r : left), roff = row * (uint32_t)Kw, aoff = row * (uint32_t)G;
    const uint32_t* const prow = packed + n0 * Kw;
    const float* const arow = alpha + n0 * G;
    const int64_t plane = N * Kw, splane = N * G;
    uint32_t bits[Q][WPL];
    float a[Q];
    auto request = [&](int s) {
        const int w0 = (4 * s + h) * WPL, wl = w0 < Kw ? w0 : Kw - WPL;  // words beyond K meet zero weights (WPL divides Kw)
#pragma unroll
        for (int i = 0; i < Q; ++i) __builtin_memcpy(bits[i], prow + i * plane + (roff + (uint32_t)wl), 4 * WPL);
        const uint32_t grp = inverse ? __umulhi((uint32_t)wl, inverse) : (uint32_t)wl;
#pragma unroll
        for (int i = 0; i < Q; ++i) a[i] = arow[i * splane + (aoff + grp)];
    };
    // activations: piece c (columns 8 c .. + 7) of a token lies at slot c ^ (token & 15) among its 16: the reads below touch every bank once
    unsigned char* const mine = smem + wave * stage;
    __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)x, 0, T * K * 2, 0x00020000);
    auto fetch = [&](int s) {
        const int slot = lane & (SLOTS - 1);
        for (int d = 0; d * TPR < T; ++d) {  // (requests of several tokens repeat the last one beyond T)
            const int tt = d * TPR + lane / SLOTS, t = tt < T ? tt : T - 1;
            const int col = 8 * (slot ^ (tt & 15));
            const uint32_t off = s * (128 * WPL) + col < K ? (uint32_t)(t * K + col) * 2u : 0x80000000u;  // beyond K: zeros
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (void __attribute__((address_space(3)))*)(mine + d * 1024), 16, off,
                                                     s * (256 * WPL), 0, 0);
        }
    };
    uint32_t base[TT], turn[TT];  // lane row h reads pieces 4 WPL h + 4 e + f of token r
#pragma unroll
    for (int i = 0; i < TT; ++i) {
        const int t = r + 16 * i < T ? r + 16 * i : T - 1;
        base[i] = (uint32_t)(t * 256 * WPL + (4 * WPL * h & ~15) * 16);
        turn[i] = (uint32_t)(((4 * WPL * h & 15) ^ (t & 15)) * 16);
    }
    f32x4 acc[TT];
#pragma unroll
    for (int i = 0; i < TT; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};

    if (first < end) {
        request(first);
        fetch(first);
    }
    for (int s = first; s < end; s += W) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        uint32_t w[WPL][Q];
#pragma unroll
        for (int i = 0; i < Q; ++i)
#pragma unroll
            for (int e = 0; e < WPL; ++e) w[e][i] = bits[i][e];
        LevelTable<Q> table;
        table.build(a);
        if ((4 * s + 4) * WPL > Kw) {  // zero weights beyond K, as Inf times a zero activation is NaN
            const uint32_t live = (4 * s + h) * WPL < Kw ? ~0u : 0u;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                table.lo[e] &= live;
                table.hi[e] &= live;
            }
        }
        if (s + W < end) request(s + W);
#pragma unroll
        for (int e = 0; e < WPL; ++e) {
            u32x4 xf[TT][4], frag[4];
#pragma unroll
            for (int i = 0; i < TT; ++i)
#pragma unroll
                for (int f = 0; f < 4; ++f)
                    xf[i][f] = *reinterpret_cast<const u32x4*>(mine + base[i] + (turn[i] ^ (uint32_t)((4 * e + f) * 16)));
            expand32<Q>(w[e], table, frag);
#pragma unroll
            for (int f = 0; f < 4; ++f)
#pragma unroll
                for (int i = 0; i < TT; ++i)
                    acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(frag[f]), as_bf16x8(xf[i][f]), acc[i], 0, 0, 0);
        }
        if (s + W < end) {  // every read of the stage has returned before its refill is asked for
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            fetch(s + W);
        }
    }

    f32x4* const own = reinterpret_cast<f32x4*>(mine) + lane;  // the wave's stage is free
#pragma unroll
    for (int i = 0; i < TT; ++i) own[64 * i] = acc[i];
    __syncthreads();
    for (int i = wave; i < TT; i += W) {
        const unsigned char* p = smem + (64 * i + lane) * 16;
        f32x4 s = *reinterpret_cast<const f32x4*>(p);
#pragma unroll 4
        for (int k = 1; k < W; ++k) s += *reinterpret_cast<const f32x4*>(p + k * stage);
        // register e of lane (r, h): row n0 + 4 h + e, token 16 i + r
        const int64_t t = 16 * i + r, n = n0 + 4 * h;
        if (t >= T || n >= N) continue;
        if (sums) {  // split contraction: sum_parts_kernel adds the parts
            *reinterpret_cast<f32x4*>(sums + ((int64_t)blockIdx.y * T + t) * ((N + 3) / 4 * 4) + n) = s;
        } else if ((N & 3) == 0) {
            *reinterpret_cast<uint2*>(y + t * N + n) = make_uint2(pack_bf16x2(s[0], s[1]), pack_bf16x2(s[2], s[3]));
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e < N) y[t * N + n + e] = f32_to_bf16(s[e]);
        }
    }
#endif
}

// ---- 33 tokens and more ---------------------------------------------------------------------------------------------
// expand32 in steps of eight columns of each byte pair, so that they can stand between matrix instructions
template <int Q>
struct Expansion {
    uint32_t neg, even, odd, c[Q > 1 ? Q - 1 : 1];
    __device__ __forceinline__ void begin(const uint32_t (&w)[Q]) {
        neg = ~w[Q - 1];
#pragma unroll
        for (int i = 0; i + 1 < Q; ++i) c[i] = w[i] ^ neg;
        even = odd = 0u;  // two-bit codes of the even and the odd columns
        if constexpr (Q >= 3) {
            even = (c[0] & 0x55555555u) | ((c[1] & 0x55555555u) << 1);
            odd = ((c[0] >> 1) & 0x55555555u) | (c[1] & 0xAAAAAAAAu);
        }
    }
    // register p of all four fragments (columns 2 p and 2 p + 1 of each byte)
    __device__ __forceinline__ void step(int p, const LevelTable<Q>& t, uint32_t (&frag)[4][4]) const {
        uint32_t ab[2], cd[2];
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            const int s = 2 * p + o;
            uint32_t sel = 0u;
            if constexpr (Q == 2) sel = (c[0] >> s) & 0x01010101u;
            if constexpr (Q >= 3) sel = ((o ? odd : even) >> (s & 6)) & 0x03030303u;
            if constexpr (Q == 4) sel |= (s >= 2 ? c[2] >> (s - 2) : c[2] << (2 - s)) & 0x04040404u;
            const uint32_t l = __builtin_amdgcn_perm(t.lo[1], t.lo[0], sel);
            const uint32_t h = __builtin_amdgcn_perm(t.hi[1], t.hi[0], sel) ^ ((neg << (7 - s)) & 0x80808080u);
            ab[o] = __builtin_amdgcn_perm(h, l, 0x05010400u);
            cd[o] = __builtin_amdgcn_perm(h, l, 0x07030602u);
        }
        frag[0][p] = __builtin_amdgcn_perm(ab[1], ab[0], 0x05040100u);
        frag[1][p] = __builtin_amdgcn_perm(ab[1], ab[0], 0x07060302u);
        frag[2][p] = __builtin_amdgcn_perm(cd[1], cd[0], 0x05040100u);
        frag[3][p] = __builtin_amdgcn_perm(cd[1], cd[0], 0x07060302u);
    }
};

constexpr int tile_wait(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }  // s_waitcnt vmcnt(n)

template <int TM, int KG>
constexpr int tile_stages() { return TM * KG <= 4 ? 3 : 2; }
template <int TM, int KG>
constexpr int tile_lds_bytes() { return KG * tile_stages<TM, KG>() * TM * 16 * 256; }

// A workgroup owns 64 TN rows x 16 TM tokens; its waves are four rows of 16 TN rows each, times KG parts of the contraction whose
// sums meet in LDS.  The activations of a unit of 128 columns go global -> LDS directly, NS - 1 units ahead, and come back as
// v_mfma_f32_16x16x32_bf16 operands; each wave expands the weights of the next unit between the matrix instructions of this one.
// A wave reads 16 bytes of a row and plane at a time, four lanes to a 64-byte piece, and a 4 x 4 transposition over the rows of
// lanes hands every lane the one word of each unit whose 32 columns it contracts over: slice f of a unit is columns
// 32 h + 8 f .. + 7 of lane row h on both sides.
//
// What bounds it: reading the activations from LDS.  With 16 rows to a wave every matrix instruction takes a fragment of its own, 1 KiB at the 145 B/ns
// that a compute unit's LDS sustains: 256 tokens, q = 4, 22.6 of 36 us for 10240 x 2560, 17.4 of 24 for 7680 x 2560.  Then start and end, and vector
// operations, 0.3 to 0.5 of the cycles (matrix instructions 0.2).  Expanding costs 22 (q = 1) to 110 (q = 4) of them per 32 weights, 4 cycles each, repeated for
// every 16 TM tokens, and beside a 16-cycle matrix instruction only two are free (7.2 ns alone and with two, 10.5 with four, 17 with
// eight).  Against activations re-ordered in memory and read from L2 by every 32 rows (us, with that kernel's re-ordering): 256 tokens,
// q = 4, of 7680 x 2560 27 -> 22, 2560 x 10240 44 -> 34, 10240 x 2560 35 -> 33; 149 tokens of 2560 x 10240, q = 1, 38 -> 21; groups
// of 32: 72 tokens of 8192 x 2048, q = 3, 26 -> 16.   (Calls that it made slower: at fused_fwd_ok.)
//
// Shapes (TM, TN, KG): (4, 1, 1), of which a compute unit holds three by their LDS and hides one's waits behind another's, and
// (8, 1, 2), which expands half as often.  128 rows to a workgroup (TN = 2), 128 or 256 tokens without the parts, and more stages
// for one workgroup less were slower or no more than 2 % faster over 74 shapes.
template <int Q, int TM, int KG, bool GROUPED>
__global__ __launch_bounds__(256 * KG, KG) void tile_fwd_kernel(const uint32_t* __restrict__ packed, const float* __restrict__ alpha,
                                                          const bf16_t* __restrict__ x, bf16_t* __restrict__ y, int64_t T,
                                                          int64_t N, int64_t K, int64_t g, int per, int token_tiles, int parts,
                                                          int items, float* __restrict__ sums) {
#if defined(__HIP_DEVICE_COMPILE__)  // the buffer-resource builtins exist in the device pass only
    constexpr int TN = 1, BM = 16 * TM, STAGE = BM * 256, NS = tile_stages<TM, KG>(), KD = BM / 16;  // KD: requests per wave and stage
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int lane = threadIdx.x & 63, r = lane & 15, h = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), kg = wave >> 2, wr = wave & 3;
    uint32_t item;
    if (!xcd_item((uint32_t)items, item)) return;
    // (divisions are done by the vector ALU: without readfirstlane the compiler takes everything after them for lane values)
    const int rest = __builtin_amdgcn_readfirstlane((int)(item / (uint32_t)token_tiles));
    const int row_tile = __builtin_amdgcn_readfirstlane((int)((uint32_t)rest / (uint32_t)parts)), part = rest - row_tile * parts;
    const int64_t t0 = (int64_t)((int)item - rest * token_tiles) * BM;
    const int64_t n0 = (int64_t)row_tile * (64 * TN) + wr * (16 * TN);
    const int Kw = (int)(K / 32), G = (int)(K / g), gw = (int)(g / 32);
    const int units = (Kw + 3) / 4, first = (part * KG + kg) * per;  // this wave's units of 128 columns: first .. first + per - 1

    // rows and tokens beyond the edge are computed, never stored; addresses are a uniform base and a 32-bit lane offset
    const int64_t nb = n0 < N ? n0 : N - 1;
    uint32_t roff[TN], aoff[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int64_t left = N - 1 - nb, row = 16 * j + r;
        roff[j] = (uint32_t)((row < left ? row : left) * Kw);
        aoff[j] = (uint32_t)((row < left ? row : left) * G);
    }
    const uint32_t* const prow = packed + nb * Kw;
    const float* const arow = alpha + nb * G;
    const int64_t plane = N * Kw, splane = N * G;

    // Activations: unit -> LDS as rows of 256 bytes, chunk (h, f) = columns 32 h + 8 f .. + 7 at 16-byte slot (h + 4 f) ^ (token & 15):
    // the fragment reads below then touch every bank once.
    __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)x, 0, (int)(T * K * 2), 0x00020000);
    uint32_t voff[KD];
    const int row4 = 4 * wr + h, code = r ^ row4;  // token of the request modulo 16; its chunk
    const int ccol = 32 * (code & 3) + 8 * (code >> 2);
#pragma unroll
    for (int k = 0; k < KD; ++k) {
        const int64_t t = t0 + 16 * k + row4;
        voff[k] = (uint32_t)((t < T ? t : T - 1) * K * 2 + 2 * ccol);
    }
    const uint32_t tail = (int64_t)(units - 1) * 128 + ccol < K ? 0u : 0x80000000u;  // beyond the descriptor: zeros
    auto dma = [&](int v, int slot) {  // (requests beyond this wave's units go nowhere: the waits count them)
        const int u = first + v;
        const uint32_t off = u >= units || v >= per ? 0x80000000u : u == units - 1 ? tail : 0u;
        const int soff = __builtin_amdgcn_readfirstlane(u < units ? u * 256 : 0);
#pragma unroll
        for (int k = 0; k < KD; ++k)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rx, (void __attribute__((address_space(3)))*)(smem + (kg * NS + slot) * STAGE + (4 * k + wr) * 1024), 16,
                voff[k] + off, soff, 0, 0);
    };
    // signs: lane row h reads words 4 h .. + 3 of 16, and keeps word h of each unit after the transposition
    uint32_t bits[TN][Q][4];
    const bool quad = (Kw & 3) == 0;
    auto load_bits = [&](int v) {
        const int w0 = 4 * (first + v) + 4 * h;  // words beyond K meet zero weights
        if (quad) {
            const uint32_t w = (uint32_t)(w0 < Kw ? w0 : Kw - 4);
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int i = 0; i < Q; ++i) __builtin_memcpy(bits[j][i], prow + i * plane + (roff[j] + w), 16);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t w = (uint32_t)(w0 + e < Kw ? w0 + e : Kw - 1);
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int i = 0; i < Q; ++i) bits[j][i][e] = prow[i * plane + (roff[j] + w)];
            }
        }
    };
    float a[TN][Q];
    auto load_alpha = [&](int v) {
        const int w = 4 * (first + v) + h, grp = GROUPED ? (w < Kw ? w : Kw - 1) / gw : 0;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int i = 0; i < Q; ++i) a[j][i] = arow[i * splane + (aoff[j] + (uint32_t)grp)];
    };
    LevelTable<Q> table[TN];
    auto tables = [&](int v) {  // of unit v; words beyond K have zero weights, as Inf times a zero activation is NaN
        if (GROUPED) {
#pragma unroll
            for (int j = 0; j < TN; ++j) table[j].build(a[j]);
        }
        if (4 * (first + v) + 4 > Kw) {  // (and so have all units from here on)
            const uint32_t live = 4 * (first + v) + h < Kw ? ~0u : 0u;
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    table[j].lo[e] &= live;
                    table[j].hi[e] &= live;
                }
        }
    };

    f32x4 acc[TN][TM];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < TM; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    uint32_t frag[2][TN][4][4];  // [buffer][row tile][slice][register]
    u32x4 xf[2][4];
    uint32_t xoff[4];
#pragma unroll
    for (int f = 0; f < 4; ++f) xoff[f] = (uint32_t)(kg * NS * STAGE + r * 256 + (((h + 4 * f) ^ r) * 16));
    auto read_x = [&](int slot, int grp) {  // group of four token tiles of a slice: slice grp / (TM / 4)
        const int f = grp / (TM / 4), i0 = grp % (TM / 4) * 4;
        const uint32_t addr = xoff[f] + (uint32_t)(slot * STAGE);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(xf[grp & 1][i]) : "v"(addr), "n"((i0 + i) * 4096));
    };
    auto arrived = [&](int p) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(xf[p][i]));
        __builtin_amdgcn_sched_barrier(0);
    };
    Expansion<Q> ex[TN];
    uint32_t pair[TN][Q][2];  // the words of an even unit and the one after it
    auto take = [&](int at) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int i = 0; i < Q; ++i)
#pragma unroll
                for (int e = 0; e < 2; ++e) pair[j][i][e] = bits[j][i][at + e];
    };
    auto turn = [&] {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int i = 0; i < Q; ++i) transpose_rows(bits[j][i]);
    };
    auto begin = [&](int e) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            uint32_t w[Q];
#pragma unroll
            for (int i = 0; i < Q; ++i) w[i] = pair[j][i][e];
            ex[j].begin(w);
        }
    };
    auto handover = [&] {
        asm volatile("s_waitcnt %0" ::"n"(tile_wait((NS - 2) * KD)) : "memory");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    auto keep_frag = [&](int b, int j, int p) {  // computed here, not moved behind a branch to where it is used
#pragma unroll
        for (int e = 0; e < 4; ++e) asm volatile("" : "+v"(frag[b][j][e][p]));
    };
    // Unit v: multiply with its weights (buffer `cur`) while those of unit v + 1 are expanded between the matrix instructions.
    auto unit = [&](int slot, auto CUR) {
        constexpr int cur = decltype(CUR)::value, nxt = 1 - cur;
        constexpr int NGRP = TM, NP = 4 * TN;
#pragma unroll
        for (int grp = 0; grp < NGRP; ++grp) {
            arrived(grp & 1);
            if (grp + 1 < NGRP) read_x(slot, grp + 1);
            __builtin_amdgcn_sched_barrier(0);
            const int f = grp / (TM / 4), i0 = grp % (TM / 4) * 4;
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[j][i0 + i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        as_bf16x8(u32x4{frag[cur][j][f][0], frag[cur][j][f][1], frag[cur][j][f][2], frag[cur][j][f][3]}),
                        as_bf16x8(xf[grp & 1][i]), acc[j][i0 + i], 0, 0, 0);
#pragma unroll
            for (int p = 0; p < NP; ++p)
                if (p * NGRP / NP == grp) {
                    ex[p / 4].step(p % 4, table[p / 4], frag[nxt][p / 4]);
                    keep_frag(nxt, p / 4, p % 4);
                }
#pragma unroll
            for (int m = 0; m < 4 * TN; ++m) {
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x2, 4, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        handover();
    };

#pragma unroll
    for (int v = 0; v < NS - 1; ++v) dma(v, v);
    load_bits(0);
    load_alpha(0);
    if (!GROUPED) {
#pragma unroll
        for (int j = 0; j < TN; ++j) table[j].build(a[j]);
    }
    turn();
    take(0);
    tables(0);
    if (GROUPED) load_alpha(1);
    begin(0);
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int p = 0; p < 4; ++p) ex[j].step(p, table[j], frag[0][j]);
    handover();
    auto after = [](int slot) { return slot + 1 == NS ? 0 : slot + 1; };
    int s0 = 0, s1 = after(0), last = NS - 1;  // stages of units v, v + 1, v - 1
    for (int v = 0; v < per; v += 2) {
        read_x(s0, 0);
        dma(v + NS - 1, last);
        if (v & 2) load_bits(v + 2);
        tables(v + 1);
        if (GROUPED) load_alpha(v + 2);
        begin(1);
        unit(s0, std::integral_constant<int, 0>{});
        read_x(s1, 0);
        dma(v + NS, s0);
        if (v & 2) {
            turn();
            take(0);
        } else {
            take(2);
        }
        tables(v + 2);
        if (GROUPED) load_alpha(v + 3);
        begin(0);
        unit(s1, std::integral_constant<int, 1>{});
        last = s1;
        s0 = after(s1);
        s1 = after(s0);
    }

    // The two halves of the contraction: each keeps half of the token tiles and hands its sums of the others over.
    constexpr int TE = TM / KG;
    asm volatile("s_waitcnt %0" ::"n"(tile_wait(0)) : "memory");
    if (KG == 2) __syncthreads();
    f32x4* const swap = reinterpret_cast<f32x4*>(smem) + lane;
    auto at = [&](int half, int i, int j) { return ((half * 4 + wr) * TE + i) * TN + j; };
    if constexpr (KG == 2) {
#pragma unroll
        for (int i = 0; i < TE; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) swap[at(kg, i, j) * 64] = kg ? acc[j][i] : acc[j][TE + i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < TE; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[j][i] = (kg ? acc[j][TE + i] : acc[j][i]) + swap[at(1 - kg, i, j) * 64];
    }
    const bool vec = (N & 3) == 0;
#pragma unroll
    for (int i = 0; i < TE; ++i) {
        const int64_t t = t0 + 16 * (kg * TE + i) + r;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const f32x4 s = acc[j][i];
            const int64_t n = n0 + 16 * j + 4 * h;
            if (t >= T || n >= N) continue;
            if (sums) {  // split contraction: sum_parts_kernel adds the parts
                *reinterpret_cast<f32x4*>(sums + ((int64_t)part * T + t) * ((N + 3) / 4 * 4) + n) = s;
            } else if (vec) {
                *reinterpret_cast<uint2*>(y + t * N + n) = make_uint2(pack_bf16x2(s[0], s[1]), pack_bf16x2(s[2], s[3]));
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < N) y[t * N + n + e] = f32_to_bf16(s[e]);
            }
        }
    }
#endif
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

static size_t sums_bytes(int64_t T, int64_t N, int parts) { return (size_t)parts * T * ((N + 3) / 4 * 4) * 4; }

// Tokens of a tile (64 or 128), parts of the contraction and units of 128 columns per wave, by an estimated time in us.  `more`:
// workgroups that share a compute unit with the first, whose waves they slow down.  Group-wise scales build a table per unit.  Parts
// cost the kernel that adds them and its fp32 sums.  Fitted to 74 shapes of 33 to 720 tokens, every shape and 1 .. 8 parts timed:
// mean error 5 %, the pick within 5 % of the fastest for 71 of them, 9 % at worst.
struct TilePlan {
    int tokens, parts, per;
    double estimate;
};
static TilePlan tile_plan(int64_t T, int64_t N, int64_t K, int64_t g, int q) {
    TilePlan best = {0, 0, 0, 1e300};
    const int64_t units = (K + 127) / 128;
    for (int groups = 1; groups <= 2; ++groups) {  // waves of that many parts
        const int64_t tiles = (N + 63) / 64 * ((T + 64 * groups - 1) / (64 * groups));
        for (int parts = 1; parts <= 8; ++parts) {
            if (parts > 1 && (2 * groups * parts > units || sums_bytes(T, N, parts) + 16 > mfma_fwd_workspace(N, K))) break;
            const double per = (double)((units + 2 * groups * parts - 1) / (2 * groups * parts) * 2), more = (double)((tiles * parts - 1) / 256);
            const double grouped = g != K ? q * (more + 1) : 0.0;
            double t = groups == 1 ? 4.0 + per * (0.34 + 0.058 * q + (0.11 + 0.082 * q) * more + 0.056 * grouped)
                                   : 4.7 + per * (0.89 + 0.154 * q + (1.07 + 0.21 * q) * more + 0.155 * grouped);
            if (parts > 1) t += 2.0 + 2.5e-6 * (double)(parts * T * N);
            if (t < best.estimate) best = TilePlan{64 * groups, parts, (int)per, t};
        }
    }
    best.estimate += 1.1e-6 * (double)(T * N);  // the result's stores
    return best;
}

static hipError_t launch_sums(const float* sums, int parts, int64_t T, int64_t N, bf16_t* y, hipStream_t st) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || parts == 1) return e;
    BCQ_LAUNCH(sum_parts_kernel, dim3((unsigned)((T * ((N + 3) / 4) + 255) / 256)), dim3(256), 0, st, sums, parts, T, N, y);
    return hipGetLastError();
}

template <int Q, int TM, int KG, bool GROUPED>
static hipError_t launch_tile(const uint32_t* packed, const float* alpha, const bf16_t* x, int64_t T, int64_t N, int64_t K,
                              int64_t g, bf16_t* y, float* sums, const TilePlan& p, hipStream_t st) {
    constexpr int LDS_B = tile_lds_bytes<TM, KG>();
    static LdsLimit limit;
    hipError_t e = limit.ensure((const void*)tile_fwd_kernel<Q, TM, KG, GROUPED>, LDS_B);
    if (e != hipSuccess) return e;
    const int token_tiles = (int)((T + 16 * TM - 1) / (16 * TM));
    const int items = (int)((N + 63) / 64) * token_tiles * p.parts;
    BCQ_LAUNCH((tile_fwd_kernel<Q, TM, KG, GROUPED>), dim3(xcd_grid(items)), dim3(256 * KG), LDS_B, st, packed, alpha, x, y, T, N, K, g,
                       p.per, token_tiles, p.parts, items, p.parts > 1 ? sums : nullptr);
    return launch_sums(sums, p.parts, T, N, y, st);
}

// Words of a lane, waves of a workgroup, parts of the contraction and segments per part, from 700 random calls of 1 to 32 tokens
// whose plans were all timed: the pick takes 1.027 times the fastest on average, and 0.67 of the time of a kernel whose waves read
// 32 rows and every scale of 128 columns apart (two calls of 3 to 6 us slower).
struct GroupPlan {
    int wpl, W, parts, per;
};
static int group_stage(int64_t T, int wpl) { return (int)((T * wpl + 3) / 4) * 1024; }  // LDS of a wave
static GroupPlan group_plan(int64_t T, int64_t N, int64_t K, int64_t g) {
    GroupPlan p;
    const int64_t gw = g / 32, tiles = (N + 15) / 16;
    int64_t segs = 0;
    // As many words as the group size allows (one load and one table for them all: 2048 x 2048 at 4 tokens 3.9 us, with two words
    // 4.2, with one 4.7), two above 16 tokens for the stages' sake, fewer where that leaves a chip with 256 waves idle.
    for (p.wpl = gw % 4 == 0 && T <= 16 ? 4 : gw % 2 == 0 ? 2 : 1;; p.wpl /= 2) {
        segs = (K + 128 * p.wpl - 1) / (128 * p.wpl);
        if (p.wpl == 1 || tiles * segs >= 256) break;
    }
    // One turn if possible; where compute units hold several workgroups, two of them have to fit.
    const int64_t room = (tiles > 256 ? 80 : 160) * 1024 / group_stage(T, p.wpl);
    const auto waves = [&](int64_t n, int64_t most) { const int64_t m = most < room ? most : room, turns = (n + m - 1) / m; return (n + turns - 1) / turns; };
    p.W = (int)waves(segs, tiles > 256 ? 8 : 16);
    // Few rows and a long contraction: parts of it on compute units of their own while they find an idle one and it saves a turn
    // (1280 x 5120, groups of 32, 29 tokens: 13.8 -> 10.8 us; 2048 x 8192, 4 tokens, in one turn 7.3, in two parts 7.6).
    p.parts = 1;
    while (p.parts < 8 && tiles * p.parts * 2 <= 256 && (segs + p.parts - 1) / p.parts >= 2 * p.W &&
           sums_bytes(T, N, 2 * p.parts) <= mfma_fwd_workspace(N, K))
        p.parts *= 2;
    p.per = (int)((segs + p.parts - 1) / p.parts);
    p.parts = (int)((segs + p.per - 1) / p.per);
    if (p.parts > 1) p.W = (int)waves(p.per, 16);
    return p;
}

template <int Q, int WPL>
static hipError_t launch_group(const uint32_t* packed, const float* alpha, const bf16_t* x, int64_t T, int64_t N, int64_t K,
                               int64_t g, bf16_t* y, float* sums, const GroupPlan& p, hipStream_t st) {
    const int stage = group_stage(T, WPL), segs = (int)((K + 128 * WPL - 1) / (128 * WPL));
    const uint32_t gw = (uint32_t)(g / 32), inverse = gw == 1 ? 0u : 0xFFFFFFFFu / gw + 1u;  // word / gw = high half of word * inverse
    const size_t lds = (size_t)p.W * stage;
    constexpr bool one_tile = WPL == 4;  // (of tokens, as group_plan has it)
    if (one_tile && T > 16) return hipErrorInvalidConfiguration;
    const auto kernel = one_tile || T <= 16 ? group_fwd_kernel<Q, WPL, 1> : group_fwd_kernel<Q, WPL, one_tile ? 1 : 2>;
    static LdsLimit limit[2];
    hipError_t e = limit[T > 16].ensure((const void*)kernel, lds);
    if (e != hipSuccess) return e;
    BCQ_LAUNCH(kernel, dim3((unsigned)((N + 15) / 16), (unsigned)p.parts), dim3((unsigned)(64 * p.W)), lds, st, packed, alpha, x, y, (int)T,
               N, (int)K, (int)gw, inverse, segs, p.per, p.W, stage, p.parts > 1 ? sums : nullptr);
    return launch_sums(sums, p.parts, T, N, y, st);
}

template <int Q>
static hipError_t launch_q(const uint32_t* packed, const float* alpha, const bf16_t* x, int64_t T, int64_t N, int64_t K,
                           int64_t g, bf16_t* y, float* sums, hipStream_t st) {
    if (T > 32) {
        const TilePlan p = tile_plan(T, N, K, g, Q);
        if (p.tokens == 64) {
            if (g != K) return launch_tile<Q, 4, 1, true>(packed, alpha, x, T, N, K, g, y, sums, p, st);
            return launch_tile<Q, 4, 1, false>(packed, alpha, x, T, N, K, g, y, sums, p, st);
        }
        if (g != K) return launch_tile<Q, 8, 2, true>(packed, alpha, x, T, N, K, g, y, sums, p, st);
        return launch_tile<Q, 8, 2, false>(packed, alpha, x, T, N, K, g, y, sums, p, st);
    }
    const GroupPlan p = group_plan(T, N, K, g);
    if (p.wpl == 4) return launch_group<Q, 4>(packed, alpha, x, T, N, K, g, y, sums, p, st);
    if (p.wpl == 2) return launch_group<Q, 2>(packed, alpha, x, T, N, K, g, y, sums, p, st);
    return launch_group<Q, 1>(packed, alpha, x, T, N, K, g, y, sums, p, st);
}

// Row-wise scales, 129 to 384 tokens, large layers: whether row tiles of 32 rows and 128 tokens (64 in smaller layers) fill one round
// of workgroups, two or one to a compute unit.
static bool one_full_round(int64_t T, int64_t N, int64_t K, int q) {
    const int64_t cols = (N + 31) / 32, tiles = cols * ((T + 127) / 128), units = (K + 127) / 128;
    const bool wide = tiles >= 256 || (tiles >= 64 && units >= 64);
    if (!wide) return cols * ((T + 63) / 64) <= 256;
    return T <= 256 && tiles <= 512 && tiles > (q == 4 ? 384 : 320);
}

// Where one kernel is faster than expanding What and multiplying.  Calls with row-wise scales, or groups of whole 512-column segments, come
// here with more than 80 tokens (the streaming kernels take them before), those with other groups with any number.
// Up to 32 tokens always (one / two kernels, us: 32 tokens, q = 4, groups of 32, of 10240 x 2592 16 / 25, of 40960 x 960 21 / 40, of 10240 x 96
// 3.3 / 7.2), with row-wise scales up to 128 unless the estimates below are clearly against
// it.  Row-wise scales, 129 to 384 tokens: except above 40 million weights, and with four planes above 256 tokens above 8
// million, unless one_full_round, and up to 100 million, from where What no longer fits the 256 MB cache in front of HBM.  These
// lines were set (65000 timings) against a one-kernel form of the rows and tokens that one_full_round counts; of 70 random calls in
// their range the present form is on the side that is more than 4 % slower in 8.  With one and two planes they are early (one / two kernels,
// us: 160 tokens of 5120 x 7840, q = 1, 29 / 43, of 8224 x 4896, q = 2, 39 / 43), with three and four about right (288 of 5120 x
// 8000, q = 3, 58 / 57, 320 of 1664 x 5056, q = 4, 26 / 25.5, 257 of 8200 x 992 19 / 17; 223 of 9344 x 2336 38 / 30).
// Group-wise scales: a line of the same kind in q and the parity of the words in a group.
// For layers of more than a million weights and 512 columns (whose time is more than start and end) the two estimates, whose errors
// are 5 to 10 %, overrule the lines where they are clear: beyond them, from 385 tokens on or with group-wise scales, one kernel where its
// estimate is a tenth below that of two (us, one / two: 421 tokens of 1312 x 5248, q = 1, groups of 128, 20.6 / 24.5, 720 of 2336 x 2336,
// q = 1, 17.5 / 21.8, 206 of 2496 x 9984, q = 2, groups of 32, 34 / 45; with equal estimates 301 of 14680 x 4096, q = 2, groups of 256,
// 98 / 70, 602 of 3720 x 6432, q = 2, 69 / 53), and two kernels where the one's is a tenth above (378 of 11392 x 2464, q = 3, 54 / 37).
// Against the forms before tile_fwd_kernel, 1159 random calls of 33 to 768 tokens: 0.87 of the time, 40 more than 4 % slower, 12 of them
// more than 8 %, worst 1.15 (140 tokens of 2720 x 2528, q = 2, 13.1 -> 15.1); no choice of route or plan would leave less than 17.
bool fused_fwd_ok(int64_t T, int64_t N, int64_t K, int64_t g, int q) {
    if (q > 4) return false;
    if (T <= 32) return true;
    // layers of fewer rows than tokens have few row tiles, and no room for the sums of parts
    if (T > 768 || (T + 31) / 32 * 32 * K * 2 > (int64_t)mfma_fwd_workspace(N, K)) return false;
    const int64_t work = N * K * T;
    if (K > 512 && N * K > 1000000) {
        const double one = tile_plan(T, N, K, g, q).estimate, two = two_kernel_estimate(T, N, K, q);
        if (0.9 * one > two && N * K <= 100000000) return false;
        if ((T > 384 || g != K) && 1.1 * one < two) return true;
    }
    if (T > 384) return false;
    if (g == K) {
        const bool large = (T > 128 && N * K > 40000000) || (T > 256 && q == 4 && N * K > 8000000);
        return !large || N * K > 100000000 || one_full_round(T, N, K, q);
    }
    const bool odd = (g / 32) % 2 != 0;
    const int level = q + (odd ? 1 : 0);
    if (odd && q > 1 && N * K < 1200000) return false;  // 1024 x 1024, q = 4, 64 tokens: 14 / 11
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
    float* sums = (float*)workspace;
    switch (q) {
        case 1: return launch_q<1>(packed, alpha, xb, T, N, K, g, yb, sums, st);
        case 2: return launch_q<2>(packed, alpha, xb, T, N, K, g, yb, sums, st);
        case 3: return launch_q<3>(packed, alpha, xb, T, N, K, g, yb, sums, st);
        default: return launch_q<4>(packed, alpha, xb, T, N, K, g, yb, sums, st);
    }
}

}  // namespace bcq

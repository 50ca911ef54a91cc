// Host side of the small-token streaming kernels (bcq_stream_kernels.h): launch plans and the single-layer launchers.
#include "bcq_stream_kernels.h"

namespace bcq {

// ---------------------------------------------------------------------------------------------------------
// gsegs > 0: the contraction axis carries scale groups of gsegs segments each and every wave must own whole groups
static StreamPlan stream_plan(int64_t T, int64_t rows, int64_t cw, int gsegs = 0) {
    StreamPlan p;
    p.segs = (cw + 15) / 16;
    p.halves = T <= 8 ? 1 : 2;
    p.tiles = (int)((T + 15) / 16);
    // One 16-row tile per wave: measured faster than two at every size (more waves keep more plane bytes in flight,
    // which is what bounds the stream; the activation operand is L2-resident either way).
    p.R = 1;
    const int64_t blocks = (rows + 16 * p.R - 1) / (16 * p.R);
    // waves per workgroup: aim at about two waves per SIMD (2048 on the chip); among the candidates from there up to
    // 8 take the first that keeps every wave at least 80 % loaded, else the best balanced
    const int wmax = (int)(p.segs < 8 ? p.segs : 8);
    int w0 = (int)((2048 + blocks - 1) / blocks);
    w0 = w0 < 1 ? 1 : (w0 > wmax ? wmax : w0);
    int best_w = w0;
    double best_eff = 0.0;
    for (int w = w0; w <= wmax; ++w) {
        const int64_t spw = (p.segs + w - 1) / w;
        const double eff = (double)p.segs / (double)(w * spw);
        if (eff >= 0.8) {
            best_w = w;
            break;
        }
        if (eff > best_eff + 1e-9) {
            best_eff = eff;
            best_w = w;
        }
    }
    p.W = best_w;
    p.segs_per_wave = (int)((p.segs + best_w - 1) / best_w);
    if (gsegs > 0) {  // whole groups per wave
        const int64_t groups = p.segs / gsegs;
        if (p.W > groups) p.W = (int)groups;
        const int64_t gpw = (groups + p.W - 1) / p.W;
        p.W = (int)((groups + gpw - 1) / gpw);
        p.segs_per_wave = (int)(gpw * gsegs);
    }
    p.grid_x = (unsigned)((rows + 16 * p.R - 1) / (16 * p.R));
    p.xq_bytes = (size_t)p.tiles * p.segs * 4 * p.halves * QBLK;
    p.sq_bytes = (size_t)p.tiles * p.segs * p.halves * QSCL;
    return p;
}

size_t stream_workspace(int64_t T, int64_t contraction, int sets) {
    const StreamPlan p = stream_plan(T, 16, contraction / 32);
    return (size_t)sets * (p.xq_bytes + p.sq_bytes);
}

// Plan of stream_lds_kernel: KW = 0 means "use stream_kernel".  It pays when the workgroups (8 / KW row tiles each)
// still fill the chip, i.e. for plane matrices with many rows (at least min_wgs workgroups).
struct LdsPlan {
    int KW, spp;
    bool exact;
    unsigned grid_x;
};
static LdsPlan lds_plan(int64_t rows, int64_t segs, int halves, int gsegs, int q_used, int min_wgs = 224) {
    LdsPlan p = {0, 0, false, 0};
    if (q_used > 4) return p;  // the ring of plane registers is sized for up to 4 planes
    const int64_t rt = (rows + 15) / 16;
    int kw = 0;
    if ((rt + 7) / 8 >= min_wgs)
        kw = 1;
    else if (halves == 1 && (rt + 3) / 4 >= min_wgs)
        kw = 2;
    if (kw == 0 || segs < 2 * LCS * kw) return p;
    int64_t spp = (segs + kw - 1) / kw;
    if (gsegs > 0) spp = (spp + gsegs - 1) / gsegs * gsegs;  // whole scale groups per part
    p.KW = kw;
    p.spp = (int)spp;
    p.exact = (spp * kw == segs) && (spp % LCS == 0);
    p.grid_x = (unsigned)((rt + (8 / kw) - 1) / (8 / kw));
    return p;
}

template <int MODE, int QP, bool TWO, bool GROUPED, int KW, bool EXACT, bool TILED>
static hipError_t launch_lds_cfg(const uint32_t* planes, const unsigned char* xq, const unsigned char* sq,
                                 const float* alpha, const bf16_t* dy, void* out, int64_t T, int64_t rows, int64_t cw,
                                 int q_used, float scale, const LdsPlan& lp, int64_t segs, int tiles, int gsegs, int G,
                                 hipStream_t st, int64_t xq_plane = 0, int64_t sq_plane = 0, uint32_t seg_magic = 0,
                                 int segs_n = 0) {
    constexpr int H = TWO ? 2 : 1;
    constexpr int LDS_B = 2 * KW * LCS * H * (4 * QBLK + QSCL);
    static LdsLimit limit;
    hipError_t e = limit.ensure((const void*)stream_lds_kernel<MODE, QP, TWO, GROUPED, KW, EXACT, TILED>, LDS_B);
    if (e != hipSuccess) return e;
    BCQ_LAUNCH((stream_lds_kernel<MODE, QP, TWO, GROUPED, KW, EXACT, TILED>), dim3(lp.grid_x, (unsigned)tiles), dim3(512),
                       LDS_B, st, planes, xq, sq, alpha, dy, out, T, rows, cw, q_used, scale, lp.spp, segs, gsegs, G, xq_plane,
                       sq_plane, seg_magic, segs_n);
    return hipGetLastError();
}

// input gradient through stream_lds_kernel: one virtual plane over q * segs_n segments
static hipError_t launch_lds_dx(const uint32_t* twin, const unsigned char* xq, const unsigned char* sq, void* out, int64_t T,
                                int64_t rows, int64_t cw, const LdsPlan& lp, int64_t vsegs, int tiles, int halves,
                                int64_t xq_plane, int64_t sq_plane, int segs_n, int G, hipStream_t st) {
    const uint32_t magic = (uint32_t)((((uint64_t)1 << 32) + (uint64_t)segs_n - 1) / (uint64_t)segs_n);
#define BCQ_LDS_DX(TT, KW, EX)                                                                                          \
    return launch_lds_cfg<STREAM_DX, 1, TT, false, KW, EX, false>(twin, xq, sq, nullptr, nullptr, out, T, rows, cw, 1, 1.f, lp, \
                                                                  vsegs, tiles, 1, G, st, xq_plane, sq_plane, magic, segs_n)
    if (halves == 2) {
        if (lp.exact) BCQ_LDS_DX(true, 1, true);
        BCQ_LDS_DX(true, 1, false);
    }
    if (lp.KW == 2) {
        if (lp.exact) BCQ_LDS_DX(false, 2, true);
        BCQ_LDS_DX(false, 2, false);
    }
    if (lp.exact) BCQ_LDS_DX(false, 1, true);
    BCQ_LDS_DX(false, 1, false);
#undef BCQ_LDS_DX
}

template <int MODE, int QP, bool TWO, bool GROUPED, bool TILED>
static hipError_t launch_lds_kw(const uint32_t* planes, const unsigned char* xq, const unsigned char* sq,
                                const float* alpha, const bf16_t* dy, void* out, int64_t T, int64_t rows, int64_t cw,
                                int q_used, float scale, const LdsPlan& lp, int64_t segs, int tiles, int gsegs, int G,
                                hipStream_t st) {
#define BCQ_LDS_GO(KW, EX) \
    return launch_lds_cfg<MODE, QP, TWO, GROUPED, KW, EX, TILED>(planes, xq, sq, alpha, dy, out, T, rows, cw, q_used, scale, lp, \
                                                          segs, tiles, gsegs, G, st)
    if (!TWO && lp.KW == 2) {
        if (lp.exact) BCQ_LDS_GO((TWO ? 1 : 2), true);
        BCQ_LDS_GO((TWO ? 1 : 2), false);
    }
    if (lp.exact) BCQ_LDS_GO(1, true);
    BCQ_LDS_GO(1, false);
#undef BCQ_LDS_GO
}

template <int MODE, bool TILED>
static hipError_t launch_lds(const uint32_t* planes, const unsigned char* xq, const unsigned char* sq, const float* alpha,
                             const bf16_t* dy, void* out, int64_t T, int64_t rows, int64_t cw, int q_used, float scale,
                             const LdsPlan& lp, int64_t segs, int tiles, int halves, bool grouped, int gsegs, int G,
                             hipStream_t st) {
#define BCQ_LDS_ARGS planes, xq, sq, alpha, dy, out, T, rows, cw, q_used, scale, lp, segs, tiles, gsegs, G, st
#define BCQ_LDS_Q(QQ)                                                                          \
    if (halves == 2) {                                                                         \
        if (grouped) return launch_lds_kw<MODE, QQ, true, true, TILED>(BCQ_LDS_ARGS);          \
        return launch_lds_kw<MODE, QQ, true, false, TILED>(BCQ_LDS_ARGS);                      \
    } else {                                                                                   \
        if (grouped) return launch_lds_kw<MODE, QQ, false, true, TILED>(BCQ_LDS_ARGS);         \
        return launch_lds_kw<MODE, QQ, false, false, TILED>(BCQ_LDS_ARGS);                     \
    }
    switch (q_used) {
        case 1: BCQ_LDS_Q(1)
        case 2: BCQ_LDS_Q(2)
        case 3: BCQ_LDS_Q(3)
        default: BCQ_LDS_Q(4)
    }
#undef BCQ_LDS_Q
#undef BCQ_LDS_ARGS
}

// g = group size of the scales along the columns of W (K of the layer); g == layer K means row-wise.
// The single-kernel form is used when a wave has one segment and all waves of the launch are resident at once
// (every wave repeats the re-coding of its segment, about 2.5 us of vector-ALU work; measured: 2560 x 2560 and
// 5120 x 1280 gain 2.3 - 2.7 us per call, 7680 x 2560 loses 1.7 us, 10240 x 2560 loses 8 us)
constexpr int FUSED_MAX_SEGS = 1;
constexpr int64_t FUSED_MAX_WAVES = 1024;
// From the decode layout (where only calls of more than four planes come here, few_fwd_kernel takes the others) it pays for one wave and
// row-wise scales: 512 x 512, q = 8 7.2 -> 6.6 us, but 4096 x 2048 8.2 -> 9.3.
constexpr unsigned FUSED_TILED_MAX_WGS = 256;

template <int MODE, int QP, bool TWO, bool TILED>
static hipError_t launch_fused_cfg(const uint32_t* planes, const bf16_t* act, const float* alpha, const bf16_t* dy,
                                   void* out, int64_t T, int64_t rows, int64_t cw, int q_used, float scale,
                                   const StreamPlan& p, int gsegs, int G, hipStream_t st) {
    constexpr int H = TWO ? 2 : 1;
    const int nout = (MODE == STREAM_DALPHA) ? q_used : 1;
    const size_t stage = (size_t)p.W * (4 * H * QBLK + H * QSCL), red = (size_t)p.W * nout * 1024;
    const size_t lds = stage > red ? stage : red;
    static LdsLimit limit;
    hipError_t e = limit.ensure((const void*)stream_fused_kernel<MODE, QP, TWO, TILED>, lds);
    if (e != hipSuccess) return e;
    BCQ_LAUNCH((stream_fused_kernel<MODE, QP, TWO, TILED>), dim3(p.grid_x, (unsigned)p.tiles), dim3((unsigned)(64 * p.W)),
                       lds, st, planes, act, alpha, dy, out, T, rows, cw, q_used, scale, p.segs_per_wave, p.segs, gsegs, G);
    return hipGetLastError();
}

template <int MODE, bool TILED>
static hipError_t launch_fused(const uint32_t* planes, const bf16_t* act, const float* alpha, const bf16_t* dy, void* out,
                               int64_t T, int64_t rows, int64_t cw, int q_used, float scale, const StreamPlan& p,
                               int gsegs, int G, hipStream_t st) {
#define BCQ_FUSED(QQ, TT) \
    return launch_fused_cfg<MODE, QQ, TT, TILED>(planes, act, alpha, dy, out, T, rows, cw, q_used, scale, p, gsegs, G, st);
#define BCQ_FUSED_Q(TT)              \
    switch (q_used) {                \
        case 1: BCQ_FUSED(1, TT)     \
        case 2: BCQ_FUSED(2, TT)     \
        case 3: BCQ_FUSED(3, TT)     \
        case 4: BCQ_FUSED(4, TT)     \
        default: BCQ_FUSED(8, TT)    \
    }
    // one half of a forward, and with it the decode layout: more than four planes only, the others are few_fwd_kernel's
    if constexpr (!TILED) {
        if (p.halves == 2) { BCQ_FUSED_Q(true) }
        if constexpr (MODE != STREAM_FWD) { BCQ_FUSED_Q(false) }
    }
    if constexpr (MODE == STREAM_FWD) {
        if (p.halves == 1 && q_used > 4) BCQ_FUSED(8, false)
    }
    return hipErrorInvalidConfiguration;
#undef BCQ_FUSED_Q
#undef BCQ_FUSED
}

// ---- forward of at most 8 tokens in one kernel ------------------------------------------------------------------------
// Segments (W) and row tiles (R) of a workgroup.  Sharing the re-coded activations between R row tiles saves 0.27 us per token and row tile
// where there are several tokens (8 tokens, q = 4, of 7680 x 2560: 10.0 -> 7.2 us), and costs up to 1.5 us where it leaves compute units without a
// workgroup or puts 16 waves into one (1024 x 4096, q = 3, one token 4.2 -> 5.3).  Three where they, and not two, keep the workgroups to one
// round, that is for 513 to 768 row tiles (10240 x 2560, q = 4, 8 tokens: two 12.3, three 8.4; 13889 x 2048, q = 3, 10.9 / 14.1).  Eight
// segments share only with many tokens and tiles (7127 x 4096, q = 1, 8 tokens 11.0 -> 7.9; 1553 x 4096, q = 2, 7 tokens 7.4 / 7.2), and where
// every compute unit has a workgroup anyway the many rows of canonical planes that many waves read at once cost more (257 x 3264, q = 4, 6
// tokens 8.5 / 9.5; from the decode layout 7.4 / 7.6).
// Up to 256 row tiles take up to 16 segments at a time instead of 8: a turn is a whole trip to memory and through the re-coding (one token of 1280 x
// 5120, q = 4, 5.3 -> 4.7 us, four 7.6 -> 6.5).  Beyond them the larger workgroups take a second round (320 tiles: 1.1 to 1.4 times the
// time); 15 and 16 waves gain nothing at one token (2048 x 8192, q = 4, 6.2 -> 6.4).
struct FewPlan {
    int W, R;
};
static FewPlan few_plan(int64_t T, int64_t rows, int segs, int q, bool rowwise, bool tiled) {
    FewPlan p;
    const int64_t tiles = (rows + 15) / 16;
    const auto waves = [&](int most) { const int turns = (segs + most - 1) / most; return (segs + turns - 1) / turns; };
    p.W = waves(8);
    const bool room = tiles <= 256 && 16 * (FEW_STAGE + few_scale_bytes(q, !rowwise)) <= 160 * 1024;
    if (room && !(rowwise && T == 1 && waves(16) > 14)) p.W = waves(16);
    bool share = T >= 3 && p.W < 8;
    if (!rowwise) share = share && tiles > (T <= 4 ? 256 : p.W <= 3 ? 0 : 128);
    if (rowwise && !tiled && tiles <= 256) share = share && q * p.W < 14;
    if (p.W == 8) share = T > 4 && tiles > 256;
    p.R = !share ? 1 : tiles > 512 && tiles <= 768 && p.W <= 5 ? 3 : 2;
    return p;
}

// Where it is faster than re-coding in a kernel of its own (the re-coding is repeated by every R row tiles): where its workgroups run in
// one round (a compute unit holds 16 waves; 9822 x 3072, groups of 1536, q = 4, six tokens in two rounds 11.2 / 19.6 us, that / this),
// and the contraction is not too long for the tokens.  us, that / this: one token of 1024 x 1024, q = 3, 5.3 / 3.3, 10240 x 2560,
// q = 4, 12.1 / 7.0, 2560 x 10240 10.6 / 7.8, 118 x 13504, q = 2, 9.4 / 6.4, but two tokens of 134 x 12416, q = 4, 12.2 / 14.9; four tokens
// 1024 x 1024 5.4 / 4.0, 10240 x 2560 12.2 / 7.2, 2048 x 8192, q = 3, 8.1 / 8.0, but 1231 x 8448, q = 1, 8.2 / 9.1, and of canonical planes
// three of 2229 x 7168, q = 4, 10.0 / 12.4; eight tokens 5.6 / 4.4, 12.3 / 8.4, 1024 x 4096 7.2 / 7.3, 1952 x 5312, q = 2, 7.6 / 8.6.  Of layers
// above 32 million weights about half are faster (11730 x 3104, q = 3, one token 14.6 / 10.1, 4346 x 9376, q = 1, six 12.9 / 16.3).
// Groups (whole segments here) read their scales from the canonical planes' side in 16-byte pieces: four tokens of 1022 x 6144, groups
// of 1024, q = 4, 9.2 / 10.4, of 72 x 9216, groups of 1536, 10.2 / 15.8, six of 2590 x 3072 9.0 / 10.5, of 8692 x 2048 9.0 / 10.6, from the decode layout
// 2339 x 3072 8.8 / 7.7 at eight, 164 x 9216 9.8 / 11.4 at three.
// Against the kernels that ran before this one, 5000 random calls of both layouts: 0.79 of the time, 34 more than 4 % slower, 6 of
// them more than 8 % (worst 1.25: four tokens of 4157 x 7680, groups of 512, q = 3, decode layout).
static bool few_fwd_ok(int64_t T, int64_t N, int64_t K, int64_t g, int q, bool tiled) {
    if (N * K > 32000000) return false;
    const FewPlan p = few_plan(T, N, (int)((K + 511) / 512), q, g == K, tiled);
    if ((N + 16 * p.R - 1) / (16 * p.R) > 256 * (16 / (p.W * p.R))) return false;
    if (g == K) return K <= (T <= 2 ? 12288 : T > 4 ? 4096 : q == 4 && !tiled ? 6144 : 8192);
    if (tiled) return K <= (T <= 2 ? 10240 : T <= 4 ? 8192 : 3072);
    if (q > 2 && N > 4096) return K <= (N > 8192 ? 1536 : 2048);
    return K <= (T <= 4 ? (q > 2 ? 4096 : 6144) : q == 4 ? 2048 : 3072);
}

template <int QP, int NT, bool TILED, bool GROUPED>
static hipError_t launch_few_cfg(const uint32_t* planes, const bf16_t* act, const float* alpha, bf16_t* y, int64_t T, int64_t rows, int64_t cw,
                                 int64_t g, int segs, const FewPlan& p, hipStream_t st) {
    const size_t lds = (size_t)p.W * FEW_STAGE + (size_t)p.W * p.R * few_scale_bytes(QP, GROUPED);
    if (lds > 160 * 1024) return hipErrorInvalidConfiguration;
    static LdsLimit limit;
    hipError_t e = limit.ensure((const void*)few_fwd_kernel<QP, NT, TILED, GROUPED>, lds);
    if (e != hipSuccess) return e;
    BCQ_LAUNCH((few_fwd_kernel<QP, NT, TILED, GROUPED>), dim3((unsigned)((rows + 16 * p.R - 1) / (16 * p.R))), dim3((unsigned)(64 * p.W * p.R)), lds, st,
                       planes, act, alpha, y, (int)T, rows, (int)cw, segs, (int)(g / 32), (int)(cw * 32 / g), p.W, p.R);
    return hipGetLastError();
}

template <bool TILED>
static hipError_t launch_few(const uint32_t* planes, const bf16_t* act, const float* alpha, bf16_t* y, int64_t T, int64_t rows, int64_t cw, int q,
                             int64_t g, hipStream_t st) {
    const int segs = (int)((cw + 15) / 16);
    const bool grouped = g != cw * 32;
    const FewPlan p = few_plan(T, rows, segs, q, !grouped, TILED);
    const int64_t NT = (T + p.R - 1) / p.R;
    if (T > 8 || p.W * p.R > 16 || p.W * p.R < 1) return hipErrorInvalidConfiguration;
#define BCQ_FEW(QQ, TT, GR) return launch_few_cfg<QQ, TT, TILED, GR>(planes, act, alpha, y, T, rows, cw, g, segs, p, st);
#define BCQ_FEW_T(QQ, GR)          \
    if (NT > 4) BCQ_FEW(QQ, 8, GR) \
    if (NT > 2) BCQ_FEW(QQ, 4, GR) \
    if (NT > 1) BCQ_FEW(QQ, 2, GR) \
    BCQ_FEW(QQ, 1, GR)
#define BCQ_FEW_G(QQ)                     \
    if (grouped) { BCQ_FEW_T(QQ, true) } \
    BCQ_FEW_T(QQ, false)
    switch (q) {
        case 1: { BCQ_FEW_G(1) }
        case 2: { BCQ_FEW_G(2) }
        case 3: { BCQ_FEW_G(3) }
        default: { BCQ_FEW_G(4) }
    }
#undef BCQ_FEW_G
#undef BCQ_FEW_T
#undef BCQ_FEW
}

template <int MODE, bool TILED = false>
static hipError_t launch_stream(const uint32_t* planes, const bf16_t* act, const float* alpha, const bf16_t* dy, void* out,
                                int64_t T, int64_t rows, int64_t cw, int q, int q_used, float scale, void* workspace,
                                int64_t g, int64_t layer_k, hipStream_t st) {
    const bool grouped = (g != layer_k);
    const int G = (int)(layer_k / g);
    const int gsegs = (grouped && MODE != STREAM_DX) ? (int)(g / 512) : 0;  // needs g % 512 == 0 (checked by the caller)
    const StreamPlan p = stream_plan(T, rows, cw, gsegs);
    if (p.W < 1 || p.W > 8 || p.R != 1) return hipErrorInvalidConfiguration;  // compiled for at most 512 threads, R = 1
    if constexpr (MODE != STREAM_DX) {
        const bool single = p.segs_per_wave <= FUSED_MAX_SEGS &&
                            (TILED ? p.halves == 1 && p.grid_x <= FUSED_TILED_MAX_WGS && p.W == 1 && q_used > 4 && !grouped
                                   : (int64_t)p.grid_x * p.tiles * p.W <= FUSED_MAX_WAVES);
        if constexpr (MODE == STREAM_FWD) {  // (what fits the general single kernel is always faster so: 598 x 3584, groups of 512, 11.1 / 9.4)
            if (T <= 8 && q <= 4 && (single || few_fwd_ok(T, rows, layer_k, g, q, TILED)))
                return launch_few<TILED>(planes, act, alpha, (bf16_t*)out, T, rows, cw, q, g, st);
        }
        if (single) return launch_fused<MODE, TILED>(planes, act, alpha, dy, out, T, rows, cw, q_used, scale, p, gsegs, G, st);
    }
    const int sets = (MODE == STREAM_DX) ? q * G : 1;
    unsigned char* xq = reinterpret_cast<unsigned char*>(workspace);
    unsigned char* sq = xq + (size_t)sets * p.xq_bytes;
    {
        const dim3 grid((unsigned)(p.tiles * p.segs), (unsigned)sets);
        BCQ_LAUNCH((quant_act_kernel<MODE>), grid, dim3(p.halves == 1 ? 128 : 256), 0, st, act, alpha, T, cw * 32, p.segs, p.halves,
                           xq, sq, p.xq_bytes, p.sq_bytes, G);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if constexpr (MODE == STREAM_DX) {
        if (cw % 16 == 0) {  // whole segments
            const int64_t vsegs = (int64_t)q_used * p.segs;
            // the per-wave kernel fetches one activation set per plane and row tile, so sharing pays from fewer
            // workgroups than for the forward (measured at 8 tokens: 10240 rows 18.0 -> 14.9 us, 12288 rows equal,
            // 6144 rows 3 % slower)
            const LdsPlan lp = lds_plan(rows, vsegs, p.halves, 0, 1, p.halves == 1 ? 160 : 224);
            // group-wise scales: a workgroup (8 / KW row tiles of the twin) takes ONE activation set, so its rows must
            // lie in one scale group; other group sizes keep the per-wave kernel (16 rows per workgroup, g % 32 == 0)
            const bool one_group = (G == 1) || (lp.KW > 0 && g % (16 * (8 / lp.KW)) == 0);
            if (lp.KW > 0 && one_group)
                return launch_lds_dx(planes, xq, sq, out, T, rows, cw, lp, vsegs, p.tiles, p.halves, (int64_t)p.xq_bytes,
                                     (int64_t)p.sq_bytes, (int)p.segs, G, st);
        }
    }
    if constexpr (MODE != STREAM_DX) {
        if (TILED || cw % 4 == 0) {
            const LdsPlan lp = lds_plan(rows, p.segs, p.halves, gsegs, q_used);
            if (lp.KW > 0)
                return launch_lds<MODE, TILED>(planes, xq, sq, alpha, dy, out, T, rows, cw, q_used, scale, lp, p.segs, p.tiles,
                                        p.halves, grouped, gsegs > 0 ? gsegs : 1, G, st);
        }
    }
    const dim3 grid(p.grid_x, (unsigned)p.tiles);
    const dim3 block((unsigned)(64 * p.W));
    const int nout = (MODE == STREAM_DALPHA) ? q_used : 1;
    const size_t lds = (size_t)p.W * p.R * nout * 64 * 4 * sizeof(float);
    const int qp = q_used <= 4 ? q_used : 8;
    const bool quad = TILED || (cw % 4 == 0);  // the decode layout has one instantiation (the flag is unused there)
#define BCQ_STREAM_GO(QQ, TT, QD, GR)                                                                                  \
    BCQ_LAUNCH((stream_kernel<MODE, 1, QQ, TT, QD, GR, TILED>), grid, block, lds, st, planes, xq, sq, alpha, dy, out, T, \
                       rows, cw, q_used, scale, p.segs_per_wave, p.segs, p.xq_bytes, p.sq_bytes, 127,                  \
                       gsegs > 0 ? gsegs : 1, G, g)
#define BCQ_STREAM_GR(QQ, TT, QD)            \
    if (grouped) {                           \
        BCQ_STREAM_GO(QQ, TT, QD, true);     \
    } else {                                 \
        BCQ_STREAM_GO(QQ, TT, QD, false);    \
    }
#define BCQ_STREAM_QD(QQ, TT)            \
    if (quad) {                          \
        BCQ_STREAM_GR(QQ, TT, true)      \
    } else {                             \
        BCQ_STREAM_GR(QQ, TT, TILED)     \
    }
#define BCQ_STREAM_Q(TT)                              \
    switch (qp) {                                     \
        case 1: BCQ_STREAM_QD(1, TT) break;           \
        case 2: BCQ_STREAM_QD(2, TT) break;           \
        case 3: BCQ_STREAM_QD(3, TT) break;           \
        case 4: BCQ_STREAM_QD(4, TT) break;           \
        default: BCQ_STREAM_QD(8, TT) break;          \
    }
    if (p.halves == 2) {
        BCQ_STREAM_Q(true)
    } else {
        BCQ_STREAM_Q(false)
    }
#undef BCQ_STREAM_Q
#undef BCQ_STREAM_QD
#undef BCQ_STREAM_GR
#undef BCQ_STREAM_GO
    return hipGetLastError();
}

size_t stream_fwd_workspace(int64_t T, int64_t K) { return stream_workspace(T, K, 1); }
size_t stream_bwd_alpha_workspace(int64_t T, int64_t K) { return stream_workspace(T, K, 1); }
size_t stream_bwd_input_workspace(int64_t T, int64_t N, int sets) { return stream_workspace(T, N, sets); }

hipError_t launch_fwd_stream(const uint32_t* packed, const float* alpha, const void* x, int64_t T, int64_t N,
                             int64_t K, int64_t g, int q, void* y, void* workspace, hipStream_t st) {
    return launch_stream<STREAM_FWD>(packed, (const bf16_t*)x, alpha, nullptr, y, T, N, K / 32, q, q, 1.f, workspace, g, K,
                                     st);
}

hipError_t launch_fwd_stream_decode(const uint32_t* tiled, const float* alpha, const void* x, int64_t T, int64_t N,
                                    int64_t K, int64_t g, int q, void* y, void* workspace, hipStream_t st) {
    return launch_stream<STREAM_FWD, true>(tiled, (const bf16_t*)x, alpha, nullptr, y, T, N, K / 32, q, q, 1.f, workspace,
                                           g, K, st);
}

// canonical packed[q][N][K/32] -> decode layout [N/16 up][K/512 up][q][64 lanes][4 words]; lane = (n % 16) + 16 g holds
// words 16 seg + 4 g .. + 3 of row n; rows and columns beyond the matrix read as 0 bits
// A wave writes one KiB (row tile, segment, plane) of each of two planes.  The units (row tile, segment) are counted through, four to a
// workgroup, so that no wave is left without one (with a grid over segments and row tiles 3 of 8 waves were, at 5 segments: 10240 x 2560,
// q = 4, 7.0 us, now 5.9; 7680 x 2560 5.4 / 5.0; 15 segments, whose rows now straddle workgroups, 4.8 / 5.0).  unit / segs is the high word of unit * inverse, the inverse 2^32 / segs rounded up, exact for units below
// 2^24 (0 stands for 2^32).  The stores are nontemporal: nothing reads the layout soon (10240 x 2560, q = 4: 6.9 -> 6.6 us,
// 2560 x 10240 5.7 -> 4.9; one plane to a wave 6.7 and 5.4, four 6.3 and 5.2, plain stores with any of them as before; a copy of the
// 26 MB takes 4.9).  QUAD: rows of whole 16-byte units (cw % 4 == 0), one load per lane.
template <bool QUAD>
__global__ __launch_bounds__(256) void pack_decode_kernel(const uint32_t* __restrict__ packed, int64_t N, int cw, uint32_t segs, uint32_t inverse,
                                                          uint32_t units, int q, q_u32x4* __restrict__ tiled) {
    const int lane = threadIdx.x & 63;
    const uint32_t unit = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (unit >= units) return;
    const uint32_t rt = inverse ? __umulhi(unit, inverse) : unit;
    const int seg = (int)(unit - rt * segs);
    const int64_t n = (int64_t)rt * 16 + (lane & 15);
    const int w0 = 16 * seg + 4 * (lane >> 4), i0 = 2 * (int)blockIdx.y;
    q_u32x4 v[2] = {{0u, 0u, 0u, 0u}, {0u, 0u, 0u, 0u}};
    if (n < N) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            if (i0 + p >= q) continue;
            const uint32_t* src = packed + ((int64_t)(i0 + p) * N + n) * cw + w0;
            if (QUAD) {
                if (w0 < cw) v[p] = *reinterpret_cast<const q_u32x4*>(src);
            } else {
#pragma unroll
                for (int jj = 0; jj < 4; ++jj)
                    if (w0 + jj < cw) v[p][jj] = src[jj];
            }
        }
    }
    q_u32x4* dst = tiled + ((int64_t)unit * q + i0) * 64 + lane;
#pragma unroll
    for (int p = 0; p < 2; ++p)
        if (i0 + p < q) __builtin_nontemporal_store(v[p], dst + p * 64);
}

size_t decode_layout_bytes(int64_t N, int64_t K, int q) {
    return (size_t)((N + 15) / 16) * (size_t)((K + 511) / 512) * (size_t)q * 1024;
}

hipError_t launch_pack_decode(const uint32_t* packed, int64_t N, int64_t K, int q, uint32_t* tiled, hipStream_t st) {
    const int cw = (int)(K / 32);
    const uint32_t segs = (uint32_t)((K + 511) / 512), units = (uint32_t)((N + 15) / 16) * segs;  // at most 2^13 * 2^8
    const uint32_t inverse = (uint32_t)((((uint64_t)1 << 32) + segs - 1) / segs);
    const dim3 grid((units + 3) / 4, (unsigned)((q + 1) / 2));
    if (cw % 4 == 0)
        BCQ_LAUNCH(pack_decode_kernel<true>, grid, dim3(256), 0, st, packed, N, cw, segs, inverse, units, q, reinterpret_cast<q_u32x4*>(tiled));
    else
        BCQ_LAUNCH(pack_decode_kernel<false>, grid, dim3(256), 0, st, packed, N, cw, segs, inverse, units, q, reinterpret_cast<q_u32x4*>(tiled));
    return hipGetLastError();
}

hipError_t launch_bwd_alpha_stream(const uint32_t* packed, const void* x, const void* dy, int64_t T, int64_t N,
                                   int64_t K, int64_t g, int q, int q_train, float grad_scale, float* dalpha,
                                   void* workspace, hipStream_t st) {
    return launch_stream<STREAM_DALPHA>(packed, (const bf16_t*)x, nullptr, (const bf16_t*)dy, dalpha, T, N, K / 32, q,
                                        q_train, grad_scale, workspace, g, K, st);
}

hipError_t launch_bwd_input_stream(const uint32_t* packed_t, const float* alpha, const void* dy, int64_t T, int64_t N,
                                   int64_t K, int64_t g, int q, void* dx, void* workspace, hipStream_t st) {
    return launch_stream<STREAM_DX>(packed_t, (const bf16_t*)dy, alpha, nullptr, dx, T, K, N / 32, q, q, 1.f, workspace,
                                    g, K, st);
}

}  // namespace bcq

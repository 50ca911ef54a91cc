// Alternating BCQ quantizer (AlphaTuning Appendix C, "Alternating Method", Eq. ap4): greedy start (Eq. ap1-ap3),
// then `iters` rounds of
//   (1) alpha <- (B^T B)^{-1} B^T w      least-squares refit of the q scales of one vector (Eq. ap4),
//   (2) every element takes the sign pattern whose level sum_i +-alpha_i is nearest to its weight.
// One workgroup of one to four waves per vector (a row, or one length-g group of a row), specialised by q.  The vector
// (fp32) and one byte of sign pattern per element stay in LDS for all rounds, so W is read from HBM once.
//
// Arithmetic: every sum, the solve (L D L^T) and the level comparison are fp64; alpha is rounded to fp32 once at
// the end.  The loop stops early at a fixed point (round (2) changed nothing) and stops BEFORE a refit whose
// Gram matrix is singular (a pivot <= 1e-9 n: two planes equal or opposite, e.g. an all-zero vector),
// keeping the current pair.  Ties between two levels go to the larger level, ties between equal levels to the
// larger pattern index (bit i of the pattern = plane i is +1).  Only the ORDER of the fp64 sums over the
// elements is free.
//
// What bounds it: a round is a chain of two barriers, a cross-lane fp64 sum, the solve (q dependent fp64 divisions; with
// square roots and a division per entry a dozen at q = 3) and 2^q distances per element.  Therefore a round makes ONE
// pass over the elements (the re-assignment and the next round's sums together), the Gram matrix is counted in integers
// from the pattern bytes (its entries are n - 2 * disagreements, exact), only wave 0 solves, and the levels are sorted
// so that a distance costs one subtraction, one strict comparison and its selects.  Four elements per lane, so that
// vectors of at most 256 elements (groups) take one wave and no cross-wave step.  Measured: 1024 x 1024, q = 3, 15
// rounds 735 -> 68 us (86 us with the sums through LDS shuffles and a Cholesky solve; before, a kernel for every q
// reduced 36 fp64 sums per round over four waves and solved in all of them).
#include "bcq_internal.h"

namespace bcq {

constexpr int ALT_MAX_WAVES = 4;

template <int Q>
struct AltShared {
    static constexpr int PAIRS = Q * (Q - 1) / 2, LEVELS = 1 << Q;
    double rhs[ALT_MAX_WAVES][Q];                             // partial B^T w (greedy start: [0] = partial |residual|)
    double alpha[Q];
    double raw[LEVELS], level[LEVELS];                        // by pattern; in descending order
    uint32_t disagree[ALT_MAX_WAVES][(PAIRS + 1) / 2 + 1];    // two 16-bit counts per word
    uint32_t changed[ALT_MAX_WAVES];
    uint32_t stop;
    uint8_t pattern[LEVELS];                                  // of the sorted levels
};

// The first of the smallest distances |x - level[c]| over descending levels, by bisection: the level above x and the one
// below, then upwards over equal distances (equal levels, or ones that the rounding of the distance makes equal).  Any
// index in range when x or a level is not finite.
template <int LEVELS>
__device__ __forceinline__ int nearest_level(const double* level, double x) {
    int pos = 0;  // levels above x
#pragma unroll
    for (int step = LEVELS / 2; step >= 1; step >>= 1) pos += level[pos + step - 1] > x ? step : 0;
    pos += level[pos] > x ? 1 : 0;
    const int below = pos < LEVELS ? pos : LEVELS - 1;
    if (pos == 0) return 0;
    const double above = fabs(x - level[pos - 1]);
    if (pos < LEVELS && !(above <= fabs(x - level[below]))) return below;
    int best = pos - 1;
    while (best > 0 && fabs(x - level[best - 1]) <= above) --best;
    return best;
}
// 2^q distances per element, or q steps and two distances: at four planes the distances, which need no per-lane addresses,
// hold (1024 x 1024 115 us); from five on bisection is faster at every size timed (15 rounds, us): 1024 x 1024 q = 5 259 ->
// 140, q = 8 1898 -> 1242; 8 vectors of 256, q = 8, one wave each 743 -> 519 (565 with four waves and distances).
constexpr int ALT_BISECT_FROM = 5;

template <int Q>
__global__ __launch_bounds__(64 * ALT_MAX_WAVES) void alternating_kernel(const float* __restrict__ W, int64_t V, int n,
                                                                         int iters, float* __restrict__ alpha,
                                                                         uint32_t* __restrict__ packed,
                                                                         int8_t* __restrict__ planes,
                                                                         int* __restrict__ status_word) {
    using Shared = AltShared<Q>;
    constexpr int PAIRS = Shared::PAIRS, LEVELS = Shared::LEVELS, PW = (PAIRS + 1) / 2;
    extern __shared__ __attribute__((aligned(16))) unsigned char alt_smem[];
    Shared& sh = *reinterpret_cast<Shared*>(alt_smem);
    float4* w4 = reinterpret_cast<float4*>(alt_smem + (sizeof(Shared) + 15) / 16 * 16);  // [n / 4]
    uint32_t* code4 = reinterpret_cast<uint32_t*>(w4 + n / 4);                           // [n / 4], a pattern per byte
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, waves = blockDim.x >> 6;
    const int quads = n / 4;
    const int64_t v = blockIdx.x;
    const float4* wrow = reinterpret_cast<const float4*>(W + v * (int64_t)n);

    // waves' partial sums, in wave order
    auto total_rhs = [&](int i) {
        double s = sh.rhs[0][i];
        for (int u = 1; u < waves; ++u) s += sh.rhs[u][i];
        return s;
    };

    // ---- greedy start: plane i takes the sign of the residual w - sum_{j<i} alpha_j b_j (each element's residual
    // is rebuilt from its pattern so far, by the same chain of fp64 subtractions), alpha_i = fp32(mean |residual|).
    // A lane only touches its own quads until the packed words are formed.
    double a[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) a[i] = 0.0;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        double s = 0.0;
        for (int k = tid; k < quads; k += blockDim.x) {
            float4 x;
            if (i == 0) {
                x = wrow[k];
                w4[k] = x;
            } else {
                x = w4[k];
            }
            const float xs[4] = {x.x, x.y, x.z, x.w};
            uint32_t c = (i == 0) ? 0u : code4[k];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                double r = (double)xs[e];
#pragma unroll
                for (int j = 0; j < i; ++j) r = ((c >> (8 * e + j)) & 1u) ? r - a[j] : r + a[j];
                s += fabs(r);
                c |= (r >= 0.0 ? 1u : 0u) << (8 * e + i);
            }
            code4[k] = c;
        }
        s = wave_sum(s);
        if (i) __syncthreads();  // the previous plane's partial sums have been read
        if (lane == 0) sh.rhs[wave][0] = s;
        __syncthreads();
        s = total_rhs(0);
        if (i == 0 && tid == 0 && status_word && !(fabs(s) <= 1.79769313486231570e308)) atomicAdd(status_word, 1);
        a[i] = (double)(float)(s / (double)n);
    }
    __syncthreads();

    // right-hand side B^T w of this wave and its counts of disagreeing signs, from the patterns c of four elements
    double rhs[Q];
    uint32_t dis[PAIRS + 1];
    auto clear_sums = [&]() {
#pragma unroll
        for (int i = 0; i < Q; ++i) rhs[i] = 0.0;
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) dis[p] = 0u;
    };
    auto add_sums = [&](const double (&x)[4], uint32_t c) {
        int p = 0;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
#pragma unroll
            for (int e = 0; e < 4; ++e) rhs[i] += ((c >> (8 * e + i)) & 1u) ? x[e] : -x[e];
#pragma unroll
            for (int j = 0; j < i; ++j) dis[p++] += __popc(((c >> i) ^ (c >> j)) & 0x01010101u);
        }
    };
    auto publish_sums = [&]() {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const double s = wave_sum(rhs[i]);
            if (lane == 0) sh.rhs[wave][i] = s;
        }
#pragma unroll
        for (int p = 0; p < PW; ++p) {  // a count is at most n <= 16384: two fit one word
            const uint32_t s = wave_sum(dis[2 * p] + ((2 * p + 1 < PAIRS ? dis[2 * p + 1] : 0u) << 16));
            if (lane == 0) sh.disagree[wave][p] = s;
        }
    };
    if (iters > 0) {
        clear_sums();
        for (int k = tid; k < quads; k += blockDim.x) {
            const float4 xf = w4[k];
            const double x[4] = {(double)xf.x, (double)xf.y, (double)xf.z, (double)xf.w};
            add_sums(x, code4[k]);
        }
        publish_sums();
        __syncthreads();
    }

    for (int it = 0; it < iters; ++it) {
        // ---- (1) Eq. ap4, by wave 0: L D L^T of the Gram matrix B^T B (diagonal = n), all lanes on the same numbers
        if (wave == 0) {
            double L[Q][Q], M[Q][Q], inv[Q], z[Q];  // G = L D L^T with unit diagonal in L, M = L D, inv = 1 / D
            bool singular = false;
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                if (!singular) {
                    double d = (double)n;
#pragma unroll
                    for (int p = 0; p < j; ++p) d -= M[j][p] * L[j][p];
                    if (!(d > 1e-9 * (double)n)) {
                        singular = true;
                    } else {
                        inv[j] = 1.0 / d;
#pragma unroll
                        for (int i = j + 1; i < Q; ++i) {
                            const int pr = i * (i - 1) / 2 + j;
                            uint32_t cnt = 0u;
                            for (int u = 0; u < waves; ++u) cnt += (sh.disagree[u][pr >> 1] >> (16 * (pr & 1))) & 0xFFFFu;
                            double s = (double)(n - 2 * (int)cnt);
#pragma unroll
                            for (int p = 0; p < j; ++p) s -= M[i][p] * L[j][p];
                            M[i][j] = s;
                            L[i][j] = s * inv[j];
                        }
                    }
                }
            }
            if (!singular) {  // uniform: all lanes hold the same numbers
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    z[i] = total_rhs(i);
#pragma unroll
                    for (int p = 0; p < i; ++p) z[i] -= L[i][p] * z[p];
                }
#pragma unroll
                for (int i = Q - 1; i >= 0; --i) {
                    double s = z[i] * inv[i];
#pragma unroll
                    for (int p = i + 1; p < Q; ++p) s -= L[p][i] * a[p];
                    a[i] = s;
                }
                // levels of the new alpha, sorted by (level, pattern) downwards.  The slots are filled in pattern order
                // first: with non-finite levels the ranks need not be a permutation.
                for (int c = lane; c < LEVELS; c += 64) {
                    double s = 0.0;
#pragma unroll
                    for (int i = 0; i < Q; ++i) s += ((c >> i) & 1) ? a[i] : -a[i];
                    sh.raw[c] = s;
                    sh.level[LEVELS - 1 - c] = s;
                    sh.pattern[LEVELS - 1 - c] = (uint8_t)c;
                }
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // one wave's LDS instructions execute in order
                for (int c = lane; c < LEVELS; c += 64) {
                    const double own = sh.raw[c];
                    int rank = 0;
#pragma unroll 8
                    for (int o = 0; o < LEVELS; ++o) {
                        const double l = sh.raw[o];
                        rank += (l > own || (!(l < own) && o > c)) ? 1 : 0;
                    }
                    sh.level[rank] = own;
                    sh.pattern[rank] = (uint8_t)c;
                }
            }
            if (lane == 0) sh.stop = singular ? 1u : 0u;
        }
        __syncthreads();
        if (sh.stop) break;
        // ---- (2) the nearest level for every element: in descending order the first of the smallest distances is the
        // one the tie rules ask for.  The next round's sums are formed from the new pattern in the same pass.
        clear_sums();
        uint32_t diff = 0u;
        for (int k = tid; k < quads; k += blockDim.x) {
            const float4 xf = w4[k];
            const double x[4] = {(double)xf.x, (double)xf.y, (double)xf.z, (double)xf.w};
            int best[4];
            if constexpr (Q >= ALT_BISECT_FROM) {
#pragma unroll
                for (int e = 0; e < 4; ++e) best[e] = nearest_level<LEVELS>(sh.level, x[e]);
            } else {
                double bd[4];
                const double l0 = sh.level[0];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    bd[e] = fabs(x[e] - l0);
                    best[e] = 0;
                }
#pragma unroll 8
                for (int c = 1; c < LEVELS; ++c) {
                    const double l = sh.level[c];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const double d = fabs(x[e] - l);
                        const bool nearer = d < bd[e];
                        bd[e] = nearer ? d : bd[e];
                        best[e] = nearer ? c : best[e];
                    }
                }
            }
            uint32_t c4 = 0u;
#pragma unroll
            for (int e = 0; e < 4; ++e) c4 |= (uint32_t)sh.pattern[best[e]] << (8 * e);
            diff |= c4 ^ code4[k];
            code4[k] = c4;
            add_sums(x, c4);
        }
        const bool wave_changed = __any(diff != 0u);
        if (lane == 0) sh.changed[wave] = wave_changed ? 1u : 0u;
        publish_sums();
        __syncthreads();
        uint32_t changed = 0u;
        for (int u = 0; u < waves; ++u) changed |= sh.changed[u];
        if (!changed) break;
    }
    __syncthreads();

    // ---- outputs: alpha[i][v], packed[i][v][n / 32], planes[i][v][n]
    const int nw = n / 32;
    if (tid == 0) {
#pragma unroll
        for (int i = 0; i < Q; ++i) alpha[(int64_t)i * V + v] = (float)a[i];
    }
    for (int idx = tid; idx < Q * nw; idx += blockDim.x) {
        const int i = idx / nw, wq = idx % nw;
        uint32_t word = 0u;
#pragma unroll
        for (int b = 0; b < 8; ++b)  // bits 0, 8, 16, 24 of a pattern quad -> a nibble
            word |= (((((code4[8 * wq + b] >> i) & 0x01010101u) * 0x01020408u) >> 24) & 0xFu) << (4 * b);
        packed[((int64_t)i * V + v) * nw + wq] = word;
    }
    if (planes) {
        uint32_t* out = reinterpret_cast<uint32_t*>(planes);
        for (int i = 0; i < Q; ++i)
            for (int k = tid; k < quads; k += blockDim.x)  // a byte per element: 1 -> 0x01, 0 -> 0xFF
                out[((int64_t)i * V + v) * quads + k] = ~(((code4[k] >> i) & 0x01010101u) * 0xFEu);
    }
}

__global__ void alt_zero_word_kernel(int* p) { *p = 0; }

template <int Q>
static hipError_t launch_q(const float* W, int64_t V, int n, int iters, float* alpha, uint32_t* packed, int8_t* planes,
                           int* status_word, hipStream_t st) {
    const size_t lds = (sizeof(AltShared<Q>) + 15) / 16 * 16 + (size_t)n * 5;
    static LdsLimit limit;
    hipError_t e = limit.ensure((const void*)alternating_kernel<Q>, lds);
    if (e != hipSuccess) return e;
    // Four elements per lane and pass.  One / two / four waves, 15 rounds, q = 3, us: 8 vectors of 128 31 / 35 / 42, 8192 of
    // them 99 / 141 / 259; 4096 of 256 65 / 100 / 170; 8 and 256 of 512 41 / 38 / 46; 256 of 1024 60 / 48 / 47, 1024 of them
    // 63 / 62 / 70; 1024 of 2560 117 / 106 / 109.
    const int waves = n <= 256 ? 1 : n <= 512 ? 2 : ALT_MAX_WAVES;
    BCQ_LAUNCH((alternating_kernel<Q>), dim3((unsigned)V), dim3(64 * waves), lds, st, W, V, n, iters, alpha, packed,
                       planes, status_word);
    return hipGetLastError();
}

hipError_t launch_quantize_alternating(const float* W, int64_t V, int64_t n, int q, int iters, float* alpha,
                                       uint32_t* packed, int8_t* planes, int* status_word, hipStream_t st) {
    if (status_word) {
        BCQ_LAUNCH(alt_zero_word_kernel, dim3(1), dim3(1), 0, st, status_word);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    switch (q) {
        case 1: return launch_q<1>(W, V, (int)n, iters, alpha, packed, planes, status_word, st);
        case 2: return launch_q<2>(W, V, (int)n, iters, alpha, packed, planes, status_word, st);
        case 3: return launch_q<3>(W, V, (int)n, iters, alpha, packed, planes, status_word, st);
        case 4: return launch_q<4>(W, V, (int)n, iters, alpha, packed, planes, status_word, st);
        case 5: return launch_q<5>(W, V, (int)n, iters, alpha, packed, planes, status_word, st);
        case 6: return launch_q<6>(W, V, (int)n, iters, alpha, packed, planes, status_word, st);
        case 7: return launch_q<7>(W, V, (int)n, iters, alpha, packed, planes, status_word, st);
        default: return launch_q<8>(W, V, (int)n, iters, alpha, packed, planes, status_word, st);
    }
}

}  // namespace bcq

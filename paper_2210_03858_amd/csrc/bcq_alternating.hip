// Alternating BCQ quantizer (AlphaTuning Appendix C, "Alternating Method", Eq. ap4): greedy start (Eq. ap1-ap3),
// then `iters` rounds of
//   (1) alpha <- (B^T B)^{-1} B^T w      least-squares refit of the q scales of one vector (Eq. ap4),
//   (2) every element takes the sign pattern whose level sum_i +-alpha_i is nearest to its weight.
// One workgroup of one or more waves per vector (a row, or one length-g group of a row), specialised by q; W is read from HBM
// once.
//
// Arithmetic: every sum, the solve (L D L^T) and the level comparison are fp64; alpha is rounded to fp32 once at
// the end.  The loop stops early at a fixed point (round (2) changed nothing) and stops BEFORE a refit whose
// Gram matrix is singular (a pivot <= 1e-9 n: two planes equal or opposite, e.g. an all-zero vector),
// keeping the current pair.  Ties between two levels go to the larger level, ties between equal levels to the
// larger pattern index (bit i of the pattern = plane i is +1).  Only the ORDER of the fp64 sums over the
// elements is free.
//
// From five planes on, and with one plane above 1024 elements (alternating_kernel), the vector (fp32) and one byte of sign
// pattern per element stay in LDS.  A round is
// a chain of two barriers, a cross-lane fp64 sum, the solve (q dependent fp64 divisions) and q steps of bisection per
// element; it makes ONE pass over the elements (the re-assignment and the next round's sums together), counts the
// Gram matrix in integers from the pattern bytes (its entries are n - 2 * disagreements, exact) and only wave 0 solves.
//
// Up to four planes (alternating_reg_kernel) the elements stay in registers, up to 32 per lane, and a round compares no
// distances: the weights are fp32, so the place where the nearest level changes is one fp32 number per pair of
// neighbouring levels, found by the distances themselves at the three floats around their middle.  The levels lie
// symmetrically about zero, so |w| is compared with the 2^(q-1) - 1 thresholds of the positive half and the sign of w
// mirrors the pattern.  Where that might not decide as the distances do (equal or nearly equal levels, a tie at a float, elements
// far smaller or larger than the levels, non-finite ones) the round takes the fp64 distances.  What bounds it: the
// chain of a round, about 20 vector operations per element, one joint cross-lane sum of all totals, the solve and the sorting,
// which every wave does for itself, so that a vector of one wave meets no barrier and any other one per round.  Measured:
// 15 rounds of 1024 x 1024: q = 3 72 -> 27 us, q = 4 119 -> 38 (against four waves, the vector in LDS and 2^q fp64
// distances per element).
//
// Where enough rounds are allowed (sort_rounds below), for vectors of one wave and with three planes of up to four (RANKED): all that a
// round needs of the elements is how many lie below each threshold and their
// sum, as every sum is a combination of those of the cells between the thresholds.  So the wave sorts the |w| once (6000
// cycles, about 1400 operations) and keeps the sums of the first of them; a threshold is then found by one comparison of the lanes'
// smallest elements and one of 16 elements, and the greedy start is found the same way.  A round of q = 3 takes 1800 cycles for 3450: solve
// 530, levels and thresholds 400 (1020 with sorting them anew: the last order is only confirmed), the search 600 where the
// elements took 1880; far code out of the loop's way is worth 500 of it, a lone wave waits for every jump.  15 rounds, us, normal weights,
// element by element -> sorted, 1024 vectors of 1024, q = 2, 3, 4: 18.1, 27.1, 38.8 -> 14.7, 18.6, 28.3; 8192 of them 64, 135, 205 -> 58, 91,
// 141; 8192 of 256 32, 74, 116 -> 25, 53, 99.  Rounds that change the levels' order, and vectors with single far elements, gain less: where waves
// are alone on their vector units the slowest vector decides, 1024 of 256, q = 4, with 0.5 % of eightfold weights 32 -> 37; weights peaked at zero
// (cubes of normal ones) 1.00 to 1.25 times the time, of several waves 1.1 to 1.5: their registers leave room for fewer waves, and their
// rounds are element by element.  Several waves sort apart and add their sums and counts at the round's barrier: q = 3, 15 rounds, 1024 vectors of
// 1280, 2560, 4096 49, 74, 86 -> 35, 64, 76.  They are compiled for three waves to a vector unit, for which 17 registers spill (64 bytes
// a lane): without spills two fit, 1638 vectors of 2560 0.78 / 0.95 of the time element by element, 1024 of 4096 0.88 / 0.87.  With two
// planes a round of several waves has too little to save (1024 of 2560 44 / 47), with four that register limit spills far more (129 / 200).
#include <type_traits>

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
    if constexpr (LEVELS == 2) return fabs(x - level[1]) < fabs(x - level[0]) ? 1 : 0;
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
#pragma unroll
            for (int e = 0; e < 4; ++e) best[e] = nearest_level<LEVELS>(sh.level, x[e]);
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

// ---- up to four planes -----------------------------------------------------------------------------------------

// Sums over the 64 lanes of NV values (NV a power of two), the same in every lane.  The first log2(NV) exchange steps halve
// the number of values a lane carries (a lane passes on what its partner keeps), so that the others move one value.
template <int NV>
__device__ __forceinline__ void wave_sums(double (&v)[NV]) {
    static_assert(NV == 1 || NV == 2 || NV == 4 || NV == 8, "a power of two");
    const int lane = threadIdx.x & 63;
    auto step = [&](auto COUNT, auto CTRL, bool upper) {  // COUNT values -> COUNT / 2
        constexpr int half = decltype(COUNT)::value / 2;
#pragma unroll
        for (int i = 0; i < half; ++i) {
            const double keep = upper ? v[i + half] : v[i], pass = upper ? v[i] : v[i + half];
            v[i] = keep + dpp_move<decltype(CTRL)::value>(pass);
        }
    };
    using std::integral_constant;
    constexpr int ROR4 = 0x124, ROR8 = 0x128, ROR1 = 0x121, ROR2 = 0x122;  // rotations inside a row of 16 lanes
    if constexpr (NV == 8) step(integral_constant<int, 8>{}, integral_constant<int, DPP_HALF_MIRROR>{}, (lane & 4) != 0);
    // (the mirror turns the places of 1 and 2 over as well: the next steps count them from there)
    if constexpr (NV >= 4) step(integral_constant<int, 4>{}, integral_constant<int, DPP_XOR1>{}, (lane & 1) != 0);
    if constexpr (NV >= 2) step(integral_constant<int, 2>{}, integral_constant<int, NV == 2 ? DPP_XOR1 : DPP_XOR2>{}, (lane & (NV == 2 ? 1 : 2)) != 0);
    double r = v[0];
    r += dpp_move<ROR8>(r);
    if constexpr (NV <= 4) r += dpp_move<ROR4>(r);
    if constexpr (NV <= 2) r += dpp_move<ROR2>(r);
    if constexpr (NV == 1) r += dpp_move<ROR1>(r);
    auto rows = [&](auto swap) {  // both operands the same value: the sums of pairs of rows
        const auto lo = swap((uint32_t)__double2loint(r)), hi = swap((uint32_t)__double2hiint(r));
        r = __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
    };
    rows([](uint32_t x) { return __builtin_amdgcn_permlane16_swap(x, x, false, false); });
    rows([](uint32_t x) { return __builtin_amdgcn_permlane32_swap(x, x, false, false); });
#pragma unroll
    for (int i = 0; i < NV; ++i) {  // the lane that holds value i
        const int l = NV == 1 ? 0 : NV == 2 ? i : NV == 4 ? (i >> 1) + 2 * (i & 1) : ((i >> 2) << 2) + ((i >> 1) & 1) + 2 * (i & 1);
        v[i] = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(r), l), __builtin_amdgcn_readlane(__double2loint(r), l));
    }
}

// Ascending order of the NE values of a lane, by odd-even merges (Batcher).
template <int NE>
__device__ __forceinline__ void sort_lane(uint32_t (&m)[NE]) {
#pragma unroll
    for (int p = 1; p < NE; p *= 2)
#pragma unroll
        for (int k = p; k >= 1; k /= 2)
#pragma unroll
            for (int j = k % p; j + k < NE; j += 2 * k)
#pragma unroll
                for (int i = 0; i < k; ++i)
                    if (i + j + k < NE && (i + j) / (2 * p) == (i + j + k) / (2 * p)) {
                        const uint32_t lo = m[i + j], hi = m[i + j + k];
                        m[i + j] = lo < hi ? lo : hi;
                        m[i + j + k] = lo < hi ? hi : lo;
                    }
}

// Ascending order of the 64 NE values of a wave (lane l ends with values NE l .. + NE - 1): the lanes' sorted runs are merged in pairs,
// a run with the mirror image of the next one first (which needs no descending runs), then at half the distance and so on.  The values
// are bits of non-negative floats: the smaller of two is their median with 0, the larger that with infinity, so that a lane keeps its
// side of an exchange in one operation.
template <int NE>
__device__ __forceinline__ void sort_wave(uint32_t (&m)[NE]) {
    const int lane = threadIdx.x & 63;
    const auto keep = [](uint32_t a, uint32_t b, float side) {
        return __float_as_uint(__builtin_amdgcn_fmed3f(__uint_as_float(a), __uint_as_float(b), side));
    };
    const auto side_of = [&](int bit) { return __uint_as_float((lane & bit) != 0 ? 0x7F800000u : 0u); };
    const auto swap16 = [](uint32_t a) { return __builtin_amdgcn_permlane16_swap(a, a, false, false); };
    const auto swap32 = [](uint32_t a) { return __builtin_amdgcn_permlane32_swap(a, a, false, false); };
    sort_lane(m);
#pragma unroll
    for (int block = 2; block <= 64; block *= 2) {  // lanes of a merged run
        const float upper = side_of(block / 2);
        uint32_t other[NE];
#pragma unroll
        for (int i = 0; i < NE; ++i) {  // of lane ^ (block - 1)
            const uint32_t v = m[NE - 1 - i];
            uint32_t o = block == 2 ? dpp_move<DPP_XOR1>(v) : block == 4 ? dpp_move<DPP_QUAD_REVERSE>(v)
                       : block == 8 ? dpp_move<DPP_HALF_MIRROR>(v) : dpp_move<DPP_MIRROR>(v);
            if (block >= 32) {
                const auto s = swap16(o);
                o = (lane & 16) ? s[0] : s[1];
            }
            if (block >= 64) {
                const auto s = swap32(o);
                o = (lane & 32) ? s[0] : s[1];
            }
            other[i] = o;
        }
#pragma unroll
        for (int i = 0; i < NE; ++i) m[i] = keep(m[i], other[i], upper);
#pragma unroll
        for (int d = block / 4; d >= 1; d /= 2) {
            const float side = side_of(d);
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                const uint32_t v = m[i];
                if (d >= 16) {  // (both values of the exchange in every lane)
                    const auto s = d == 32 ? swap32(v) : swap16(v);
                    m[i] = keep(s[0], s[1], side);
                } else {
                    constexpr int ROR8 = 0x128;
                    const uint32_t o = d == 8 ? dpp_move<ROR8>(v) : d == 4 ? dpp_move<DPP_QUAD_REVERSE>(dpp_move<DPP_HALF_MIRROR>(v))
                                     : d == 2 ? dpp_move<DPP_XOR2>(v) : dpp_move<DPP_XOR1>(v);
                    m[i] = keep(v, o, side);
                }
            }
        }
#pragma unroll
        for (int d = NE / 2; d >= 1; d /= 2)
#pragma unroll
            for (int i = 0; i < NE; ++i)
                if ((i & d) == 0) {
                    const uint32_t lo = m[i], hi = m[i + d];
                    m[i] = lo < hi ? lo : hi;
                    m[i + d] = lo < hi ? hi : lo;
                }
    }
}

// the largest of the lanes' values, in every lane
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
    const auto larger = [](uint32_t a, uint32_t b) { return a > b ? a : b; };
    v = larger(v, dpp_move<DPP_XOR1>(v));
    v = larger(v, dpp_move<DPP_XOR2>(v));
    v = larger(v, dpp_move<DPP_HALF_MIRROR>(v));
    v = larger(v, dpp_move<DPP_MIRROR>(v));
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = larger(a[0], a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return larger(b[0], b[1]);
}

// Sum of the values of the lanes before this one.
__device__ __forceinline__ double sum_before(double v) {
    using std::integral_constant;
    constexpr int SHR = 0x110;  // from the lane n places down in the row of 16, zero where there is none
    const auto from = [](double x, auto N) {
        constexpr int c = SHR + decltype(N)::value;
        return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), c, 0xF, 0xF, true),
                                __builtin_amdgcn_update_dpp(0, __double2loint(x), c, 0xF, 0xF, true));
    };
    v += from(v, integral_constant<int, 1>{});
    v += from(v, integral_constant<int, 2>{});
    v += from(v, integral_constant<int, 4>{});
    v += from(v, integral_constant<int, 8>{});
    const auto at = [&](int l) {
        return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
    };
    const double r0 = at(15), r1 = r0 + at(31), r2 = r1 + at(47);
    const int row = (threadIdx.x & 63) >> 4;
    return from(v, integral_constant<int, 1>{}) + (row == 0 ? 0.0 : row == 1 ? r0 : row == 2 ? r1 : r2);
}

template <int Q, int MW>
struct AltRegShared {
    static constexpr int LEVELS = 1 << Q, PAIRS = Q * (Q - 1) / 2, SUMS = Q + (PAIRS + 2) / 3, TH = LEVELS > 2 ? LEVELS / 2 - 1 : 1;
    double part[2][MW][SUMS > TH ? SUMS : TH];  // waves' totals of a round, rounds in turn: sums, or those below the thresholds
    uint32_t under[2][MW][TH];                // and the elements below them
    double absolute[MW];                      // sums of |w|
    double level[MW][LEVELS], raw[MW][LEVELS];  // every wave sorts for itself
    uint32_t changed[2][MW];
    uint32_t extreme[MW][2];                  // `low` and `high` of the waves
    uint8_t pattern[MW][LEVELS];
};

// QL: quads of elements per lane; MW: waves at most; RANKED: rounds from the sorted elements.
template <int Q, int QL, int MW, bool RANKED>
__global__ __launch_bounds__(64 * MW, RANKED && MW > 1 ? 3 : 1) void alternating_reg_kernel(const float* __restrict__ W, int64_t V, int n, int iters,
                                                                  float* __restrict__ alpha, uint32_t* __restrict__ packed,
                                                                  int8_t* __restrict__ planes, int* __restrict__ status_word) {
    using Shared = AltRegShared<Q, MW>;
    constexpr int PAIRS = Shared::PAIRS, LEVELS = Shared::LEVELS, HALF = LEVELS / 2, SUMS = Shared::SUMS;
    constexpr int NV = SUMS <= 1 ? 1 : SUMS <= 2 ? 2 : SUMS <= 4 ? 4 : 8;
    constexpr int NE = 4 * QL, TH = Shared::TH;
    static_assert(!RANKED || (Q > 1 && QL <= 4), "16 elements of a lane to a search");
    extern __shared__ __attribute__((aligned(16))) unsigned char alt_smem[];
    Shared& sh = *reinterpret_cast<Shared*>(alt_smem);
    uint32_t* code4 = reinterpret_cast<uint32_t*>(alt_smem + (sizeof(Shared) + 15) / 16 * 16);  // [n / 4], for the output
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int waves = MW == 1 ? 1 : blockDim.x >> 6;
    const int quads = n / 4;
    const int64_t v = blockIdx.x;
    const float4* wrow = reinterpret_cast<const float4*>(W + v * (int64_t)n);

    // this lane's elements: quad tid + u * blockDim.x; beyond the vector zeros with all signs equal, which add nothing
    float x[QL][4];
    uint32_t code[QL], mask[QL];
#pragma unroll
    for (int u = 0; u < QL; ++u) {
        const int k = tid + u * 64 * waves;
        const float4 f = k < quads ? wrow[k] : float4{0.f, 0.f, 0.f, 0.f};
        mask[u] = k < quads ? ~0u : 0u;
        code[u] = 0u;
        x[u][0] = f.x + 0.f;  // -0 becomes +0
        x[u][1] = f.y + 0.f;
        x[u][2] = f.z + 0.f;
        x[u][3] = f.w + 0.f;
    }

    const auto of_lane = [](double v, int l) {
        return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
    };

    // Smallest non-zero and largest |w| as bits, which order like the numbers (0 - 1 and so zeros come last).
    uint32_t low = 0u, high = 0u;
#pragma unroll
    for (int u = 0; u < QL; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t m = __float_as_uint(x[u][e]) & 0x7FFFFFFFu;
            low = ~m + 1u > low ? ~m + 1u : low;
            high = m > high ? m : high;
        }
    low = wave_max(low);
    high = wave_max(high);
    if (MW > 1) {
        if (lane == 0) {
            sh.extreme[wave][0] = low;
            sh.extreme[wave][1] = high;
        }
        __syncthreads();
        for (int u = 0; u < waves; ++u) {
            low = sh.extreme[u][0] > low ? sh.extreme[u][0] : low;
            high = sh.extreme[u][1] > high ? sh.extreme[u][1] : high;
        }
    }
    const float smallest = low ? __uint_as_float(0u - low) : 3.402823466e38f, largest = __uint_as_float(high);
    // Not with an element so small against the levels (the largest of which is rarely below an eighth of the largest element) that every
    // round will take the fp64 distances: such a vector would pay for its sorting and not use it (q = 4, cubes of normal weights, 15 rounds,
    // us, sorted / not: 65536 vectors of 128 882 / 740).
    const bool ranked = RANKED && __all(high < 0x7F800000u && smallest >= 1.2e-10f * largest);
    // Sorted |w| of the wave (beyond the vector above every threshold), at lane * (NE + 1) + i, and the sums of the first of them, that of
    // the first NE l + i at 65 i + l: all that a round needs of the elements is how many lie below each threshold, and their sum.
    double* const prefixes = reinterpret_cast<double*>(alt_smem + (sizeof(Shared) + 15) / 16 * 16 + (n + 15) / 16 * 16);
    double* const prefix = prefixes + wave * (65 * NE);
    uint32_t* const sorted = reinterpret_cast<uint32_t*>(prefixes + waves * (65 * NE)) + wave * (64 * (NE + 1));
    uint32_t lane_first = 0u;  // the smallest of the lane's NE
    double absolute = 0.0;
    if (ranked) {
        uint32_t m[NE];
#pragma unroll
        for (int u = 0; u < QL; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) m[4 * u + e] = mask[u] ? __float_as_uint(x[u][e]) & 0x7FFFFFFFu : 0x7F800000u;
        sort_wave(m);
        lane_first = m[0];
        double upto[NE + 1];
        upto[0] = 0.0;
#pragma unroll
        for (int i = 0; i < NE; ++i) upto[i + 1] = upto[i] + (m[i] < 0x7F800000u ? (double)__uint_as_float(m[i]) : 0.0);
        const double before = sum_before(upto[NE]);
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            sorted[lane * (NE + 1) + i] = m[i];
            prefix[65 * i + lane] = before + upto[i];
        }
        if (lane == 63) prefix[64] = before + upto[NE];
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        absolute = of_lane(before + upto[NE], 63);
        if (MW > 1) {
            if (lane == 0) sh.absolute[wave] = absolute;
            __syncthreads();
            absolute = 0.0;
            for (int u = 0; u < waves; ++u) absolute += sh.absolute[u];
        }
    }

    // B^T w and, three counts of at most 16384 to a double, the disagreeing signs of pairs of planes
    double sum[NV];
    auto form_sums = [&]() {
        double rhs[Q];
        uint32_t dis[PAIRS + 1];
#pragma unroll
        for (int i = 0; i < Q; ++i) rhs[i] = 0.0;
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) dis[p] = 0u;
#pragma unroll
        for (int u = 0; u < QL; ++u) {
            const uint32_t c = code[u], inv = ~c;
            int p = 0;
#pragma unroll
            for (int i = 0; i < Q; ++i) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {  // the sign bit flipped where the plane bit is 0
                    const double xd = (double)x[u][e];
                    const uint32_t flip = (inv << (31 - 8 * e - i)) & 0x80000000u;
                    rhs[i] += __hiloint2double(__double2hiint(xd) ^ (int)flip, __double2loint(xd));
                }
#pragma unroll
                for (int j = 0; j < i; ++j) dis[p++] += __popc(((c >> i) ^ (c >> j)) & 0x01010101u);
            }
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) sum[i] = 0.0;
#pragma unroll
        for (int i = 0; i < Q; ++i) sum[i] = rhs[i];
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) sum[Q + p / 3] += (double)dis[p] * (double)(1ll << (16 * (p % 3)));
        wave_sums(sum);
    };
    // the pattern of every element from the thresholds of |w| and the patterns between them; non-zero where one changes
    auto assign = [&](const float (&thr)[HALF], uint64_t lut) {
        const uint32_t lo = (uint32_t)lut, hi = (uint32_t)(lut >> 32);
        float t[HALF];  // (values: of elements of the array the compiler makes branches)
#pragma unroll
        for (int k = 0; k + 1 < HALF; ++k) {
            t[k] = thr[k];
            asm("" : "+v"(t[k]));
        }
        uint32_t diff = 0u;
#pragma unroll
        for (int u = 0; u < QL; ++u) {
            uint32_t sel = 0u, neg = 0u;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float m = fabsf(x[u][e]);
                uint32_t idx = 0u;  // thresholds above |w|
                if constexpr (HALF == 8) {
                    const bool far = m < t[3];
                    const float second = far ? t[5] : t[1], near = far ? t[4] : t[0], other = far ? t[6] : t[2];
                    const bool b = m < second;
                    const float third = b ? other : near;
                    idx = (far ? 4u : 0u) + (b ? 2u : 0u) + (m < third ? 1u : 0u);
                } else {
#pragma unroll
                    for (int k = 0; k + 1 < HALF; ++k) idx += m < t[k] ? 1u : 0u;
                }
                sel |= idx << (8 * e);
                neg |= (uint32_t)((int)__float_as_uint(x[u][e]) >> 31) & ((uint32_t)(LEVELS - 1) << (8 * e));
            }
            const uint32_t c4 = (__builtin_amdgcn_perm(hi, lo, sel) ^ neg) & mask[u];
            diff |= c4 ^ code[u];
            code[u] = c4;
        }
        return diff;
    };
    // Of the last round, while `known`: its thresholds, patterns (outermost first) and the elements and sums below the thresholds; of
    // the patterns, the planes of lane k's level and of the one below it as sign flips, and lane p's part in the sums: the p-th
    // of B^T w, then of the elements of B^T B off its diagonal, as combination of the sums (counts) below the thresholds.  `owed`:
    // the codes are still to be assigned from thresholds and patterns.
    float thr[HALF];
    uint64_t lut = 0u;
    uint32_t flip_up[Q], flip_down[Q];
    double part[HALF];
    int under[TH];
    double below[TH];
    bool known = false, owed = false, from_below = false;
#pragma unroll
    for (int k = 0; k < TH; ++k) {
        under[k] = 0;
        below[k] = 0.0;
    }
    const auto flipped = [](double v, uint32_t flip) { return __hiloint2double(__double2hiint(v) ^ (int)flip, __double2loint(v)); };
    uint32_t planes_of_lane = 1u;  // one plane, or two
    {
        int p = 0;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            planes_of_lane = lane == i ? 1u << i : planes_of_lane;
#pragma unroll
            for (int j = 0; j < i; ++j, ++p) planes_of_lane = lane == Q + p ? (1u << i) | (1u << j) : planes_of_lane;
        }
    }
    const uint32_t pair = lane >= Q ? 1u : 0u;

    const auto describe = [&] {  // flips and parts of the patterns
#pragma unroll
        for (int i = 0; i < Q; ++i) {  // (lanes beyond the last level repeat it)
            const int k = lane < HALF - 1 ? lane : HALF - 1;
            const uint32_t mirrored = k == HALF - 1 ? 1u : 0u, next = (uint32_t)(lut >> (8 * (k + 1 - (int)mirrored)));
            flip_up[i] = ~(uint32_t)(lut >> (8 * k + i)) << 31;
            flip_down[i] = ((next >> i) ^ mirrored ^ 1u) << 31;
        }
        double sign = 0.0;
#pragma unroll
        for (int c = 0; c < HALF; ++c) {  // a plane counts with its sign, a pair with the product of its signs
            const double next = ((uint32_t)__popc((uint32_t)(lut >> (8 * c)) & planes_of_lane) & 1u) != pair ? 1.0 : -1.0;
            part[c] = next - sign;
            sign = next;
        }
    };
    // Of the sorted elements: the last lane whose smallest lies below threshold k, its elements, and the sums up to them; then the number
    // and the sum of all elements below the threshold.
    int first[TH];
    uint32_t near[TH];
    double sums[TH];
    const auto look = [&](int k) {
        const int lanes = __popcll(__ballot(lane_first < __float_as_uint(thr[k])));
        first[k] = lanes > 1 ? lanes - 1 : 0;
        near[k] = sorted[first[k] * (NE + 1) + (lane & (NE - 1))];
        sums[k] = prefix[first[k] + (lane < NE ? 65 * lane : 1)];
    };
    const auto count = [&](int k) {
        const int in = __popcll(__ballot(near[k] < __float_as_uint(thr[k])) & ((1ull << NE) - 1ull));
        below[k] = of_lane(sums[k], in);
        return first[k] * NE + in;
    };
    // ---- greedy start, from the sorted elements: the sign of plane i changes, in every cell of the planes before it, at the cell's level
    // (the sum of their scales with its signs), and alpha_i is the mean distance from there.  Not where an element lies as close
    // to that place as the rounding of the residuals, or all of them do nearly.
    double a[Q];
    bool started = false;
    if constexpr (RANKED) {
        if (ranked) {
            a[0] = (double)(float)(absolute / (double)n);
            double level[HALF];  // of the cells so far, uppermost first
            level[0] = a[0];
            bool close = false;
            int all_under[TH];  // of all waves
            double all_below[TH];
#pragma unroll
            for (int i = 1; i < Q; ++i) {
                constexpr int none = -1;
                const int step = 1 << (Q - 1 - i), cells = 1 << (i - 1);
                double total = 0.0;
#pragma unroll
                for (int c = 0; c < cells; ++c) {
                    const int k = (2 * c + 1) * step - 1, above = c > 0 ? k - step : none, beneath = c + 1 < cells ? k + step : none;
                    const float f = (float)level[c];
                    float t = (double)f < level[c] ? __uint_as_float(__float_as_uint(f) + 1u) : f;
                    t = level[c] > 0.0 ? t : 0.f;
                    if (above != none) t = fminf(t, thr[above]);
                    if (beneath != none) t = fmaxf(t, thr[beneath]);
                    thr[k] = t;
                    look(k);
                }
#pragma unroll
                for (int c = 0; c < cells; ++c) {
                    const int k = (2 * c + 1) * step - 1;
                    const double m = level[c], eps = 1e-14 * a[0];
                    close = close || fabs((double)__uint_as_float(near[k]) - m) <= eps || fabs((double)__uint_as_float(lane_first) - m) <= eps;
                    all_under[k] = under[k] = count(k);
                    all_below[k] = below[k];
                    if (MW > 1 && lane == 0) {
                        sh.part[i & 1][wave][k] = below[k];
                        sh.under[i & 1][wave][k] = (uint32_t)under[k];
                    }
                }
                if (MW > 1) {  // over the waves, in wave order
                    __syncthreads();
#pragma unroll
                    for (int c = 0; c < cells; ++c) {
                        const int k = (2 * c + 1) * step - 1;
                        all_under[k] = 0;
                        all_below[k] = 0.0;
                        for (int u = 0; u < waves; ++u) {
                            all_under[k] += (int)sh.under[i & 1][u][k];
                            all_below[k] += sh.part[i & 1][u][k];
                        }
                    }
                }
#pragma unroll
                for (int c = 0; c < cells; ++c) {
                    const int k = (2 * c + 1) * step - 1, above = c > 0 ? k - step : none, beneath = c + 1 < cells ? k + step : none;
                    const double m = level[c];
                    const int n_above = (above == none ? n : all_under[above]) - all_under[k], n_beneath = all_under[k] - (beneath == none ? 0 : all_under[beneath]);
                    const double s_above = (above == none ? absolute : all_below[above]) - all_below[k];
                    const double s_beneath = all_below[k] - (beneath == none ? 0.0 : all_below[beneath]);
                    total += (s_above - m * (double)n_above) + (m * (double)n_beneath - s_beneath);
                }
                close = close || !(total >= 1e-3 * absolute);  // (their differences keep 2^-40 of it)
                a[i] = (double)(float)(total / (double)n);
#pragma unroll
                for (int c = cells - 1; c >= 0; --c) {
                    const double m = level[c];
                    level[2 * c] = m + a[i];
                    level[2 * c + 1] = m - a[i];
                }
            }
#pragma unroll
            for (int c = 0; c < HALF; ++c) {
                uint64_t pattern = 1u;
#pragma unroll
                for (int i = 1; i < Q; ++i) pattern |= (uint64_t)(((c >> (Q - 1 - i)) & 1) ^ 1) << i;
                lut |= pattern << (8 * c);
            }
            started = MW == 1 ? __all(!close) : __syncthreads_and(!close);
            known = owed = from_below = started;
            describe();
        }
    }
    // ---- greedy start, element by element: plane i takes the sign of the residual w - sum_{j<i} alpha_j b_j (each element's residual
    // is rebuilt from its pattern so far, by the same chain of fp64 subtractions), alpha_i = fp32(mean |residual|).
    if (!started) {
#pragma unroll
        for (int i = 0; i < Q; ++i) a[i] = 0.0;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            double s = 0.0;
#pragma unroll
            for (int u = 0; u < QL; ++u) {
                uint32_t c = code[u];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    double r = (double)x[u][e];
#pragma unroll
                    for (int j = 0; j < i; ++j) r = ((c >> (8 * e + j)) & 1u) ? r - a[j] : r + a[j];
                    s += mask[u] ? fabs(r) : 0.0;
                    c |= (r >= 0.0 ? 1u : 0u) << (8 * e + i);
                }
                code[u] = c & mask[u];
            }
            s = wave_sum(s);
            if (MW > 1) {
                if (lane == 0) sh.part[i & 1][wave][0] = s;
                __syncthreads();
                s = 0.0;
                for (int u = 0; u < waves; ++u) s += sh.part[i & 1][u][0];
            }
            if (i == 0 && tid == 0 && status_word && !(fabs(s) <= 1.79769313486231570e308)) atomicAdd(status_word, 1);
            a[i] = (double)(float)(s / (double)n);
        }
        if (iters > 0) form_sums();
    }

    for (int it = 0; it < iters; ++it) {
        // The exchanges take turns from plane 0 of the greedy start on, round `it` after plane Q - 1: between the reads of one and the next
        // writes of the same buffer lies the other one's barrier, so that no wave overwrites what a slower one still reads.
        const int turn = (Q + it) & 1;
        bool changed_elsewhere = false;
        int all_under[TH];
        double all_below[TH];
#pragma unroll
        for (int k = 0; k < TH; ++k) {
            all_under[k] = under[k];
            all_below[k] = below[k];
        }

        if (MW > 1) {  // totals over the waves, in wave order; every wave leaves the loop with the others
            const bool from = RANKED && from_below;
            if (lane == 0) {
                if (from) {
#pragma unroll
                    for (int k = 0; k < TH; ++k) {
                        sh.part[turn][wave][k] = below[k];
                        sh.under[turn][wave][k] = (uint32_t)under[k];
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < SUMS; ++i) sh.part[turn][wave][i] = sum[i];
                }
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < SUMS; ++i) sum[i] = 0.0;
#pragma unroll
            for (int k = 0; k < TH; ++k) {
                all_under[k] = 0;
                all_below[k] = 0.0;
            }
            for (int u = 0; u < waves; ++u) {
                if (from) {
#pragma unroll
                    for (int k = 0; k < TH; ++k) {
                        all_below[k] += sh.part[turn][u][k];
                        all_under[k] += (int)sh.under[turn][u][k];
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < SUMS; ++i) sum[i] += sh.part[turn][u][i];
                }
                if (it > 0) changed_elsewhere = changed_elsewhere || sh.changed[turn ^ 1][u] != 0u;
            }
            if (it > 0 && !changed_elsewhere) break;
        }
        // B^T w and the elements of B^T B off its diagonal
        double rhs[Q], gram[PAIRS + 1];
        if (RANKED && from_below) {
            double v = part[0] * (pair ? (double)n : absolute);
#pragma unroll
            for (int k = 0; k + 1 < HALF; ++k) v = __builtin_fma(part[k + 1], pair ? (double)all_under[k] : all_below[k], v);
#pragma unroll
            for (int i = 0; i < Q; ++i) rhs[i] = of_lane(v, i);
#pragma unroll
            for (int p = 0; p < PAIRS; ++p) gram[p] = of_lane(v, Q + p);
        } else {
#pragma unroll
            for (int i = 0; i < Q; ++i) rhs[i] = sum[i];
#pragma unroll
            for (int p = 0; p < PAIRS; ++p) {
                const uint64_t counts = (uint64_t)__double_as_longlong(sum[Q + p / 3] + 4503599627370496.0);  // 2^52: an integer in the mantissa
                gram[p] = (double)(n - 2 * (int)((counts >> (16 * (p % 3))) & 0xFFFFu));
            }
        }
        // ---- (1) Eq. ap4: L D L^T of the Gram matrix B^T B (diagonal = n), all lanes on the same numbers
        double L[Q][Q], M[Q][Q], inv[Q], z[Q];  // G = L D L^T with unit diagonal in L, M = L D, inv = 1 / D
        bool singular = false;
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            double d = (double)n;
#pragma unroll
            for (int p = 0; p < j; ++p) d -= M[j][p] * L[j][p];
            singular |= !(d > 1e-9 * (double)n);
            inv[j] = 1.0 / d;
#pragma unroll
            for (int i = j + 1; i < Q; ++i) {
                double s = gram[i * (i - 1) / 2 + j];
#pragma unroll
                for (int p = 0; p < j; ++p) s -= M[i][p] * L[j][p];
                M[i][j] = s;
                L[i][j] = s * inv[j];
            }
        }
        if (__builtin_expect(singular, 0)) break;
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            z[i] = rhs[i];
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
        // ---- the positive half of the levels: lane c < HALF holds pattern c (last plane +1) or its mirror, whichever is positive
        double size = 0.0;
#pragma unroll
        for (int i = 0; i < Q; ++i) size += fabs(a[i]);
        bool clear = (size < 1e30) & (size > 1e-25) & ((double)largest <= 1048576.0 * size) & ((double)smallest >= 9.3e-10 * size);
        double up = 0.0, down = 0.0;  // of lane k: level k and level k + 1, the one below the last being its mirror
        float mine = 0.f;             // lane k < HALF - 1: the first float that is nearer to level k than to level k + 1
        uint64_t patterns = lut;      // of the positive levels, outermost first
        // As long as the last round's order still is one, nothing has to be sorted; and where no float lies as close to the middle of two
        // levels as the rounding of the distances (2^-52 of them), the next one above it is the threshold.
        bool ordered = false;
        if (RANKED && known) {
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                up += flipped(a[i], flip_up[i]);
                down += flipped(a[i], flip_down[i]);
            }
            const double mid = 0.5 * (up + down);
            const float f = (float)mid;
            const double past = (double)f - mid;
            mine = past > 0.0 ? f : __uint_as_float(__float_as_uint(f) + 1u);
            const bool sure = (lane + 1 >= HALF) | ((mid >= 9.6e-7 * size) & (fabs(past) > 1e-14 * size));
            ordered = __all(clear & (up - down >= 1e-9 * size) & sure);
        }
        if (__builtin_expect(!ordered, 0)) {
            double own = 0.0;
#pragma unroll
            for (int i = 0; i < Q; ++i) own += (i == Q - 1 || ((lane >> i) & 1)) ? a[i] : -a[i];
            const uint32_t own_pattern = ((uint32_t)(lane & (HALF - 1)) | (uint32_t)HALF) ^ (own < 0.0 ? (uint32_t)(LEVELS - 1) : 0u);
            own = fabs(own);
            int rank = 0;
            double lv[HALF];
#pragma unroll
            for (int c = 0; c < HALF; ++c) {
                lv[c] = of_lane(own, c);
                rank += lv[c] > own ? 1 : 0;
            }
            // sorted downwards: level k is the one of rank k (all different, or `clear` fails below)
            up = down = 0.0;
            patterns = 0u;
            uint32_t found = 0u;
#pragma unroll
            for (int c = 0; c < HALF; ++c) {
                const int r = __builtin_amdgcn_readlane(rank, c);
                const uint32_t pat = (uint32_t)__builtin_amdgcn_readlane((int)own_pattern, c);
                patterns |= (uint64_t)pat << (8 * r);
                found |= 1u << r;
                up = lane == r ? lv[c] : up;
                down = lane + 1 == r ? lv[c] : down;
            }
            clear = clear && found == (1u << HALF) - 1u;
            if (lane == HALF - 1) down = -up;
            if (lane < HALF) clear = clear && up - down >= 1e-9 * size;
            if (HALF > 1) {
                const double mid = 0.5 * (up + down);
                const float f = (float)mid;
                const float t[3] = {__uint_as_float(__float_as_uint(f) - 1u), f, __uint_as_float(__float_as_uint(f) + 1u)};
                bool outer[3], tie = false;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const double du = fabs((double)t[c] - up), dd = fabs((double)t[c] - down);
                    outer[c] = du < dd;
                    tie = tie || du == dd;  // there the two signs of w part
                }
                if (lane + 1 < HALF) clear = clear && mid >= 9.6e-7 * size && !tie && !outer[0] && outer[2];
                mine = outer[1] ? t[1] : t[2];
            }
            clear = __all(clear);
        }
        // ---- (2) the nearest level for every element
        uint32_t diff = 0u;
        if (__builtin_expect(ordered || clear, 1)) {
            // While the patterns stay in their order an element changes where a count does; its pattern can wait until the end or
            // until a round that needs it.
            const bool same = ordered || (RANKED && known && patterns == lut);
            if (RANKED && __builtin_expect(!same && owed, 0)) assign(thr, lut);
#pragma unroll
            for (int k = 0; k + 1 < HALF; ++k) thr[k] = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(mine), k));
            if (__builtin_expect(!same, 0)) {
                diff = assign(thr, patterns);
                lut = patterns;
                if (ranked) describe();
            }
            if (ranked) {
#pragma unroll
                for (int k = 0; k < TH; ++k) look(k);
#pragma unroll
                for (int k = 0; k < TH; ++k) {
                    const int elements = count(k);
                    if (same) diff |= (uint32_t)(elements ^ under[k]);
                    under[k] = elements;
                }
            }
            owed = same;
            known = ranked;
        } else {
            if (RANKED && owed) assign(thr, lut);
            known = owed = false;
            // distances to all levels, sorted by (level, pattern) downwards: the first of the smallest ones is the one the tie
            // rules ask for.  The slots are filled in pattern order first: with non-finite levels the ranks need not be a
            // permutation.  (One wave's LDS instructions execute in order.)
            double* level = sh.level[wave];
            double* raw = sh.raw[wave];
            uint8_t* pattern = sh.pattern[wave];
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            if (lane < LEVELS) {
                double s = 0.0;
#pragma unroll
                for (int i = 0; i < Q; ++i) s += ((lane >> i) & 1) ? a[i] : -a[i];
                raw[lane] = s;
                level[LEVELS - 1 - lane] = s;
                pattern[LEVELS - 1 - lane] = (uint8_t)lane;
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            if (lane < LEVELS) {
                const double mine_l = raw[lane];
                int place = 0;
                for (int o = 0; o < LEVELS; ++o) {
                    const double l = raw[o];
                    place += (l > mine_l || (!(l < mine_l) && o > lane)) ? 1 : 0;
                }
                level[place] = mine_l;
                pattern[place] = (uint8_t)lane;
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
#pragma unroll
            for (int u = 0; u < QL; ++u) {
                double bd[4];
                int best[4];
                const double l0 = level[0];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    bd[e] = fabs((double)x[u][e] - l0);
                    best[e] = 0;
                }
#pragma unroll 1
                for (int c = 1; c < LEVELS; ++c) {
                    const double l = level[c];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const double d = fabs((double)x[u][e] - l);
                        const bool nearer = d < bd[e];
                        bd[e] = nearer ? d : bd[e];
                        best[e] = nearer ? c : best[e];
                    }
                }
                uint32_t c4 = 0u;
#pragma unroll
                for (int e = 0; e < 4; ++e) c4 |= (uint32_t)pattern[best[e]] << (8 * e);
                c4 &= mask[u];
                diff |= c4 ^ code[u];
                code[u] = c4;
            }
        }
        const bool changed = __any(diff != 0u);
        if (MW == 1 && !changed) break;
        if (MW > 1 && lane == 0) sh.changed[turn][wave] = changed ? 1u : 0u;
        from_below = known;
        if (!from_below) form_sums();
    }
    if (RANKED && owed) assign(thr, lut);
#pragma unroll
    for (int u = 0; u < QL; ++u)
        if (mask[u]) code4[tid + u * 64 * waves] = code[u];
    __syncthreads();

    // ---- outputs: alpha[i][v], packed[i][v][n / 32], planes[i][v][n]
    const int nw = n / 32;
    if (tid == 0) {
#pragma unroll
        for (int i = 0; i < Q; ++i) alpha[(int64_t)i * V + v] = (float)a[i];
    }
    for (int idx = tid; idx < Q * nw; idx += 64 * waves) {
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
            for (int k = tid; k < quads; k += 64 * waves)  // a byte per element: 1 -> 0x01, 0 -> 0xFF
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
    // four elements per lane and pass (8 vectors of 256, q = 8, 15 rounds: one wave 519 us, four 565)
    const int waves = n <= 256 ? 1 : n <= 512 ? 2 : ALT_MAX_WAVES;
    BCQ_LAUNCH((alternating_kernel<Q>), dim3((unsigned)V), dim3(64 * waves), lds, st, W, V, n, iters, alpha, packed,
                       planes, status_word);
    return hipGetLastError();
}

template <int Q, int QL, int MW, bool RANKED>
static hipError_t launch_reg_form(const float* W, int64_t V, int n, int iters, float* alpha, uint32_t* packed, int8_t* planes,
                                  int* status_word, hipStream_t st) {
    const int waves = (n / 4 + 64 * QL - 1) / (64 * QL);
    const size_t sorted = RANKED ? (size_t)waves * (65 * 4 * QL * 8 + 64 * (4 * QL + 1) * 4) : 0;
    const size_t lds = (sizeof(AltRegShared<Q, MW>) + 15) / 16 * 16 + (size_t)(n + 15) / 16 * 16 + sorted;
    static LdsLimit limit;
    hipError_t e = limit.ensure((const void*)alternating_reg_kernel<Q, QL, MW, RANKED>, lds);
    if (e != hipSuccess) return e;
    BCQ_LAUNCH((alternating_reg_kernel<Q, QL, MW, RANKED>), dim3((unsigned)V), dim3(64 * waves), lds, st, W, V, n, iters, alpha, packed,
                       planes, status_word);
    return hipGetLastError();
}

// From how many allowed rounds on the elements are sorted.  What counts are the rounds that vectors take before their fixed point: of normal
// weights and 32, 64, 128, 256 elements 2, 3, 4, 6 with two planes, 4, 6, 10, 12 with three, 6, 9, 12, 14 with four, so that short vectors with
// two planes never repay their sorting, and with four planes, whose round needs seven searches, only where they may take more than 8 rounds.
// 15 rounds, us, element by element / sorted: q = 2, 32768 vectors of 32 49.6 / 52.2, 16384 of 64 35.4 / 32.4, q = 3 104 / 94 and 84 / 68,
// q = 4 195 / 205 and 156 / 140, 8 rounds 122 / 119, 1024 of 256 15.6 / 16.2.  Four waves: 12 rounds of 640 vectors of 4096 are equal or,
// with heavy tails, slower by up to 1.12, 15 rounds 0.82 to 0.98 of the time with normal weights (worst, 512 vectors of 3328 with heavy tails, 1.06).
static int sort_rounds(int q, int n) {
    constexpr int never = 1 << 30;
    if (n > 1024) return n > 3072 ? 15 : 12;
    if (q != 3 && n < 64) return never;
    return q == 4 && n <= 256 ? 12 : 8;
}

template <int Q, int QL, int MW>
static hipError_t launch_reg(const float* W, int64_t V, int n, int iters, float* alpha, uint32_t* packed, int8_t* planes,
                             int* status_word, hipStream_t st) {
    if constexpr ((Q > 1 && MW == 1) || (Q == 3 && QL == 4)) {
        if (iters >= sort_rounds(Q, n)) return launch_reg_form<Q, QL, MW, true>(W, V, n, iters, alpha, packed, planes, status_word, st);
    }
    return launch_reg_form<Q, QL, MW, false>(W, V, n, iters, alpha, packed, planes, status_word, st);
}

// As many elements per lane as one wave's registers hold, then more waves.  q = 3, 15 rounds, us, one wave against one to four
// with 4 / 8 / 16 elements per lane: 1024 vectors of 1024 27 against 52 / 38 / 31, 256 of them 26 against 27 / 28 / 30, 1024 of
// 512 22 against 33 / 26 / 31, 4096 of 256 41 (with 8 and 16: 51, 73); 1024 of 2560 73 with 16 (112 through LDS).
// Above 4096 elements 32 per lane and up to 8 waves: every wave solves and sorts for itself, so that 16 waves of 16 elements,
// whose registers spill besides, were slower than LDS where vectors are many (918 of 4480, q = 2, 3, 4: through LDS 87, 166,
// 302 us, with 16 waves 103, 235, 556, with 8 75, 126, 213; 500 of 16384, q = 4: 765, 692, 242).  With one plane there is
// next to nothing to solve, and the registers only keep waves away: 918 of 4480 8 us through LDS, 14 to 16 from registers,
// 3000 of 1120 9.4 and 10.9.
template <int Q>
static hipError_t launch_reg_q(const float* W, int64_t V, int n, int iters, float* alpha, uint32_t* packed, int8_t* planes,
                               int* status_word, hipStream_t st) {
    if (n <= 256) return launch_reg<Q, 1, 1>(W, V, n, iters, alpha, packed, planes, status_word, st);
    if (n <= 512) return launch_reg<Q, 2, 1>(W, V, n, iters, alpha, packed, planes, status_word, st);
    if (n <= 1024) return launch_reg<Q, 4, 1>(W, V, n, iters, alpha, packed, planes, status_word, st);
    if constexpr (Q == 1) {
        return launch_q<1>(W, V, n, iters, alpha, packed, planes, status_word, st);
    } else {
        if (n <= 4096) return launch_reg<Q, 4, 4>(W, V, n, iters, alpha, packed, planes, status_word, st);
        return launch_reg<Q, 8, 8>(W, V, n, iters, alpha, packed, planes, status_word, st);
    }
}

hipError_t launch_quantize_alternating(const float* W, int64_t V, int64_t n, int q, int iters, float* alpha,
                                       uint32_t* packed, int8_t* planes, int* status_word, hipStream_t st) {
    if (status_word) {
        BCQ_LAUNCH(alt_zero_word_kernel, dim3(1), dim3(1), 0, st, status_word);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    switch (q) {
        case 1: return launch_reg_q<1>(W, V, (int)n, iters, alpha, packed, planes, status_word, st);
        case 2: return launch_reg_q<2>(W, V, (int)n, iters, alpha, packed, planes, status_word, st);
        case 3: return launch_reg_q<3>(W, V, (int)n, iters, alpha, packed, planes, status_word, st);
        case 4: return launch_reg_q<4>(W, V, (int)n, iters, alpha, packed, planes, status_word, st);
        case 5: return launch_q<5>(W, V, (int)n, iters, alpha, packed, planes, status_word, st);
        case 6: return launch_q<6>(W, V, (int)n, iters, alpha, packed, planes, status_word, st);
        case 7: return launch_q<7>(W, V, (int)n, iters, alpha, packed, planes, status_word, st);
        default: return launch_q<8>(W, V, (int)n, iters, alpha, packed, planes, status_word, st);
    }
}

}  // namespace bcq

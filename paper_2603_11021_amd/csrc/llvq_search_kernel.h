// Nearest point of the ball cut Lambda_24(m_max) for a real vector of 24 coordinates (paper Sec. 3, Sec. 3.1):
// the search over leaders (classes) and Golay words, scored by cosine (angular, for shape-gain) or by Euclidean
// distance (spherical shaping).  Included by llvq_kernels.hip.
//
// Given a class and a Golay word the best arrangement follows from sorting (rearrangement inequality):
//   odd class : x_i = 1 + 2 c_i (mod 4) fixes every sign, so <w, x> = sum coef_k * y_(k) with y_i = +-w_i by c_i
//               sorted descending and coef = +a (a = 1 mod 4) / -a (a = 3 mod 4) sorted descending;
//   even class: the 2-mod-4 values on supp(c), the 0-mod-4 values outside, each list descending onto the positions
//               by descending |w_i|, signs those of w_i; if the number of negative signs on supp(c) has the wrong
//               parity for condition (iii) of Sec. 2.3, the position of supp(c) with the smallest |w_i| (it holds
//               the smallest value) changes sign, which costs 2 * a_min * |w|_min.
//
// A wave handles one input vector w at a time, in two stages.
//
// Which (parity, Golay word) pairs can hold the winner.  A point x of shell m (norm r = sqrt(16 m)) that belongs to the
// residues of a pair (x_i = 0, 2 mod 4 by the word's bit, or 1, 3 mod 4) satisfies, for any scale t > 0,
//     <w, x> = (t^2 |w|^2 + r^2 - |t w - x|^2) / (2 t),     |t w - x|^2 >= D(word) = sum_i dist^2(t w_i, residues of bit i),
// so D bounds the score of every class of the shell on this word at once.  With t = r cos0 / |w| (cos0 near the cosine that the
// best point reaches) the bound on <w, x> / (|w| r) is k - D / (2 r^2 cos0), k = (1 + cos0^2) / (2 cos0): tight enough
// that 2.6 of the 8192 pairs (at most 11 in thousands of Gaussian vectors) reach the best score.  D of all words is a
// matrix product: with s_i = +-1 for the word's bit, D = const + sum_i delta_i s_i, and a word is the sum of two of 64 words
// (six message bits each), s_i = h_i l_i: [64 x 24 words h, signs applied to delta] x [24 x 64 words l], four 32 x 32
// tiles of two MFMAs (K = 24 in 32, one of the spare k carries the constant) for a shell and a parity, one operand constant, the other
// the same registers under a sign mask.  The smallest bound over the shells is kept per word, two parities packed in fp16
// (rounded down; the rounding of delta to fp16 is allowed for).
//
// The exact score of the pairs whose bound is within reach, 32 at a time, one per lane: the word's inputs are sorted, and the
// scores of all classes against the sorted inputs are a dense contraction scores[class][pair] = sum_k C[class][k] Z[k][pair]
// on the matrix cores.  The class values are small integers, exact in bf16; the inputs are split exactly into three bf16
// terms (8 + 8 + 8 mantissa bits), so three bf16 MFMA passes accumulate in fp32 what an fp32 product would.  Pairs are
// taken while their bound reaches the best score so far; none is left out, so the result is that of scoring every class on
// every word.  The class inside the winning tile is found by scoring that tile for the winning pair in fp32 on the vector
// ALUs, which also yields the reported score.
//
// Scoring every class on every word (the sorts and 21 MFMAs per word) took 13.7 ms for 65,536 blocks; see search_kernel.
#pragma once

namespace {

// Batcher's merge-exchange network for any n, largest element first; all indices are compile-time constants
template <int N, typename T, typename CE>
__device__ __forceinline__ void sort_network(T (&v)[N], CE ce) {
#pragma unroll
    for (int p = 1; p < N; p <<= 1) {
#pragma unroll
        for (int k = p; k >= 1; k >>= 1) {
#pragma unroll
            for (int j = k % p; j + k < N; j += 2 * k) {
#pragma unroll
                for (int i = 0; i < k; i++) {
                    if (i + j + k < N && (i + j) / (2 * p) == (i + j + k) / (2 * p)) ce(v[i + j], v[i + j + k]);
                }
            }
        }
    }
}

constexpr int kSearchWaves = 4;                 // waves per workgroup of search_kernel
constexpr float kSearchCos0 = 0.967f;           // cosine of the best point of Lambda_24(13) for Gaussian vectors: 0.962 .. 0.972
constexpr float kSearchScale = 64.0f;           // bounds are kept as 64 D / r^2: delta stays clear of the fp16 subnormals
// Slack of the first round of exact scores, in these units: on Gaussian vectors 11 pairs lie within it and nineteen times
// in twenty it holds the pair whose score ends the search.
constexpr float kSearchSlack = 1.1f;
// Both only set how much is scored exactly; the result does not depend on them.  Other inputs and unions, 65,536 blocks with their
// indices, against scoring everything (ms): angular, m_max = 13: Gaussian 0.82, Laplace 0.81, Cauchy 0.85, four nonzeros 0.90,
// one large coordinate 0.76 (13.9); Gaussian at m_max = 8, 5, 2: 0.67, 0.66, 0.74 (10.1, 9.4, 8.8); four nonzeros at m_max = 3: 5.5 (9.1).
// Euclidean, m_max = 13: Gaussian 0.84, Cauchy 8.5 (13.2): far outside the ball many points are nearly equally far.  Slower than
// scoring everything only where most words tie: all coordinates equal at m_max = 5, 23.8 (9.4).
constexpr uint32_t kSearchScratch = 512;        // dwords of LDS per wave: see SearchScratch

// LDS of a wave.  delta: [shell - 2][parity][32 k] fp16, k = 0..23 delta, k = 24, 25 the constant in two terms, the rest zero
struct SearchScratch {
    uint32_t* delta;      // 24 x 16 dwords
    float* w;             // 24
    uint32_t* list;       // 32 pairs: word h | word l << 6 | parity << 12
    float* z;             // 24 sorted inputs and two repair costs of the best pair so far
};
__device__ __forceinline__ SearchScratch search_scratch(uint32_t* base) {
    return SearchScratch{base, reinterpret_cast<float*>(base + 384), base + 408, reinterpret_cast<float*>(base + 440)};
}

// tables of the search in LDS, shared by the waves of a workgroup
struct SearchTabs {
    const uint4* a;           // class tiles as A operands, [tile][2][64]
    const float* scale;       // [tile][half][16]: factor (angular) or offset (Euclidean) of the class
    const uint32_t* gol;      // the 64 words of message bits 6..11, then the 64 of message bits 0..5
};
constexpr uint32_t kSearchTabDwords = llvq::kMaxSearchTiles * (2 * 64 * 4 + 32) + 128;

// word of the cyclic code of generator 0xC75 (paper Sec. 2.3), overall parity in bit 23
__device__ __forceinline__ uint32_t golay_word(uint32_t msg) {
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < 12; k++) c ^= ((msg >> k) & 1u) ? 0xC75u << k : 0u;
    return c | ((uint32_t)__popc(c) & 1u) << 23;
}

template <int METRIC>
__device__ __forceinline__ SearchTabs load_search_tabs(uint32_t* lds, const llvq::SearchLayout& lay, const uint4* __restrict__ tile_a,
                                                       const float* __restrict__ tile_scale) {
    uint4* a = reinterpret_cast<uint4*>(lds);
    float* scale = reinterpret_cast<float*>(lds + llvq::kMaxSearchTiles * 512);
    uint32_t* gol = lds + llvq::kMaxSearchTiles * (512 + 32);
    for (uint32_t i = threadIdx.x; i < lay.n_tiles * 128u; i += blockDim.x) a[i] = tile_a[i];
    for (uint32_t i = threadIdx.x; i < lay.n_tiles * 32u; i += blockDim.x)
        scale[i] = tile_scale[(i >> 5) * llvq::kSearchTileScaleFloats + METRIC * 32 + (i & 31u)];
    for (uint32_t i = threadIdx.x; i < 128u; i += blockDim.x) gol[i] = golay_word(i < 64u ? i << 6 : i - 64u);
    return SearchTabs{a, scale, gol};
}

// the constant operands of the bounds: sign masks of the words h (A rows) and +-1 of the words l (B columns)
struct SearchSigns {
    u32x4 h[2][2], l[2][2];                      // [32-word tile][k block]
};
__device__ __forceinline__ SearchSigns search_signs() {
    const uint32_t lane = threadIdx.x & 63u, half = lane >> 5;
    SearchSigns s;
#pragma unroll
    for (uint32_t t = 0; t < 2; t++) {
        const uint32_t u = 32u * t + (lane & 31u), ch = golay_word(u << 6), cl = golay_word(u);
#pragma unroll
        for (uint32_t kb = 0; kb < 2; kb++) {
#pragma unroll
            for (uint32_t j = 0; j < 4; j++) {
                const uint32_t k = 16u * kb + 8u * half + 2u * j;               // k >= 24: bits 24.. of the words are zero
                s.h[t][kb][j] = ((ch >> k) & 1u) << 15 | ((ch >> (k + 1u)) & 1u) << 31;
                s.l[t][kb][j] = 0x3C003C00u | ((cl >> k) & 1u) << 15 | ((cl >> (k + 1u)) & 1u) << 31;
            }
        }
    }
    return s;
}

// v over the 64 lanes, the same value in every lane
__device__ __forceinline__ float wave_max(float v) {
#define LLVQ_DPP_MAX(CTRL, ROWS) v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, v), __builtin_bit_cast(int, v), CTRL, ROWS, 0xF, false)))
    LLVQ_DPP_MAX(0xB1, 0xF); LLVQ_DPP_MAX(0x4E, 0xF); LLVQ_DPP_MAX(0x141, 0xF); LLVQ_DPP_MAX(0x140, 0xF); LLVQ_DPP_MAX(0x142, 0xA); LLVQ_DPP_MAX(0x143, 0xC);
#undef LLVQ_DPP_MAX
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
__device__ __forceinline__ float wave_sum_all(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wave_sum_to_last(v)), 63));
}
__device__ __forceinline__ float lane_value(float v, uint32_t lane) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), (int)lane));
}

// exact three-way split of eight fp32 values into bf16 terms, two per dword
__device__ __forceinline__ void split_bf16(const float (&v)[8], u32x4 (&out)[3]) {
#pragma unroll
    for (int d = 0; d < 4; d++) {
        float a = v[2 * d], b = v[2 * d + 1];
#pragma unroll
        for (int t = 0; t < 3; t++) {
            // the upper halves of a and b side by side (a in the low half): one byte permute, which also truncates
            out[t][d] = __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
            if (t < 2) {
                a -= __uint_as_float(__float_as_uint(a) & 0xFFFF0000u);
                b -= __uint_as_float(__float_as_uint(b) & 0xFFFF0000u);
            }
        }
    }
}

// best score of one class tile over the lane's 16 accumulator rows.  Angular metric: score = product x factor of the class.
// Euclidean metric: score = product + offset of the class, and the offsets are what the accumulators start from.
template <int METRIC>
__device__ __forceinline__ float tile_best(const u32x4 (&A)[2], const u32x4 (&B)[2][3], const float (&scale)[16]) {
    float16_t acc;
#pragma unroll
    for (int r = 0; r < 16; r++) acc[r] = METRIC == 0 ? 0.0f : scale[r];
#pragma unroll
    for (int t = 0; t < 3; t++) {
#pragma unroll
        for (int kb = 0; kb < 2; kb++) acc = Mma<bf16x2_t>::mma(A[kb], B[kb][t], acc);
    }
    float x[16];
#pragma unroll
    for (int r = 0; r < 16; r++) x[r] = METRIC == 0 ? acc[r] * scale[r] : acc[r];
    float best = fmaxf(x[0], x[1]);
#pragma unroll
    for (int r = 2; r < 16; r += 2) best = fmaxf(fmaxf(x[r], x[r + 1]), best);       // compiles to v_max3_f32
    return best;
}

// The nearest point for the vector whose coordinate i lane i < 24 holds in `wi` (the other lanes: 0).  Every lane returns its
// coordinate (lanes >= 24: 0); score is <w, x> / ||x|| or <w, x> - ||x||^2 / 2, the same in all lanes; rec the class's record.
template <int METRIC>
__device__ __forceinline__ int search_block(const llvq::SearchRec* __restrict__ recs, const llvq::SearchLayout& lay, uint32_t m_max, const SearchTabs& T,
                                            const SearchSigns& S, const SearchScratch& scr, float wi, float& score, uint32_t& rec) {
    const uint32_t lane = threadIdx.x & 63u, half = lane >> 5;
    const float kappa = (1.0f + kSearchCos0 * kSearchCos0) / (2.0f * kSearchCos0);
    // a power of two that brings the largest coordinate to [1, 2): the norm is then formed without overflow
    const float wmax = wave_max(fabsf(wi));
    const float up = wmax > 0.0f ? ldexpf(1.0f, max(-126, min(126, -ilogbf(wmax)))) : 1.0f;
    const float ws = wi * up;
    const float norm_s = sqrtf(wave_sum_all(ws * ws)), inv_norm = norm_s > 0.0f ? 1.0f / norm_s : 0.0f;
    // the vector that is scored: any multiple of w for the angular metric, w itself for the Euclidean one
    const float wv = METRIC == 0 ? ws : wi;
    const float norm = METRIC == 0 ? norm_s : norm_s / up;
    if (lane < 24u) scr.w[lane] = ws * inv_norm;

    // ---- delta and constants of all shells: lane = (shell, parity) of the low five bits, coordinates 12 half .. + 11 ----
    // A bound is alpha + beta D: angular 64 D / r^2; Euclidean 64 gamma (C0 - upper bound of the score), gamma = 1 / max(|w|, 1)
    const uint32_t f = lane & 31u, par = f & 1u, m = 2u + (f >> 1);
    const bool shell_ok = f < 24u && m <= m_max;
    const float r2 = 16.0f * (float)m, r = sqrtf(r2);
    float alpha = 0.0f, beta = kSearchScale / r2, c0 = 0.0f;
    const float gamma = 1.0f / fmaxf(norm, 1.0f), wg = norm * gamma;
    if constexpr (METRIC != 0) {
        const float reach = wg * r * kappa - gamma * 0.5f * r2;       // gamma x score of a point of the shell with D = 0
        c0 = wave_max(shell_ok ? reach : -INFINITY);
        alpha = kSearchScale * (c0 - reach);
        beta = kSearchScale * wg / (2.0f * kSearchCos0 * r);
    }
    float floor_f;                                                    // no word's bound is below this
    {
        const float ts = r * kSearchCos0 * 0.25f, p4 = 0.25f * (float)par;
        float sum = 0.0f, lowest = 0.0f, spread = 0.0f;
        uint32_t packed[6];
#pragma unroll
        for (int j = 0; j < 6; j++) {
            half2_t d;
#pragma unroll
            for (int e = 0; e < 2; e++) {
                const float u0 = fmaf(scr.w[12u * half + (uint32_t)(2 * j + e)], ts, -p4), u1 = u0 - 0.5f;
                const float a = u0 - rintf(u0), b = u1 - rintf(u1);   // quarter distances to the residues of bit 0 and bit 1
                const float a2 = a * a, b2 = b * b, del = (a2 - b2) * (8.0f * beta);
                sum += a2 + b2;
                lowest += fminf(a2, b2);
                spread += fabsf(del);
                d[e] = (_Float16)del;
            }
            packed[j] = __builtin_bit_cast(uint32_t, d);
        }
        sum += __shfl_xor(sum, 32);
        lowest += __shfl_xor(lowest, 32);
        spread += __shfl_xor(spread, 32);
        const float margin = spread * 0x1p-11f + 2e-3f;               // rounding of delta, of the constant and of t w
        const float base = fmaf(8.0f * beta, sum, alpha) - margin;
        floor_f = shell_ok ? fmaf(16.0f * beta, lowest, alpha) - margin : INFINITY;
        if (f < 24u) {
#pragma unroll
            for (int j = 0; j < 6; j++) scr.delta[f * 16u + 6u * half + (uint32_t)j] = packed[j];
            if (half == 0) {
                const _Float16 hi = (_Float16)base, lo = (_Float16)(base - (float)hi);
                scr.delta[f * 16u + 12u] = __builtin_bit_cast(uint32_t, half2_t{hi, lo});
            }
        }
    }
    // Shells by the smallest value their bounds can take; the first pass takes those that can matter for a vector as hard
    // as a Gaussian one, what the best score does not rule out afterwards is looked at in a second pass.
    const float floor_min = -wave_max(-floor_f);
    uint64_t waiting = __builtin_amdgcn_ballot_w64(shell_ok && half == 0), todo;        // bit 2 (m - 2) + parity
    todo = __builtin_amdgcn_ballot_w64(half == 0 && floor_f <= fmaf(0.75f, fabsf(floor_min), floor_min) + 0.25f);

    float best = -INFINITY, reach = -INFINITY;     // best score so far; bounds up to `reach` can still hold a better one
    uint32_t best_tile = 0, best_c = 0;
    bool first = true;
    if (lane < 26u) scr.z[lane] = 0.0f;
    while (todo) {
        half2_t run[4][16];                        // [32 x 32 tile][register]: smallest bound of the even pair, of the odd pair
#pragma unroll
        for (int t = 0; t < 4; t++) {
#pragma unroll
            for (int v = 0; v < 16; v++) run[t][v] = __builtin_bit_cast(half2_t, 0x7C007C00u);
        }
        waiting &= ~todo;
        for (uint32_t sh = 0; sh < 12u; sh++) {
            const uint32_t pair = (uint32_t)(todo >> (2u * sh)) & 3u;
            if (!pair) continue;
            waiting &= ~((uint64_t)3u << (2u * sh));                  // both parities of the shell are looked at together
            u32x4 raw[2][2];
#pragma unroll
            for (int p = 0; p < 2; p++) {
#pragma unroll
                for (int kb = 0; kb < 2; kb++) raw[p][kb] = *reinterpret_cast<const u32x4*>(scr.delta + (2u * sh + (uint32_t)p) * 16u + 8u * (uint32_t)kb + 4u * half);
            }
#pragma unroll
            for (int R = 0; R < 2; R++) {
#pragma unroll
                for (int C = 0; C < 2; C++) {
                    float16_t t[2];
#pragma unroll
                    for (int p = 0; p < 2; p++) {
                        float16_t zero;
#pragma unroll
                        for (int v = 0; v < 16; v++) zero[v] = 0.0f;
                        t[p] = Mma<half2_t>::mma(raw[p][1] ^ S.h[R][1], S.l[C][1], Mma<half2_t>::mma(raw[p][0] ^ S.h[R][0], S.l[C][0], zero));
                    }
#pragma unroll
                    for (int v = 0; v < 16; v++)
                        run[2 * R + C][v] = __builtin_elementwise_min(run[2 * R + C][v], __builtin_bit_cast(half2_t, __builtin_amdgcn_cvt_pkrtz(t[0][v], t[1][v])));
                }
            }
        }
        if (first) {
            half2_t lo = run[0][0];
#pragma unroll
            for (int t = 0; t < 4; t++) {
#pragma unroll
                for (int v = 0; v < 16; v++) lo = __builtin_elementwise_min(lo, run[t][v]);
            }
            reach = -wave_max(-fminf((float)lo[0], (float)lo[1])) + kSearchSlack;
        }
        for (;;) {
            // ---- pairs within reach, up to 32; taken pairs are struck out ----
            const _Float16 lim = (_Float16)(reach + fabsf(reach) * 0x1p-10f + 1e-3f);
            uint32_t n = 0;
#pragma unroll
            for (int t = 0; t < 4; t++) {
#pragma unroll
                for (int v8 = 0; v8 < 2; v8++) {
                    half2_t lo = run[t][8 * v8];
#pragma unroll
                    for (int v = 1; v < 8; v++) lo = __builtin_elementwise_min(lo, run[t][8 * v8 + v]);
                    if (n >= 32u || !__builtin_amdgcn_ballot_w64(lo[0] <= lim || lo[1] <= lim)) continue;
#pragma unroll
                    for (int v = 8 * v8; v < 8 * v8 + 8; v++) {
#pragma unroll
                        for (int p = 0; p < 2; p++) {
                            const bool hit = run[t][v][p] <= lim;
                            const uint64_t hits = __builtin_amdgcn_ballot_w64(hit);
                            if (hits) {
                                const uint32_t pos = n + __builtin_amdgcn_mbcnt_hi((uint32_t)(hits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hits, 0u));
                                if (hit && pos < 32u) {
                                    const uint32_t h = 32u * (uint32_t)(t >> 1) + 8u * (uint32_t)(v >> 2) + 4u * half + (uint32_t)(v & 3), l = 32u * (uint32_t)(t & 1) + (lane & 31u);
                                    scr.list[pos] = h | l << 6 | (uint32_t)p << 12;
                                    run[t][v][p] = __builtin_bit_cast(_Float16, (uint16_t)0x7C00u);
                                }
                                n += (uint32_t)__popcll(hits);
                            }
                        }
                    }
                }
            }
            if (norm_s == 0.0f) {                  // w = 0: every point of a shell scores the same, and word 0 has odd classes on all
                if (!first) break;
                scr.list[0] = 1u << 12;
                n = 1;
            }
            first = false;
            if (n == 0) break;
            n = min(n, 32u);
            // ---- exact scores: lanes l and l + 32 share pair l ----
            const uint32_t entry = scr.list[min(lane & 31u, n - 1u)], odd = entry >> 12;
            const uint32_t c = T.gol[entry & 63u] ^ T.gol[64u + ((entry >> 6) & 63u)];
            // Sorted as unsigned keys, largest first.  Odd pair: w_i negated where the word has a 1, in an order-preserving
            // code; even pair: |w_i| with the word's bit on top (the support first).
            uint32_t key[24], neg = 0;
#pragma unroll
            for (int i = 0; i < 24; i++) {
                const uint32_t u = __float_as_uint(lane_value(wv, (uint32_t)i)), cb = (c << (31 - i)) & 0x80000000u;
                const uint32_t y = u ^ cb;
                neg ^= ((u & 0x80000000u) && (float)0.0f != __uint_as_float(u)) ? cb : 0u;
                key[i] = odd ? y ^ ((uint32_t)((int32_t)y >> 31) | 0x80000000u) : (u & 0x7FFFFFFFu) | cb;
            }
            sort_network<24>(key, [](uint32_t& a, uint32_t& b) { const uint32_t hi = max(a, b), lo = min(a, b); a = hi; b = lo; });
            float z[24];
#pragma unroll
            for (int i = 0; i < 24; i++) {
                const uint32_t k = key[i];
                z[i] = __uint_as_float(odd ? k ^ (~(uint32_t)((int32_t)k >> 31) | 0x80000000u) : k & 0x7FFFFFFFu);
            }
            // even pair: cost of negating the smallest magnitude on the support, for the parity of negative signs it has and lacks
            const uint32_t wt = (uint32_t)__popc(c);
            const float xmin = (odd || wt == 0u) ? 0.0f : (wt == 8u ? z[7] : (wt == 12u ? z[11] : (wt == 16u ? z[15] : z[23])));
            const float pen0 = neg ? xmin : 0.0f, pen1 = neg ? 0.0f : xmin;
            const uint32_t group = odd ? 0u : (wt == 0u ? 1u : (wt == 8u ? 2u : (wt == 12u ? 3u : (wt == 16u ? 4u : 5u))));
            u32x4 B[2][3];
            {
                float lo8[8], hi8[8];
#pragma unroll
                for (int i = 0; i < 8; i++) {
                    lo8[i] = half ? z[8 + i] : z[i];
                    hi8[i] = half ? (i == 0 ? pen0 : (i == 1 ? pen1 : 0.0f)) : z[16 + i];
                }
                split_bf16(lo8, B[0]);
                split_bf16(hi8, B[1]);
            }
            float mine = -INFINITY;
            uint32_t mine_tile = 0;
            for (uint32_t g = 0; g < 6u; g++) {
                if (!__builtin_amdgcn_ballot_w64(group == g)) continue;
                const uint32_t t0 = lay.grp_tile_first[g], t1 = t0 + lay.grp_tile_count[g];
                for (uint32_t ct = t0; ct < t1; ct++) {
                    const u32x4 A[2] = {__builtin_bit_cast(u32x4, T.a[(ct * 2u) * 64u + lane]), __builtin_bit_cast(u32x4, T.a[(ct * 2u + 1u) * 64u + lane])};
                    float scale[16];
#pragma unroll
                    for (int k = 0; k < 4; k++) {
                        const float4 q = *reinterpret_cast<const float4*>(T.scale + ct * 32u + half * 16u + 4u * (uint32_t)k);
                        scale[4 * k] = q.x; scale[4 * k + 1] = q.y; scale[4 * k + 2] = q.z; scale[4 * k + 3] = q.w;
                    }
                    const float b = tile_best<METRIC>(A, B, scale);
                    if (group == g && b > mine) { mine = b; mine_tile = ct; }
                }
            }
            const float top = wave_max(mine);
            if (top > best) {
                best = top;
                const uint32_t src = (uint32_t)__builtin_ctzll(__builtin_amdgcn_ballot_w64(mine == top));
                best_tile = __builtin_amdgcn_readlane(mine_tile, src);
                best_c = __builtin_amdgcn_readlane(c, src);
                if (lane == src) {
#pragma unroll
                    for (int i = 0; i < 24; i++) scr.z[i] = z[i];
                    scr.z[24] = pen0;
                    scr.z[25] = pen1;
                }
            }
            // bounds that a better score can have (scores are rounded: a little more)
            if constexpr (METRIC == 0) {
                const float lb = best * inv_norm;
                reach = kSearchScale * 2.0f * kSearchCos0 * (kappa - (lb - 4e-6f * fabsf(lb)));
            } else {
                reach = kSearchScale * (c0 - gamma * (best - 4e-6f * (fabsf(best) + 0.5f * 16.0f * (float)m_max)));
            }
        }
        todo = norm_s == 0.0f ? 0ull : __builtin_amdgcn_ballot_w64(half == 0 && floor_f <= reach) & waiting;
    }

    // ---- the class inside the winning tile: lane = row of the tile, fp32 ----
    const bool odd_tile = best_tile < lay.grp_tile_first[1];
    const uint32_t row = lane & 31u;
    const bool valid = row < lay.tile_rows[best_tile];
    const uint32_t j = lay.tile_first_rec[best_tile] + (valid ? row : 0u);
    const llvq::SearchRec& Q = recs[j];
    float acc = 0.0f;
#pragma unroll
    for (int k = 0; k < 24; k++) acc = fmaf(Q.coef[k], scr.z[k], acc);
    acc = fmaf(-Q.amin2, Q.kappa ? scr.z[25] : scr.z[24], acc);
    const float cand = valid ? fmaf(acc, Q.mul[METRIC], Q.bias[METRIC]) : -INFINITY;
    const float top = wave_max(cand);
    rec = __builtin_amdgcn_readlane(j, (uint32_t)__builtin_ctzll(__builtin_amdgcn_ballot_w64(cand == top) | (1ull << 63)));
    score = METRIC == 0 ? top / up : top;
    // ---- its coordinates: lane i = position i, placed by rank (ties by position) ----
    const llvq::SearchRec& R = recs[rec];
    const uint32_t i = min(lane, 23u), ci = (best_c >> i) & 1u, u = __float_as_uint(wv);
    const uint32_t y = u ^ (ci << 31);
    const uint32_t key = odd_tile ? y ^ ((uint32_t)((int32_t)y >> 31) | 0x80000000u) : (u & 0x7FFFFFFFu) | (ci << 31);
    uint32_t rank = 0;
#pragma unroll
    for (uint32_t k = 0; k < 24u; k++) {
        const uint32_t kk = __builtin_amdgcn_readlane(key, k);
        rank += (kk > key || (kk == key && k < lane)) ? 1u : 0u;
    }
    const int a = (int)R.coef[min(rank, 23u)];
    int x;
    if (odd_tile) {
        x = ci ? -a : a;
    } else {
        const bool minus = wv < 0.0f;
        x = minus ? -a : a;
        const uint32_t wt = (uint32_t)__popc(best_c);
        const uint32_t negpar = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(minus && ci && lane < 24u)) & 1u;
        if (wt > 0u && negpar != R.kappa && rank == wt - 1u) x = -x;
    }
    return lane < 24u ? x : 0;
}

// One step of the block-wise loop of paper App. B (Alg. 1), per row: the block v = W[row][0..23] that has been given its nearest
// direction x is replaced by g * x / ||x|| with g = ||v|| rounded to fp16 (the norm-preserving "gain reset" of paper
// Sec. 3.3), and E U_QQ^-1 for the error E = v - g x / ||x|| is kept for the propagation.
// levels != nullptr: the optional scalar gain quantiser of App. B Alg. 1 -- g is the nearest of n_levels fp16
// reconstruction levels (ascending; ties go to the lower level) instead of the rounded norm.
struct RetractStep {
    float* W;                     // the block column, rows ldw apart
    const float* U;               // its diagonal block of the factor, rows ldu apart
    size_t ldu;
    float* E;                     // [rows][24]; nullptr: the last block column, nothing to propagate to
    uint16_t* gain;               // of the block column, gain_stride apart
    size_t gain_stride;
    const uint16_t* levels;
    int n_levels;
};

// v and x: coordinate of lane i < 24 (other lanes: 0); U: the diagonal block in LDS, [24][24].  Written as part of
// search_kernel: a lane's coordinates are in registers there, and two launches of the loop (11.8 us of arithmetic and dispatch
// per block column of 4096 rows, of 95 us in all) go.
__device__ __forceinline__ void retract_row(const RetractStep& step, size_t row, size_t ldw, float v, int xi, const float* U) {
    const uint32_t lane = threadIdx.x & 63u;
    const float x = (float)xi;
    float n2 = 0.0f, x2 = 0.0f;
#pragma unroll
    for (uint32_t i = 0; i < 24u; i++) {
        const float vi = lane_value(v, i), xv = lane_value(x, i);
        n2 = fmaf(vi, vi, n2);
        x2 = fmaf(xv, xv, x2);
    }
    const float norm = sqrtf(n2);
    __half gh = __float2half_rn(norm);
    if (step.levels) {
        // the nearest level of every 64th, then the nearest of the lanes' (the lowest of equals)
        float best = INFINITY;
        uint32_t k_best = 0xFFFFFFFFu;
        for (uint32_t k = lane; k < (uint32_t)step.n_levels; k += 64u) {
            const float d = fabsf(norm - __half2float(__ushort_as_half(step.levels[k])));
            if (d < best) { best = d; k_best = k; }
        }
        const float d_min = -wave_max(-best);
        if (d_min < INFINITY) {
            uint32_t k = best == d_min ? k_best : 0xFFFFFFFFu;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) k = min(k, (uint32_t)__shfl_xor((int)k, off));
            gh = __ushort_as_half(step.levels[k]);
        }
    }
    const float q = __half2float(gh) / sqrtf(x2) * x;
    if (lane < 24u) step.W[row * ldw + lane] = q;
    if (lane == 0) step.gain[row * step.gain_stride] = __half_as_ushort(gh);
    if (!step.E) return;
    // e U_QQ = E: column i is final once the columns before it are taken out
    float e = v - q;
#pragma unroll
    for (uint32_t i = 0; i < 24u; i++) {
        const float u = U[i * 24u + min(lane, 23u)];
        const float ei = lane_value(e, i) / lane_value(u, i);
        e = lane == i ? ei : lane > i ? fmaf(-ei, u, e) : e;
    }
    if (lane < 24u) step.E[row * 24 + lane] = e;
}

// RETRACT: the vectors are the rows of step.W (w_in is not used), and every one goes through a step of the block-wise loop
template <int METRIC, bool RETRACT>
__global__ void __launch_bounds__(64 * kSearchWaves, 2) search_kernel(const llvq::SearchRec* __restrict__ recs, llvq::SearchLayout lay, uint32_t m_max,
                                                                     const uint4* __restrict__ tile_a, const float* __restrict__ tile_scale,
                                                                     const float* __restrict__ w_in, size_t ldw, size_t n, int8_t* __restrict__ pts,
                                                                     float* __restrict__ score_out, RetractStep step) {
    uint32_t* lds = reinterpret_cast<uint32_t*>(g_lds);
    const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const SearchTabs T = load_search_tabs<METRIC>(lds, lay, tile_a, tile_scale);
    const SearchScratch scr = search_scratch(lds + kSearchTabDwords + wave * kSearchScratch);
    float* U = reinterpret_cast<float*>(lds + kSearchTabDwords + kSearchWaves * kSearchScratch);
    for (uint32_t i = lane; i < 384u; i += 64u) scr.delta[i] = 0u;   // k = 26..31 stay zero
    if constexpr (RETRACT) {
        for (uint32_t i = threadIdx.x; i < 24u * 24u; i += blockDim.x) U[i] = step.U[(size_t)(i / 24u) * step.ldu + i % 24u];
    }
    __syncthreads();
    const SearchSigns S = search_signs();
    for (size_t v = (size_t)blockIdx.x * kSearchWaves + wave; v < n; v += (size_t)gridDim.x * kSearchWaves) {
        const float wi = lane < 24u ? (RETRACT ? step.W : w_in)[ldw * v + lane] : 0.0f;
        float score;
        uint32_t rec;
        const int x = search_block<METRIC>(recs, lay, m_max, T, S, scr, wi, score, rec);
        if (lane < 24u) pts[24 * v + lane] = (int8_t)x;
        if constexpr (RETRACT) retract_row(step, v, ldw, wi, x, U);
        else if (lane == 0 && score_out) score_out[v] = score;
    }
}

}  // namespace

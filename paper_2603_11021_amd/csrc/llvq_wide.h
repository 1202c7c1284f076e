// Step-by-step placement of App. A step 4 for the larger unions of shells, Lambda_24(m_max) with 14 <= m_max <= 19 (paper Table 1,
// row m = 19: 23,546,209,100,646,960 points, 55-bit indices): plain integer arithmetic, subsets unranked against a table of binomial
// coefficients.  The kernels decode these unions with the tables of llvq_decode_core.h (layout Lay19); wide_place is for what
// those tables cannot describe, the few classes with subsets of more than 16 slots or more than four minority values (3 in
// a million indices).
#pragma once
#include <cstdint>
#include <vector>

#include "llvq_tables.h"

#if defined(__HIPCC__)
#define LLVQ_WHD __host__ __device__ inline
#else
#define LLVQ_WHD inline
#endif

namespace llvq {

constexpr int kWideMaxM = 19;
constexpr int kWideMaxMinor = 5;      // distinct values of the outer domain besides the outside value
constexpr int kWideMaxDirect = 4;     // distinct 2-mod-4 values of a direct F1 word

// flags of WideRec
enum { WF_ODD = 1, WF_F1DIRECT = 2, WF_OUTER_ALL = 4, WF_FEN = 8, WF_KAPPA = 16 };

struct alignas(16) WideRec {
    uint64_t Pin;                 // arrangements of the minority values on their q slots
    uint32_t P1;                  // arrangements of the direct F1 word (1 when there is none)
    uint32_t A;                   // Golay refinements of the class: 1, 759, 2576 or 4096
    float    rnorm;               // 1 / sqrt(16 m)
    uint16_t goff;                // first Golay word of the class in the (weight, message) order
    uint8_t  B, w, m, n, q, flags;
    uint8_t  nm, nd;              // numbers of minority values / of direct F1 values
    uint8_t  mc[kWideMaxMinor];   // multiplicities of the minority values, descending value order
    uint8_t  dc[kWideMaxDirect];  // multiplicities of the direct F1 values, descending value order
    int8_t   outside;             // value on the outer domain's slots outside U (signed for odd classes, see below)
    int8_t   mv[kWideMaxMinor];   // minority values; odd classes: the value taken where the Golay word has a 0
    int8_t   dv[kWideMaxDirect];  // direct F1 values
    uint8_t  pad[13];
};
static_assert(sizeof(WideRec) == 64, "WideRec layout");

LLVQ_WHD uint32_t wide_popc(uint32_t v) { return (uint32_t)__builtin_popcount(v); }

// the k-subset of {0 .. nbits-1} with colex rank `rank` (numeric order of the masks of popcount k)
LLVQ_WHD uint32_t wide_colex_unrank(const uint32_t* binom, int nbits, int k, uint32_t rank) {
    uint32_t mask = 0;
    for (int pos = nbits - 1; pos >= 0 && k > 0; pos--) {
        const uint32_t c = binom[pos * 25 + k];            // subsets of size k among positions below pos
        if (rank >= c) { mask |= 1u << pos; rank -= c; k--; }
    }
    return mask;
}

// the low bits of src laid onto the set bits of mask, lowest first
LLVQ_WHD uint32_t wide_deposit(uint32_t src, uint32_t mask) {
    uint32_t out = 0;
    while (mask) {
        const uint32_t low = mask & (0u - mask);
        if (src & 1u) out |= low;
        src >>= 1;
        mask ^= low;
    }
    return out;
}

// Lays the values of a word (multiplicities cnt[0..nv-1], descending value order) onto the set bits of `slots`
// according to the mixed-radix rank rho: digit of the largest value least significant, each digit the colex rank of
// the subset that value takes among the slots still free; the last value takes what is left.  put(i, positions of value i).
template <class Put>
LLVQ_WHD void wide_inner_word(const uint32_t* binom, const uint8_t* cnt, int nv, uint64_t rho, uint32_t slots, Put put) {
    uint32_t freemask = slots;
    for (int i = 0; i + 1 < nv; i++) {
        const int nfree = (int)wide_popc(freemask);
        const uint32_t radix = binom[nfree * 25 + cnt[i]];
        const uint32_t digit = (uint32_t)(rho % radix);
        rho /= radix;
        const uint32_t occ = wide_deposit(wide_colex_unrank(binom, nfree, cnt[i], digit), freemask);
        put(i, occ);
        freemask &= ~occ;
    }
    put(nv - 1, freemask);
}

// App. A step 4 for a block of class R whose Golay word c and digits are known: calls emit(positions, code, value) for the
// outside value (code 0), the minority values (codes 1, 2, ..) and the direct F1 values (codes 8, 9, ..) and returns the
// positions whose sign is flipped.
template <class Emit>
LLVQ_WHD uint32_t wide_place(const uint32_t* binom, const WideRec& R, uint32_t c, uint32_t s, uint32_t d, uint64_t rin, uint32_t rho1, Emit emit) {
    const bool odd = R.flags & WF_ODD, outer_all = R.flags & WF_OUTER_ALL, f1direct = R.flags & WF_F1DIRECT;
    const uint32_t om = outer_all ? 0xFFFFFFu : (~c & 0xFFFFFFu);
    // the q-subset U of the outer domain's n slots: slots 0..11 low, the rest high; ordered by the number j of high
    // slots, then the colex rank of the high part, then that of the low part
    const int n = R.n, q = R.q, nl = n < 12 ? n : 12, nh = n - nl;
    int j = q - nl > 0 ? q - nl : 0;
    const int jmax = q < nh ? q : nh;
    uint32_t base = 0;
    for (; j < jmax; j++) {
        const uint32_t cnt = binom[nh * 25 + j] * binom[nl * 25 + (q - j)];
        if (d < base + cnt) break;
        base += cnt;
    }
    const uint32_t dl = d - base, div = binom[nl * 25 + (q - j)];
    const uint32_t U_rel = wide_colex_unrank(binom, nl, q - j, dl % div) | (wide_colex_unrank(binom, nh, j, dl / div) << 12);
    const uint32_t U = wide_deposit(U_rel, om);
    emit(om & ~U, 0, (int)R.outside);
    if (R.nm) wide_inner_word(binom, R.mc, R.nm, rin, U, [&](int i, uint32_t occ) { emit(occ, 1 + i, (int)R.mv[i]); });
    if (f1direct) wide_inner_word(binom, R.dc, R.nd, rho1, c, [&](int i, uint32_t occ) { emit(occ, 8 + i, (int)R.dv[i]); });
    // signs: even classes take w - 1 free bits on the word's support (the last slot is forced by condition (iii)),
    // then one bit per slot of U; odd classes are negated where the word has a 1
    if (odd) return c;
    const uint32_t wm1 = R.w ? R.w - 1u : 0u;
    uint32_t s1 = s & ((1u << wm1) - 1u);
    const uint32_t forced = ((R.flags & WF_FEN) ? 1u : 0u) & (((R.flags & WF_KAPPA) ? 1u : 0u) ^ wide_popc(s1)) & 1u;
    s1 |= forced << wm1;
    return wide_deposit(s1, c) | wide_deposit(s >> wm1, U);
}

// host-side tables of a wide context
struct WideTables {
    TableLayout tab;
    std::vector<unsigned char> blob;   // the tables of llvq_decode_core.h in layout Lay19, the WideRecs and the binomial coefficients
    uint64_t shell_off[24];            // index of the first point of shell m (N(m-1)); entries above m_max hold N(m_max)
};

// Builds the tables for Lambda_24(m_max), 2 <= m_max <= 19.  Returns false on an internal inconsistency.
bool build_wide_tables(int m_max, WideTables& out);

}  // namespace llvq

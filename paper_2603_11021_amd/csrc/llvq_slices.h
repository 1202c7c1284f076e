// Integer arithmetic of slice_kernel that host tests walk over whole ranges of sizes: how a product is cut into workgroups, and
// where the kernel reads its words.
#pragma once
#include "llvq_decode_core.h"

namespace llvq {

// Products whose partial sums llvq.h promises to add in the same order from call to call (M > 64): those with more strips of 256
// rows x 256 tokens (128 x 512 from M = 384 on) than half the compute units.  slice_kernel needs no atomics there.
inline bool fixed_order(int num_cu, int M, int N) {
    if (M <= 64) return false;
    const int64_t rows = M < 384 ? 256 : 128, tokens = M < 384 ? 256 : 512;
    return ((N + rows - 1) / rows) * ((M + tokens - 1) / tokens) * 2 > num_cu;
}

// 32-row tiles per workgroup and slices of K per workgroup for passes of TT token tiles
constexpr int slice_tiles(int TT) { return TT <= 2 ? 2 : 4; }

// How long a launch takes, in us: rounds of workgroups x (steps x the time of a step + tables and final sum), and, when the rows'
// block pairs are split over workgroups, 335 atomics per ns and the clearing of y.  The times are fitted to 238 products in
// slice_kernel and 212 in strip_kernel (512 .. 128256 rows, 960 .. 28680 columns, 48 .. 383 tokens): 2 to 5 % off in the mean.
struct LaunchCost {
    int num_cu;
    double step, ends;
    double us(uint64_t wgs, uint64_t ksplit, uint64_t steps, uint64_t sums) const {
        const uint64_t rounds = (wgs * ksplit + (uint64_t)num_cu - 1) / (uint64_t)num_cu;
        return (double)rounds * ((double)steps * step + ends) + (ksplit > 1 ? (double)ksplit * (double)sums / 335e3 + 3.0 : 0.0);
    }
};

struct SlicePlan {
    int token_tiles;     // tiles of 32 tokens per pass: 2, 3 or 4
    int passes;
    int strip_rows;
    int ksplit;          // workgroups that share the block pairs of a row
    double us;           // estimate
};

// n_items matrices of N[i] rows and KB blocks per row in one launch.  Passes of at most 128 tokens, as even as token tiles
// allow, and the split with the smallest estimate.  two_terms: bf16 weights, which take twice the products.
inline SlicePlan slice_plan(int num_cu, int M, int KB, bool two_terms, const int* N, int n_items) {
    SlicePlan p;
    const int tiles = (M + 31) / 32;
    p.passes = (tiles + 3) / 4;
    const int per_pass = (tiles + p.passes - 1) / p.passes;
    p.token_tiles = per_pass <= 2 ? 2 : per_pass;
    p.strip_rows = 32 * slice_tiles(p.token_tiles);
    const uint64_t slices = (uint64_t)(16 / slice_tiles(p.token_tiles)), spt = ((uint64_t)KB + 1) / 2;
    uint64_t wgs = 0, rows = 0;
    bool split = true;
    for (int i = 0; i < n_items; i++) {
        wgs += (uint64_t)((N[i] + p.strip_rows - 1) / p.strip_rows) * (uint64_t)p.passes;
        rows += (uint64_t)N[i];
        split = split && !fixed_order(num_cu, M, N[i]);
    }
    const double steps[2][3] = {{3.2, 3.2, 3.5}, {3.8, 4.0, 4.7}};
    const LaunchCost cost = {num_cu, steps[two_terms][p.token_tiles - 2], 6.0};
    for (uint64_t ks = 1; ks <= 64 && (ks == 1 || (split && ks * slices <= spt)); ks++) {
        const double t = cost.us(wgs, ks, (spt + ks * slices - 1) / (ks * slices), (uint64_t)M * rows);
        if (ks == 1 || t < p.us) { p.us = t; p.ksplit = (int)ks; }
    }
    return p;
}

// strip_kernel: strips of 256 rows x 256 tokens, the block pairs of a row over as many workgroups as the chip has compute units
// for, at least eight steps each; 65 .. 383 tokens, where fixed_order counts the same strips.
constexpr int kStripRows = 256, kStripTokens = 256, kStripMinM = 65, kStripMaxM = 383;
struct StripPlan {
    int strips, passes, ksplit;
    double us;
};
inline StripPlan strip_plan(int num_cu, int M, int KB, bool two_terms, int N) {
    StripPlan p;
    p.strips = (N + kStripRows - 1) / kStripRows;
    p.passes = (M + kStripTokens - 1) / kStripTokens;
    const int spt = (KB + 1) / 2, most = spt / 8 > 1 ? spt / 8 : 1, room = num_cu / (p.strips * p.passes);
    p.ksplit = room < 1 ? 1 : room < most ? room : most;
    p.us = LaunchCost{num_cu, two_terms ? 3.1 : 2.4, 10.0}.us((uint64_t)p.strips * (uint64_t)p.passes, (uint64_t)p.ksplit,
                                                              (uint64_t)((spt + p.ksplit - 1) / p.ksplit), (uint64_t)M * (uint64_t)N);
    return p;
}

// Whether a product takes strip_kernel: it decodes a block once per 256 tokens where slice_kernel does per 128, but two waves per
// SIMD take longer over a step, and 256 x 256 tiles fill the chip only where there are many.  Measured (us, strip against
// slice): 14336 x 14352, M = 250 fp16 236 / 262, M = 256 bf16 289 / 345; 11008 x 8208, M = 129 fp16 112 / 143; 65536 x 4104, M = 256 bf16
// 308 / 472; 65536 x 480, M = 300 bf16 90 / 112; 14336 x 4104, M = 250 fp16 104 / 84; 4096 x 4104, M = 256 bf16 64 / 45; 65536 x 4104, M = 128
// bf16 304 / 245.  On 344 such products the choice by estimate is 0.1 % slower in the mean, 4.5 % at most, than the faster of the two.
inline bool strip_faster(int num_cu, int M, int KB, bool two_terms, int N) {
    return M >= kStripMinM && M <= kStripMaxM && strip_plan(num_cu, M, KB, two_terms, N).us < slice_plan(num_cu, M, KB, two_terms, &N, 1).us;
}

// Whether matrices that share x do better one after the other, those that gain from it in strip_kernel, than in one launch of
// slice_kernel (two of 28672 x 4104 at M = 256, bf16: 371 against 449 us; 65536 and 1024 rows 330 against 563 us).
inline bool strips_apart(int num_cu, int M, int KB, bool two_terms, const int* N, int n_items) {
    double apart = 0.0;
    bool any = false;
    for (int i = 0; i < n_items; i++) {
        const bool strip = strip_faster(num_cu, M, KB, two_terms, N[i]);
        any = any || strip;
        apart += strip ? strip_plan(num_cu, M, KB, two_terms, N[i]).us : slice_plan(num_cu, M, KB, two_terms, N + i, 1).us;
    }
    return any && apart < slice_plan(num_cu, M, KB, two_terms, N, n_items).us;
}

// The words of a row tile, as 32-bit block offsets from block `first` of the matrix (wave-uniform).  Words are read in pairs, so
// where the strip holds a single block (the last row of a matrix with one block per row) `first` is the block before the
// strip: there is one, because a matrix of a single block is not given to the kernel.
struct SliceWords {
    size_t first;
    uint32_t row;        // offset of the lane's row (at most 127 rows of fewer than 2^24 blocks)
    uint32_t last;       // offset of the matrix's last block, clamped to 2^31 - 1; at least 1
};

// row0: first row of the workgroup's strip, wrow: the lane's row (a row past the matrix reads the last one); N KB >= 2.
LLVQ_HD SliceWords slice_words(int row0, int wrow, int N, int KB) {
    SliceWords s;
    const size_t left = (size_t)(N - row0) * (size_t)KB;               // blocks from the strip's first to the matrix's last
    const uint32_t back = left == 1 ? 1u : 0u;
    s.first = (size_t)row0 * (size_t)KB - back;
    s.row = (uint32_t)((wrow < N ? wrow : N - 1) - row0) * (uint32_t)KB + back;
    s.last = (uint32_t)(left < 0x80000000u ? left : (size_t)0x80000000u) - 1u + back;
    return s;
}

// Offset of the pair of neighbouring words that lane half `half` reads for the two steps `step`, `step + 1`: its block is the
// first of the pair, or the second (`late`) where it is the matrix's last.  real == false: a pair that is never used.
LLVQ_HD uint32_t slice_pair(const SliceWords& s, uint32_t step, uint32_t half, uint32_t KB, bool real, bool& late) {
    const uint32_t b = 2 * (step + half), k = s.row + (b < KB - 1 ? b : KB - 1);
    late = k >= s.last;
    return real ? late ? k - 1 : k : 0;
}

}  // namespace llvq

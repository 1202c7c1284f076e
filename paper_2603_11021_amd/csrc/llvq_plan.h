// How llvq_matmul cuts a product of 33 or more activation rows into workgroups, which kernel it takes, and where slice_kernel reads
// its words: plain arithmetic that host tests walk over whole ranges of sizes.
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
// block pairs are split over workgroups, 335 atomics per ns and the clearing of y.  The times are fitted to 574 products in
// slice_kernel, 212 in strip_kernel and 374 in panel_kernel (300 .. 128256 rows, 480 .. 28680 columns, 48 .. 1024 tokens, both
// types): 2 to 6 % off in the mean.
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

// strip_kernel: strips of 256 rows x all of 65 .. 256 tokens, the block pairs of a row over as many workgroups as the chip has
// compute units for, at least eight steps each.
constexpr int kStripRows = 256, kStripMinM = 65, kStripMaxM = 256;
struct StripPlan {
    int strips, ksplit;
    double us;
};
inline StripPlan strip_plan(int num_cu, int M, int KB, bool two_terms, int N) {
    StripPlan p;
    p.strips = (N + kStripRows - 1) / kStripRows;
    const int spt = (KB + 1) / 2, most = spt / 8 > 1 ? spt / 8 : 1, room = num_cu / p.strips;
    p.ksplit = room < 1 ? 1 : room < most ? room : most;
    p.us = LaunchCost{num_cu, two_terms ? 3.1 : 2.4, 10.0}.us((uint64_t)p.strips, (uint64_t)p.ksplit, (uint64_t)((spt + p.ksplit - 1) / p.ksplit),
                                                              (uint64_t)M * (uint64_t)N);
    return p;
}

// panel_kernel: panels of 128 rows x 512 tokens, the block pairs of a row over as many workgroups as the chip has compute units for,
// at least sixteen steps each.  From 257 tokens on (two of its eight waves' tokens in use; slice_kernel needs a third pass), where
// its 32-bit byte offsets into x reach.
constexpr int kPanelRows = 128, kPanelTokens = 512, kPanelMinM = 257;
struct PanelPlan {
    int strips, passes, ksplit;
    double us;
};
inline bool panel_reaches(int M, int KB) { return M >= kPanelMinM && (uint64_t)M * (uint64_t)KB * 48u < (1ull << 32); }
inline PanelPlan panel_plan(int num_cu, int M, int KB, bool two_terms, const int* N, int n_items) {
    PanelPlan p;
    uint64_t rows = 0;
    p.strips = 0;
    for (int i = 0; i < n_items; i++) { p.strips += (N[i] + kPanelRows - 1) / kPanelRows; rows += (uint64_t)N[i]; }
    p.passes = (M + kPanelTokens - 1) / kPanelTokens;
    const int spt = (KB + 1) / 2, most = spt / 16 > 1 ? spt / 16 : 1, room = num_cu / (p.strips * p.passes);
    p.ksplit = room < 1 ? 1 : room < most ? room : most;
    p.us = LaunchCost{num_cu, two_terms ? 2.6 : 1.8, 12.0}.us((uint64_t)p.strips * (uint64_t)p.passes, (uint64_t)p.ksplit,
                                                              (uint64_t)((spt + p.ksplit - 1) / p.ksplit), (uint64_t)M * rows);
    return p;
}

// The kernel that a product of M >= 33 rows takes: the one with the smallest estimate.  slice_kernel keeps four waves on a SIMD and
// cuts finely, but decodes a block once per 128 tokens; strip_kernel decodes it once per 256 and panel_kernel once per 512, with two
// waves per SIMD and tiles that fill the chip only where there are many.  Measured (us, slice / strip / panel):
//   4096 x 4104, M = 256 bf16 45 / 64 / -;  14336 x 4104, M = 250 fp16 84 / 104 / -;  65536 x 4104, M = 128 bf16 245 / 304 / -;
//   14336 x 14352, M = 250 fp16 262 / 236 / -, M = 256 bf16 345 / 289 / -;  65536 x 4104, M = 256 bf16 472 / 308 / -;
//   4096 x 4104, M = 320 fp16 51 / 65 / 56, M = 512 fp16 60 / 92 / 71, M = 1024 fp16 91 / - / 102;  1024 x 4104, M = 512 fp16 30 / 42 / 51,
//   M = 1024 bf16 49 / 75 / 67;  4096 x 14352, M = 512 bf16 201 / - / 165;  14336 x 4104, M = 320 bf16 162 / 172 / 146, M = 1024 fp16
//   337 / 276 / 176;  65536 x 480, M = 300 bf16 112 / 91 / 81.
// Against the faster of two measured kernels the choice loses 0.1 % in the mean and 6 % at most, over 374 products with M >= 257
// (slice or panel) and 236 with 129 <= M <= 256 (slice or strip).
enum Route { kRouteSlice, kRouteStrip, kRoutePanel };
struct RouteCost {
    Route route;
    double us;
};
inline RouteCost best_route(int num_cu, int M, int KB, bool two_terms, int N) {
    RouteCost best = {kRouteSlice, slice_plan(num_cu, M, KB, two_terms, &N, 1).us};
    if (M >= kStripMinM && M <= kStripMaxM) {
        const double us = strip_plan(num_cu, M, KB, two_terms, N).us;
        if (us < best.us) best = {kRouteStrip, us};
    }
    if (panel_reaches(M, KB)) {
        const double us = panel_plan(num_cu, M, KB, two_terms, &N, 1).us;
        if (us < best.us) best = {kRoutePanel, us};
    }
    return best;
}

// Matrices that share x: all in one launch of slice_kernel or of panel_kernel, or one after the other, each as best_route says, where
// the estimates add up to less (or to the same as one launch of panel_kernel: gate and up that each fill the chip gain nothing
// from sharing a launch).  Measured (us, one launch of slice_kernel against one after the other): two of 28672 x 4104 at M = 256,
// bf16, 449 / 371; 65536 and 1024 rows 563 / 330.
enum MultiRoute { kMultiSlice, kMultiPanel, kMultiApart };
inline MultiRoute multi_route(int num_cu, int M, int KB, bool two_terms, const int* N, int n_items) {
    double best = slice_plan(num_cu, M, KB, two_terms, N, n_items).us, apart = 0.0;
    MultiRoute route = kMultiSlice;
    if (panel_reaches(M, KB)) {
        const double us = panel_plan(num_cu, M, KB, two_terms, N, n_items).us;
        if (us < best) { best = us; route = kMultiPanel; }
    }
    for (int i = 0; i < n_items; i++) apart += best_route(num_cu, M, KB, two_terms, N[i]).us;
    return apart < best || (apart == best && route == kMultiPanel) ? kMultiApart : route;
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

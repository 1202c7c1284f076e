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

struct SlicePlan {
    int token_tiles;     // tiles of 32 tokens per pass: 2, 3 or 4
    int passes;
    int strip_rows;
    int ksplit;          // workgroups that share the block pairs of a row
};

// n_items matrices of N[i] rows and KB blocks per row in one launch.  Passes of at most 128 tokens, as even as token tiles
// allow.  The split: the smallest estimated time in us, rounds of workgroups x (steps of a slice x the time of a step + tables
// and final sum), and, when the rows are split, 335 atomics per ns and the clearing of y (all measured).
inline SlicePlan slice_plan(int num_cu, int M, int KB, const int* N, int n_items) {
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
    const double step = p.token_tiles == 2 ? 2.7 : p.token_tiles == 3 ? 3.1 : 3.6;
    double best = 0.0;
    p.ksplit = 1;
    for (uint64_t ks = 1; ks <= 64 && (ks == 1 || (split && ks * slices <= spt)); ks++) {
        const uint64_t rounds = (wgs * ks + num_cu - 1) / num_cu;
        const double t = (double)rounds * ((double)((spt + ks * slices - 1) / (ks * slices)) * step + 6.0) +
                         (ks > 1 ? (double)ks * (double)M * (double)rows / 335e3 + 3.0 : 0.0);
        if (ks == 1 || t < best) { best = t; p.ksplit = (int)ks; }
    }
    return p;
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

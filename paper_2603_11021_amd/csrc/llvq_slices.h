// Where slice_kernel reads its words: plain integer arithmetic, one source for the kernel and for the host test that walks it
// over whole matrices.
#pragma once
#include "llvq_decode_core.h"

namespace llvq {

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

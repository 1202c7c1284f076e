// Constant tables of the LLVQ dequantiser: layout shared by the host-side builder
// (llvq_tables.cpp) and the gfx950 kernels (llvq_kernels.hip).
//
// The dequantiser of the paper's App. A needs, per index: shell/class lookup in cumulative tables,
// the unflattening of the class-local index into (r, s, I''), and a "local combinatorial
// reconstruction".  Here every one of these steps is a lookup in a small table held in LDS:
//   gs      4096 Golay words ordered by (weight, message)                      [paper Sec. 2.3]
//   bucket  top bits of the index -> first candidate class                      [App. A steps 1-2]
//   cls_off cumulative class offsets; cls: one ClassRec per class               [App. A steps 2-3]
//   split   ranking tables of the q-subsets of n slots (12 low + n-12 high)     [App. A step 4]
//   lut12   colex rank -> 12-bit mask, grouped by popcount
//   inner   rank of an arrangement of the minority values -> two bit planes
//   pdep6   deposit of <=6 compressed bits into a 6-bit mask
//   spread6 the same deposit, result spread to one nibble per position
#pragma once
#include <cstdint>
#include <vector>

namespace llvq {

struct alignas(16) ClassRec {
    double   invPP;      // 1/(P1*Pin), nudged upwards so that floor(x*invPP) == x / PP for x < 2^48
    uint32_t PP;         // P1 * Pin
    float    invP1;      // 1/P1 rounded up (exact quotients for dividends < 2^22)
    uint32_t f0;         // bit fields, see F0_* below
    uint32_t f1;         // bit fields, see F1_* below
    uint16_t P1;         // arrangements of the direct F1 word (1 when there is none)
    uint16_t tb1;        // first entry of the direct F1 word's table in `inner`
    uint16_t tb0;        // first entry of the outer domain's inner-word table in `inner`
    uint16_t sp;         // split entry of j is split[sp + j]
};
static_assert(sizeof(ClassRec) == 32, "ClassRec layout");

// Values of the codes 0..7 of a class, one byte each.  Two tables of their own, since a kernel needs one of them:
// fp8 e4m3 (sign bit = bit 7) or int8.
struct ClassVals {
    uint32_t lo, hi;
};

// The same together, for the kernels that read records from global memory: a record's pieces then lie in one cache line.
// The vector cache looks up one lane at a time, so lines count: the seven layers of a Llama-3-8B-shaped block at M = 1 take
// 109.2 us with these, 109.5 with records of 48 bytes, 110.4 with the values in LDS and 110.9 with the values in a table of
// their own in global memory.
struct alignas(64) FullRec {
    ClassRec rec;
    ClassVals v8, vi;
};
static_assert(sizeof(FullRec) == 64, "FullRec layout");

// f0: [0] odd  [1] f1_direct (even class, 0 < w <= 16: F1 planes go through the codeword)
//     [2] outer_all (outer domain = all 24 positions: odd classes and w = 24)
//     [3..7] wm1 = max(w-1,0)  [8] forced-sign enable  [9] kappa (parity of negative F1 signs)
//     [10..14] B  [15..18] m  [19..23] n (slots of the outer domain)  [24..28] q (subset size)
//     Lay19 (whose decoder needs neither n nor q): m takes [15..19], bits 16..23 of tb0 sit in [20..27]
enum { F0_TB0_HI = 20 };
enum { F0_ODD = 0, F0_F1DIRECT = 1, F0_OUTER_ALL = 2, F0_WM1 = 3, F0_FEN = 8, F0_KAPPA = 9,
       F0_B = 10, F0_M = 15, F0_N = 19, F0_Q = 24 };
// f1: [0..11] first Golay word of the class in gs  [12..13] code of A  [14..18] guess shift
//     [19..22] jmax  [23..28] row of the guess table  [29] placed step by step (Lay19 only)
enum { F1_GOFF = 0, F1_ACODE = 12, F1_GSHIFT = 14, F1_JMAX = 19, F1_GROW = 23, F1_STEPS = 29 };

struct alignas(16) SplitEnt {
    uint32_t base;       // number of subsets with fewer high slots
    float    inv;        // 1 / C(nl, q-j), rounded up
    uint16_t div;        // C(nl, q-j)
    uint16_t b12lo;      // lut12 base of popcount q-j
    uint16_t b12hi;      // lut12 base of popcount j
    uint16_t pad;
};
static_assert(sizeof(SplitEnt) == 16, "SplitEnt layout");

// Fixed byte offsets of the tables inside the blob.  The first kLdsBytes of the blob are copied verbatim into LDS
// by every kernel; the offsets are compile-time constants so that the kernels can fold them into the offset field
// of the LDS instructions.  The two large tables that are read once or twice per block (the sorted Golay words and
// the inner-word planes) come last: a kernel either copies the whole blob into LDS or only the first kLdsBytes and
// reads those two through the vector L1/L2 (a shorter table copy per launch, at the price of three global gathers
// per block).
constexpr uint32_t kSpreadPitch = 65;      // dwords per mask row of spread6: entry (F, m) at F * 65 + m, so that equal m of
                                           // different masks (all-zero sources are frequent) fall into different LDS banks
constexpr uint32_t kPdepPitch  = 68;       // bytes per mask row of pdep6 (17 dwords, for the same reason)
struct Lay13 {
    static constexpr bool kWide = false;
    static constexpr uint32_t kOffSpread6 = 0;        // 64 x 65 x u32
    static constexpr uint32_t kOffPdep6   = 16640;    // 64 x 68 x u8
    static constexpr uint32_t kOffLut12   = 20992;    // 4096 x u16
    static constexpr uint32_t kOffBucket  = 29184;    // 4096 x u16: 8 x class id (the byte offset of its entry in cls_off)
    static constexpr uint32_t kOffGuess   = 37376;    // up to 48 rows x 64 x u8
    static constexpr uint32_t kOffAtab    = 40448;    // 4 x {A, 1/A} doubles
    static constexpr uint32_t kOffClsOff  = 40512;    // (ncls + 4) x u64, ncls <= 383: offsets, N, and three entries above every index
    static constexpr uint32_t kOffRnorm   = 43616;    // 16 x float: 1/sqrt(16 m)
    static constexpr uint32_t kOffSplit   = 43680;    // up to 188 x SplitEnt
    static constexpr uint32_t kOffCls     = 46688;    // ncls x ClassRec
    static constexpr uint32_t kOffVt8     = 58944;    // ncls x ClassVals, fp8
    static constexpr uint32_t kOffVti     = 62016;    // ncls x ClassVals, int8
    static constexpr uint32_t kLdsBytes   = 65088;    // end of the tables that every kernel keeps in LDS
    static constexpr uint32_t kOffGs      = 65088;    // 4096 x u32
    static constexpr uint32_t kOffInner   = 81472;    // inner-word planes, u32
    static constexpr uint32_t kMaxBlob    = 81472 + 4 * 65536;   // the inner-word table bases are 16-bit entry numbers
    static constexpr uint32_t kOffFullRec = (kMaxBlob + 127u) & ~127u;    // ncls x FullRec, in global memory only
    static constexpr uint32_t kBucketShift = 36;      // bucket index = I >> 36 (4096 buckets cover 48 bits)
    static constexpr uint64_t kWordMask   = (1ull << 48) - 1;    // bits of a 64-bit word that hold index and gain code
};

// The unions up to shell 19: 1,457 classes, 55-bit indices, at most 2^49.6 points per class (so the quotients stay exact
// in fp64), 5 MB of inner-word planes.  The planes and whatever follows the Golay words stay in global memory: 69 KB of
// class records beside the small tables and the Golay words would fit LDS, but then one workgroup fills a compute unit and
// a launch copies 146 KB.  Classes that three-bit value codes with two 16-bit planes cannot describe (subsets of more than
// 16 slots or more than four minority values: 3 in a million indices) carry F1_STEPS and are placed step by step from
// their WideRec (llvq_wide.h).  Against the step-by-step decoder with all tables in global memory that this replaced:
// 4096 x 4104 at M = 1 236 -> 16.9 us, 4 M blocks to int8 430 -> 58 us (M = 16: 21.1 us).
struct Lay19 {
    static constexpr bool kWide = true;
    static constexpr uint32_t kOffSpread6 = 0;
    static constexpr uint32_t kOffPdep6   = 16640;
    static constexpr uint32_t kOffLut12   = 20992;
    static constexpr uint32_t kOffBucket  = 29184;
    static constexpr uint32_t kOffGuess   = 37376;    // up to 63 rows x 64 x u8
    static constexpr uint32_t kOffAtab    = 41408;
    static constexpr uint32_t kOffClsOff  = 41472;    // (ncls + 4) x u64, ncls <= 1457
    static constexpr uint32_t kOffRnorm   = 53168;    // 20 x float
    static constexpr uint32_t kOffSplit   = 53248;    // up to 512 x SplitEnt
    static constexpr uint32_t kLdsBytes   = 61440;
    static constexpr uint32_t kOffGs      = 61440;    // 4096 x u32
    static constexpr uint32_t kOffFullRec = 77824;    // ncls x FullRec (global memory, like all that follows)
    static constexpr uint32_t kOffWideRec = 171072;   // ncls x WideRec
    static constexpr uint32_t kOffBinom   = 264320;   // 25 x 25 x u32
    static constexpr uint32_t kOffInner   = 266832;   // inner-word planes
    static constexpr uint32_t kMaxBlob    = 266832 + 4 * (1u << 24);
    static constexpr uint32_t kBucketShift = 43;      // 4096 buckets cover 55 bits
    static constexpr uint64_t kWordMask   = (1ull << 56) - 1;
};
constexpr uint32_t kGuessBuckets = 64;     // buckets of the subset-split guess table per (n, q)

struct TableLayout {
    uint32_t lds_bytes;      // first part of the blob: the tables every kernel keeps in LDS
    uint32_t blob_bytes;     // up to the end of the inner-word planes (kernels that want all tables in LDS copy this many bytes)
    uint32_t ncls;
    uint32_t inner_entries;
    uint64_t npoints;        // N(m_max)
};

// ---- tables of the encoder-side index map (point -> index), a blob of their own ---------------------
// One record per class, in class order.  The point's class is found by hashing the key below; the code of each
// coordinate (the same nibble codes the decoder produces) comes from an 8-entry table indexed by |x| >> 1.
struct alignas(16) EncRec {
    uint64_t offset;            // index of the first point of the class
    uint32_t key;               // sum |x|^4  |  (sum |x|) << 20  |  parity << 29: identifies the leader
    uint32_t f0;                // the bit fields of ClassRec::f0
    uint32_t ctab_lo, ctab_hi;  // nibble code of the absolute value 2k (even classes) or 2k+1 (odd), k = 0..7
    uint32_t Pin;               // arrangements of the inner word of the outer domain
    uint32_t e1;                // bit fields, see E1_* below
    uint16_t P1;                // arrangements of the direct F1 word
    uint16_t sp;                // split entry of j is split[sp + j]
    uint16_t rad0[2];           // radices of the first two digits of the outer domain's inner word
    uint16_t rad1[2];           // the same for the direct F1 word
    uint32_t pad;
};
static_assert(sizeof(EncRec) == 48, "EncRec layout");
// e1: [0..11] first Golay word of the class in gs  [12..13] code of A  [14..15] digits of the outer inner word
//     [16..17] digits of the direct F1 word  [18] first symbol of the outer inner word (0 or 1)
enum { E1_GOFF = 0, E1_ACODE = 12, E1_DIG0 = 14, E1_DIG1 = 16, E1_SYM0 = 18 };

constexpr uint32_t kEncGs     = 0;        // 4096 x u32, the decoder's sorted Golay words
constexpr uint32_t kEncGinv   = 16384;    // 4096 x u16: low 12 bits of a word -> its position in gs
constexpr uint32_t kEncRank12 = 24576;    // 4096 x u16: colex rank of a 12-bit mask among the masks of its popcount
constexpr uint32_t kEncPext6  = 32768;    // 4096 x u8: extraction of the bits of a 6-bit source under a 6-bit mask
constexpr uint32_t kEncHash   = 36864;    // 2 x 512 x HashEnt: cuckoo table of the class keys
constexpr uint32_t kEncG16    = 45056;    // 16 x 17 x u16: masks of popcount p whose bits 12..15 are below H
constexpr uint32_t kEncSplit  = 46080;    // the decoder's SplitEnt array
constexpr uint32_t kEncCls    = 51712;    // ncls x EncRec
constexpr uint32_t kEncBlob   = 70144;    // 68.5 KB
constexpr uint32_t kEncHashBits = 9;      // slots per half of the cuckoo table

// a key sits in slot (key * mult[h]) >> (32 - kEncHashBits) of half h, for h = 0 or h = 1
struct HashEnt {
    uint32_t key;     // 0xFFFFFFFF: empty
    uint32_t cid;
};

struct EncLayout {
    uint32_t bytes;          // bytes of the encoder blob = bytes resident in LDS
    uint32_t ncls;
    uint32_t hash_mult[2];   // multipliers of the two halves of the cuckoo table
    uint32_t m_max;
};

// ---- tables of the nearest-point search: one record per class, read with wave-uniform (scalar) loads ----
// coef: the 24 coefficients the sorted input is multiplied with.  Odd class: +a for a = 1 (mod 4), -a for
// a = 3 (mod 4), in descending order.  Even class: the 2-mod-4 values in descending order (w of them), then the
// 0-mod-4 values in descending order.
struct alignas(128) SearchRec {
    float    coef[24];
    float    mul[2];     // score = <w, x> * mul[metric] + bias[metric]: {1 / sqrt(16 m), 1}
    float    bias[2];    //                                              {0, -||x||^2 / 2 = -8 m}
    float    amin2;      // twice the smallest 2-mod-4 value (0 when there is none): cost factor of the parity repair
    uint32_t kappa;      // parity that the number of negative F1 signs must have
    uint32_t cid;        // class id
    uint32_t w;          // Golay weight of the class (odd classes: 0)
};
static_assert(sizeof(SearchRec) == 128, "SearchRec layout");

// records are ordered: all odd classes, then the even classes grouped by weight 0, 8, 12, 16, 24
constexpr int kMaxSearchTiles = 16;
struct SearchLayout {
    uint32_t n_odd;
    uint32_t even_first[5];
    uint32_t even_count[5];
    uint32_t total;
    // the same records cut into tiles of 32 classes for the matrix cores; group 0 = odd, 1..5 = even weights 0, 8, 12, 16, 24
    uint32_t n_tiles;
    uint32_t grp_tile_first[6];
    uint32_t grp_tile_count[6];
    uint32_t tile_first_rec[kMaxSearchTiles];
    uint32_t tile_rows[kMaxSearchTiles];      // valid classes in the tile (the rest is padding)
};
// Matrix-core operands of a tile: A[tile][kb][lane] = eight bf16 values, class row lane % 32, k = 16 kb + 8 (lane / 32) + t.
// k = 0..23: the record's coef; even classes: k = 24 holds -amin2 when kappa = 0, k = 25 holds -amin2 when kappa = 1.
// Scale[tile][metric][lane / 32][r]: the factor (angular metric) or the offset (Euclidean metric) of the class in
// accumulator slot r (row 8 (r / 4) + 4 (lane / 32) + r % 4).  Padding rows repeat the first class of the tile.
constexpr uint32_t kSearchTileABytes = 2 * 64 * 16;
constexpr uint32_t kSearchTileScaleFloats = 2 * 2 * 16;

// nibble slot (0..7) of chunk position 0..5 inside a spread6 entry
static constexpr int kNibbleSlot[6] = {0, 2, 1, 3, 4, 6};

struct Tables {
    TableLayout lay;
    uint64_t shell_off[16];  // index of the first point of shell m (N(m-1)); entries above m_max hold N(m_max)
    std::vector<unsigned char> blob;
    EncLayout enc_lay;
    std::vector<unsigned char> enc_blob;
    SearchLayout search_lay;
    std::vector<SearchRec> search_recs;
    std::vector<uint16_t> search_tile_a;      // n_tiles x 2 x 64 x 8 bf16
    std::vector<float> search_tile_scale;     // n_tiles x kSearchTileScaleFloats
};

// Builds every table for Lambda_24(m_max), 2 <= m_max <= 13.  Returns false on an internal inconsistency.
bool build_tables(int m_max, Tables& out);

}  // namespace llvq

// Test-only harness: runs the library's table builder and its index -> block reconstruction on the host CPU
// so that the host logic (tables, digit extraction, ranking) can be compared with the oracle without a GPU.
// It is not part of the library and nothing in the product links to it.
#include <cstdint>
#include <cstring>

#include "../../paper_2603_11021_amd/csrc/llvq_decode_core.h"
#include "../../paper_2603_11021_amd/csrc/llvq_encode_core.h"
#include "../../paper_2603_11021_amd/csrc/llvq_plan.h"
#include "../../paper_2603_11021_amd/csrc/llvq_tables.h"
#include "../../paper_2603_11021_amd/csrc/llvq_wide.h"

static llvq::Tables g_tabs;
static bool g_ok = false;

// The whole of App. A for these unions in one call, step by step and without the decoder's tables: its class records, offsets, Golay
// words and binomial coefficients are those of the blob that llvq_create copies to the device.
struct WidePtrs {
    const llvq::WideRec* recs;
    const uint64_t* cls_off;   // first index of every class, then N
    const uint32_t* gs;        // 4096 Golay words ordered by (weight, message)
    const uint32_t* binom;     // 25 x 25 binomial coefficients C(n, k) at [n * 25 + k]
    uint32_t ncls;
    uint64_t npoints;
};

// index I < npoints -> 24 int8 coordinates (six dwords, position order)
static void wide_decode(const WidePtrs& T, uint64_t I, uint32_t (&out)[6]) {
    // App. A steps 1-2: the class whose range of indices holds I
    uint32_t lo = 0, hi = T.ncls;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (I >= T.cls_off[mid]) lo = mid; else hi = mid;
    }
    const llvq::WideRec R = T.recs[lo];
    // step 3: r = Ic mod A, then B sign bits, then I'' = (d * Pin + rin) * P1 + rho1
    uint64_t t = I - T.cls_off[lo];
    const uint32_t r = (uint32_t)(t % R.A);
    t /= R.A;
    const uint32_t s = (uint32_t)(t & ((1ull << R.B) - 1ull));
    t >>= R.B;
    const uint32_t rho1 = (uint32_t)(t % R.P1);
    t /= R.P1;
    const uint64_t rin = t % R.Pin;
    const uint32_t d = (uint32_t)(t / R.Pin);
    // step 4: Golay word, placement, signs
    int8_t x[24] = {};
    const uint32_t neg = llvq::wide_place(T.binom, R, T.gs[R.goff + r], s, d, rin, rho1, [&](uint32_t occ, int, int v) {
        for (int p = 0; p < 24; p++) if ((occ >> p) & 1u) x[p] = (int8_t)v;
    });
    for (int p = 0; p < 24; p++) if ((neg >> p) & 1u) x[p] = (int8_t)-x[p];
    for (int k = 0; k < 6; k++)
        out[k] = (uint32_t)(uint8_t)x[4 * k] | ((uint32_t)(uint8_t)x[4 * k + 1] << 8) | ((uint32_t)(uint8_t)x[4 * k + 2] << 16) |
                 ((uint32_t)(uint8_t)x[4 * k + 3] << 24);
}

extern "C" {

int emul_init(int m_max) {
    g_ok = llvq::build_tables(m_max, g_tabs);
    return g_ok ? 0 : -1;
}

uint32_t emul_lds_bytes() { return g_tabs.lay.blob_bytes; }     // the most any kernel copies into LDS
uint32_t emul_num_classes() { return g_tabs.lay.ncls; }
uint64_t emul_num_points() { return g_tabs.lay.npoints; }
uint32_t emul_inner_entries() { return g_tabs.lay.inner_entries; }

// returns the number of out-of-range indices (decoded to zero)
uint64_t emul_decode_i8(const uint64_t* idx, uint64_t n, int8_t* out) {
    const llvq::TabPtrs T = llvq::make_tab_ptrs(g_tabs.blob.data(), g_tabs.blob.data(), g_tabs.lay);
    uint64_t bad = 0;
    for (uint64_t k = 0; k < n; k++) {
        if (idx[k] >= T.npoints) { bad++; std::memset(out + 24 * k, 0, 24); continue; }
        uint32_t w[4], o[6];
        const llvq::BlockInfo bi = llvq::decode_block(T, idx[k], w);
        llvq::nibbles_to_i8(w, bi.vti_lo, bi.vti_hi, o);
        std::memcpy(out + 24 * k, o, 24);
    }
    return bad;
}

uint32_t emul_enc_bytes() { return g_tabs.enc_lay.bytes; }

// pts: n x 24 int8; idx receives the index or all ones; returns the number of vectors that are not points
uint64_t emul_encode(const int8_t* pts, uint64_t n, uint64_t* idx) {
    const llvq::EncPtrs T = llvq::make_enc_ptrs(g_tabs.enc_blob.data(), g_tabs.enc_lay);
    uint64_t bad = 0;
    for (uint64_t k = 0; k < n; k++) {
        uint32_t x[6];
        std::memcpy(x, pts + 24 * k, 24);
        idx[k] = llvq::encode_block(T, x);
        bad += idx[k] == llvq::kInvalidIndex;
    }
    return bad;
}

// ---- the decoder of the larger unions (m_max up to 19) ------------------------------------------------------
static llvq::WideTables g_wide;

int emul_wide_init(int m_max) { return llvq::build_wide_tables(m_max, g_wide) ? 0 : -1; }
uint32_t emul_wide_num_classes() { return g_wide.tab.ncls; }
uint64_t emul_wide_num_points() { return g_wide.tab.npoints; }
uint64_t emul_wide_shell_offset(int m) { return (m >= 0 && m < 24) ? g_wide.shell_off[m] : 0; }

uint64_t emul_wide_decode_i8(const uint64_t* idx, uint64_t n, int8_t* out) {
    using llvq::Lay19;
    const unsigned char* blob = g_wide.blob.data();
    const WidePtrs T = {reinterpret_cast<const llvq::WideRec*>(blob + Lay19::kOffWideRec), reinterpret_cast<const uint64_t*>(blob + Lay19::kOffClsOff),
                        reinterpret_cast<const uint32_t*>(blob + Lay19::kOffGs), reinterpret_cast<const uint32_t*>(blob + Lay19::kOffBinom),
                        g_wide.tab.ncls, g_wide.tab.npoints};
    uint64_t bad = 0;
    for (uint64_t k = 0; k < n; k++) {
        if (idx[k] >= T.npoints) { bad++; std::memset(out + 24 * k, 0, 24); continue; }
        uint32_t o[6];
        wide_decode(T, idx[k], o);
        std::memcpy(out + 24 * k, o, 24);
    }
    return bad;
}

// the same indices through the table-driven decoder in the layout of these unions (what the kernels run)
uint64_t emul_wide_tab_decode_i8(const uint64_t* idx, uint64_t n, int8_t* out) {
    const auto T = llvq::make_tab_ptrs<llvq::Lay19>(g_wide.blob.data(), g_wide.blob.data(), g_wide.tab);
    uint64_t bad = 0;
    for (uint64_t k = 0; k < n; k++) {
        if (idx[k] >= T.npoints) { bad++; std::memset(out + 24 * k, 0, 24); continue; }
        uint32_t w[4], o[6];
        const llvq::BlockInfo bi = llvq::decode_block(T, idx[k], w);
        llvq::nibbles_to_i8(w, bi.vti_lo, bi.vti_hi, o);
        std::memcpy(out + 24 * k, o, 24);
    }
    return bad;
}

// ---- the words slice_kernel reads ---------------------------------------------------------------------------
// Walks every lane of every strip of `strip_rows` rows through the pairs it fetches (all steps of a row, or the first and the
// last 64 of a long one) and returns how many of them do not lie inside the N x KB words or do not hold the lane's block where
// `late` says it is.
uint64_t emul_slice_pairs_wrong(int N, int KB, int strip_rows) {
    uint64_t wrong = 0;
    const int64_t words = (int64_t)N * KB;
    const int steps = (KB + 1) / 2;
    for (int row0 = 0; row0 < N; row0 += strip_rows)
        for (int r = 0; r < strip_rows; r++) {
            const llvq::SliceWords sw = llvq::slice_words(row0, row0 + r, N, KB);
            const int row = row0 + r < N ? row0 + r : N - 1;
            for (int st = 0; st < steps; st = (st == 63 && steps > 128) ? steps - 64 : st + 1)
                for (int half = 0; half < 2; half++)
                    for (int real = 0; real < 2; real++) {
                        bool late = false;
                        const uint32_t kk = llvq::slice_pair(sw, (uint32_t)st, (uint32_t)half, (uint32_t)KB, real != 0, late);
                        const int64_t pair = (int64_t)sw.first + (int64_t)(uint64_t)kk;      // kk is an unsigned offset in the kernel too
                        bool ok = pair >= 0 && pair + 1 < words;
                        if (real) {
                            const int b = 2 * (st + half) < KB ? 2 * (st + half) : KB - 1;
                            ok = ok && pair + (late ? 1 : 0) == (int64_t)row * KB + b;
                        }
                        wrong += !ok;
                    }
        }
    return wrong;
}

// How n_items matrices are multiplied on a device of num_cu compute units: token tiles, passes, rows per strip and split of K of one
// launch of slice_kernel; split of K of strip_kernel (first matrix) and of one launch of panel_kernel; the route of the first
// matrix alone (0 slice, 1 strip, 2 panel) and of all (0 slice, 1 panel, 2 one after the other).
void emul_plan(int num_cu, int M, int KB, int two_terms, const int* N, int n_items, int* out) {
    const bool two = two_terms != 0;
    const llvq::SlicePlan p = llvq::slice_plan(num_cu, M, KB, two, N, n_items);
    out[0] = p.token_tiles; out[1] = p.passes; out[2] = p.strip_rows; out[3] = p.ksplit;
    out[4] = llvq::strip_plan(num_cu, M, KB, two, N[0]).ksplit;
    out[5] = llvq::panel_plan(num_cu, M, KB, two, N, n_items).ksplit;
    out[6] = llvq::best_route(num_cu, M, KB, two, N[0]).route;
    out[7] = llvq::multi_route(num_cu, M, KB, two, N, n_items);
}

}  // extern "C"

// Plan and workspace of the ranked order of a test's records (sort.hip), host only.
#pragma once

#include <cstddef>
#include <cstdint>

namespace gss {

constexpr uint32_t kRankBlock = 1u << 16;  // cells per workgroup of the packing kernel (1024 words of 64)
// the largest table and list that one workgroup orders in LDS (k_rank_small)
constexpr uint32_t kSmallCells = 1u << 18, kSmallRecords = 1u << 14;

// Whether hit words of that size are ranked (not too small, nor beyond 32-bit cells).
inline bool rank_uses_hits(uint64_t bytes) { return bytes * 8 > kSmallCells && bytes * 8 <= (1ull << 31); }

// The plan for a test's records: from the test's hit words where
// it kept them (bit cells, already marked).  Otherwise bit cells cost an atomic a
// record (2 M took 169 us), byte cells a byte written and one read a cell (96 M took
// 45 us): bits where a record comes to 240 cells or more.  Then the cells cost little
// (an eighth of a byte written and read) and so does the workspace, and the radix sort
// (158 us for 43 K records, 238 us for 815 K) is left for cells beyond 2^31; the
// kernels index cells by 32 bits.
struct RankPlan {
    uint32_t w_log2 = 0;
    uint64_t cells = 0, words = 0, blocks = 0;
    size_t marks = 0, packed = 0;  // bytes
    bool hits = false, bits = false, fits = false, small = false;

    // ids issued, words of a row and of a chunk of it, records kept; whether the test's
    // hit words are there, and the ids that they cover
    RankPlan(uint64_t ids, uint32_t W, uint32_t RWc, uint64_t kept, bool has_hits, uint64_t hits_ids) {
        while ((1u << w_log2) < W) ++w_log2;  // a power of two of words per issued id
        cells = (ids << w_log2) + 64;
        words = (cells + 63) / 64;
        small = cells <= kSmallCells && kept <= kSmallRecords;
        hits = has_hits && !small;
        if (hits) {  // the test's own bit cells
            w_log2 = 0;
            while ((1u << w_log2) < RWc) ++w_log2;
            words = (hits_ids * RWc + 511) / 512 * 8;
            cells = words * 64;
        }
        blocks = (cells + kRankBlock - 1) / kRankBlock;
        bits = hits || kept < cells / 240;
        marks = hits ? 0 : (words * (bits ? 8 : 64) + 255) / 256 * 256;
        packed = (words * (bits ? 4 : 16) + 255) / 256 * 256;
        fits = cells <= (1ull << 31);
    }

    // device memory of its kernels (none for a small table)
    uint64_t bytes() const { return small ? 0 : marks + packed + (blocks * 4 + 255) / 256 * 256; }
    // whether the order can be made by ranking with that much: otherwise the radix sort makes it
    bool fits_in(uint64_t have) const { return small || (fits && bytes() <= have); }
};

// The workspace of the ranked order: what is at ws already (bytes of it, null: nothing),
// or allocated here (own).  Every allocation may give up the hit words, and the plan
// without them can need more or be none at all, so that plan() is asked again after each.
struct RankSpace {
    bool ranked = false;  // false: no plan fits, the radix sort
    char *ws = nullptr, *own = nullptr;
    uint64_t bytes = 0;
};

template <class PlanFn, class Alloc, class Release>
RankSpace rank_space(PlanFn plan, char *ws, uint64_t bytes, Alloc alloc, Release release) {
    RankSpace s;
    const RankPlan p = plan();
    if (p.fits_in(ws ? bytes : 0)) {
        s.ranked = true;
        s.ws = ws;
        s.bytes = ws ? bytes : 0;
        return s;
    }
    if (!p.fits) return s;
    char *own = alloc(p.bytes());  // null: no room
    if (!own) return s;
    if (!plan().fits_in(p.bytes())) {
        release(own);
        return s;
    }
    s.ranked = true;
    s.ws = s.own = own;
    s.bytes = p.bytes();
    return s;
}

}  // namespace gss

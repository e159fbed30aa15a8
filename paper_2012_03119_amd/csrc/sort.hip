// Ordered reports (GSS_TEST_SORTED): the kept records of a test, ordered by
// (clause id, word).  Two ways, one result:
//
// Ranked (rank_records): a test has at most one record per (clause id, word), so a
// record's place is the number of records at smaller (id, word) cells.  One pass
// over the report segments marks the cells (a byte store each: no two records share
// one, so no atomics; where the records are few among the cells, a bit each), one over
// the cells takes the running counts of words of 64, and one more over the segments
// stores each record at its place.  Where the test kept the marks itself (its hit words,
// store_hits) the first pass is left out.  The records are read twice, or once with hit
// words, and written once, straight from the segments.
//
// Radix (sort_records), where there are more than 2^31 cells or they do not fit the
// memory budget: a least-significant-digit radix sort written for this library.  The key packs clause id and word ((id << word_bits) | word); each
// pass orders the 16-byte records stably by one 8-bit digit of it:
//
//   1. per workgroup tile of 4096 records, the count of each digit (LDS);
//   2. one exclusive scan over the counts, digit-major, so that the records of
//      digit d from tile b start after every smaller digit and after digit d of
//      the tiles before b;
//   3. per tile, every record's rank among the equal digits before it: within a
//      wavefront from the lanes below it that share its digit (eight ballots),
//      across the tile's wavefronts and rounds from counts kept in LDS.
//
// A pass whose digit is the same for every record (the high bits of small ids)
// is skipped; a first read of the records counts every pass's digits at once.
#include "gss_internal.h"

#include <algorithm>

namespace gss {
namespace {

constexpr uint32_t kSortThreads = 256;                   // four wavefronts
constexpr uint32_t kSortRounds = 16;                     // records per thread per tile
constexpr uint32_t kSortTile = kSortThreads * kSortRounds;
constexpr uint32_t kRadix = 256;
constexpr uint32_t kMaxPasses = 8;                       // keys of up to 64 bits

__device__ inline uint64_t record_key(const gss_report &r, uint32_t word_bits) {
    return ((uint64_t)r.clause_id << word_bits) | r.word;
}

__device__ inline uint32_t lanes_below_mask(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// counts[p][d]: records whose digit p is d.
__global__ __launch_bounds__(kSortThreads) void k_sort_digits(const gss_report *r, uint64_t n, uint32_t word_bits,
                                                              uint32_t n_passes, unsigned long long *counts) {
    __shared__ uint32_t h[kMaxPasses][kRadix];
    for (uint32_t i = threadIdx.x; i < kMaxPasses * kRadix; i += blockDim.x) (&h[0][0])[i] = 0;
    __syncthreads();
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t k = record_key(r[i], word_bits);
        for (uint32_t p = 0; p < n_passes; ++p) atomicAdd(&h[p][(k >> (8 * p)) & 0xFF], 1u);
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n_passes * kRadix; i += blockDim.x)
        if ((&h[0][0])[i]) atomicAdd(&counts[i], (unsigned long long)(&h[0][0])[i]);
}

// hist[d * n_tiles + b]: records of tile b whose digit (at `shift`) is d.
__global__ __launch_bounds__(kSortThreads) void k_sort_tile_counts(const gss_report *r, uint64_t n, uint32_t word_bits,
                                                                   uint32_t shift, uint32_t *hist, uint32_t n_tiles) {
    __shared__ uint32_t h[kRadix];
    h[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t lo = (uint64_t)blockIdx.x * kSortTile, hi = min(n, lo + kSortTile);
    for (uint64_t i = lo + threadIdx.x; i < hi; i += kSortThreads)
        atomicAdd(&h[(record_key(r[i], word_bits) >> shift) & 0xFF], 1u);
    __syncthreads();
    hist[(uint64_t)threadIdx.x * n_tiles + blockIdx.x] = h[threadIdx.x];
}

// Scan of many counts in three launches: sums of chunks of 4096, their scan by one
// workgroup, the chunks again from their bases.  One workgroup alone read 610
// counts a thread, one line each, for the 625 K counts of 10 M records: 1.2 ms for
// each of the four passes' scans.
constexpr uint32_t kScanChunk = 4096;

__global__ __launch_bounds__(256) void k_scan_sums(const uint32_t *x, uint64_t m, uint32_t *sums) {
    __shared__ uint32_t part[4];
    const uint64_t lo = (uint64_t)blockIdx.x * kScanChunk + threadIdx.x;
    uint32_t v = 0;
#pragma unroll
    for (uint32_t k = 0; k < kScanChunk; k += 256) v += lo + k < m ? x[lo + k] : 0u;
    for (uint32_t off = 32; off; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x / 64] = v;
    __syncthreads();
    if (threadIdx.x == 0) sums[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

// x becomes its exclusive scan; sums: the chunks' bases.  Round r takes 256 counts.
__global__ __launch_bounds__(256) void k_scan_apply(uint32_t *x, uint64_t m, const uint32_t *sums) {
    __shared__ uint32_t wave_sum[2][4];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t lo = (uint64_t)blockIdx.x * kScanChunk + threadIdx.x;
    uint32_t v[kScanChunk / 256];
#pragma unroll
    for (uint32_t k = 0; k < kScanChunk / 256; ++k) v[k] = lo + 256 * k < m ? x[lo + 256 * k] : 0u;
    uint32_t run = sums[blockIdx.x];
#pragma unroll
    for (uint32_t k = 0; k < kScanChunk / 256; ++k) {
        uint32_t s = v[k];
#pragma unroll
        for (uint32_t d = 1; d < 64; d <<= 1) {
            const uint32_t y = __shfl_up(s, d);
            if (lane >= d) s += y;
        }
        if (lane == 63) wave_sum[k & 1][wave] = s;
        __syncthreads();  // the other half of wave_sum is rewritten only behind the next round's barrier
        uint32_t before = run;
#pragma unroll
        for (uint32_t w = 0; w < 4; ++w) {
            before += w < wave ? wave_sum[k & 1][w] : 0u;
            run += wave_sum[k & 1][w];
        }
        if (lo + 256 * k < m) x[lo + 256 * k] = before + s - v[k];
    }
}

// In-place exclusive scan of m counts by one workgroup of 1024 threads, each
// taking a contiguous share (also the store's compaction offsets).
__global__ __launch_bounds__(1024) void k_sort_scan(uint32_t *x, uint64_t m) {
    __shared__ uint32_t part[1024];
    const uint32_t t = threadIdx.x;
    const uint64_t per = (m + 1023) / 1024, lo = t * per, hi = min(m, lo + per);
    uint32_t sum = 0;
    for (uint64_t i = lo; i < hi; ++i) sum += x[i];
    part[t] = sum;
    __syncthreads();
    for (uint32_t off = 1; off < 1024; off <<= 1) {  // inclusive Hillis-Steele scan
        const uint32_t v = t >= off ? part[t - off] : 0u;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    uint32_t run = t ? part[t - 1] : 0u;
    for (uint64_t i = lo; i < hi; ++i) {
        const uint32_t v = x[i];
        x[i] = run;
        run += v;
    }
}

// Stable scatter of one digit: the tile's records go in rounds of 256 (record
// lo + 256 * round + thread), so that index order is (round, wavefront, lane).
__global__ __launch_bounds__(kSortThreads) void k_sort_scatter(const gss_report *in, gss_report *out, uint64_t n,
                                                               uint32_t word_bits, uint32_t shift,
                                                               const uint32_t *offsets, uint32_t n_tiles) {
    constexpr uint32_t kWaves = kSortThreads / 64;
    __shared__ uint32_t base[kRadix];           // where the tile's records of each digit start, plus those placed
    __shared__ uint32_t per_wave[kWaves][kRadix];
    const uint32_t t = threadIdx.x, wave = t / 64;
    base[t] = offsets[(uint64_t)t * n_tiles + blockIdx.x];
    const uint64_t lo = (uint64_t)blockIdx.x * kSortTile, hi = min(n, lo + kSortTile);
    for (uint32_t round = 0; round < kSortRounds; ++round) {
        for (uint32_t w = 0; w < kWaves; ++w) per_wave[w][t] = 0;
        __syncthreads();
        const uint64_t i = lo + (uint64_t)round * kSortThreads + t;
        const bool valid = i < hi;
        gss_report rec{};
        uint32_t d = 0;
        if (valid) {
            rec = in[i];
            d = (uint32_t)((record_key(rec, word_bits) >> shift) & 0xFF);
        }
        // the lanes of this wavefront holding the same digit
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (uint32_t b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t rank = lanes_below_mask(peers);  // peers in lower lanes
        if (valid && rank == 0) per_wave[wave][d] = (uint32_t)__builtin_popcountll(peers);
        __syncthreads();
        if (valid) {
            uint32_t pos = base[d] + rank;
            for (uint32_t w = 0; w < wave; ++w) pos += per_wave[w][d];
            out[pos] = rec;
        }
        __syncthreads();
        uint32_t placed = 0;
        for (uint32_t w = 0; w < kWaves; ++w) placed += per_wave[w][t];
        base[t] += placed;
        __syncthreads();
    }
}

// ---- ranked order ------------------------------------------------------------

// Marks the cell id << w_log2 | word of every kept record, where the test kept no hit
// words (rows under 8 words or over 64, the aggregate pre-test); one workgroup per segment.
// A cell is a byte, stored, or (BITS) a bit, set by an atomic.  Bound by the segments'
// reads (8 of each record's 16 bytes are used, but whole lines come in), or by the
// atomics, carried out past the per-XCD caches at about 12 G a second.  No test writes a
// record outside the table; one would be left out (here and below) rather than written.
template <bool BITS>
__global__ __launch_bounds__(256) void k_rank_mark(const gss_report *reports, const uint32_t *counts, uint32_t seg_cap,
                                                   uint32_t n_segments, uint32_t w_log2, uint32_t n_cells,
                                                   void *cells) {
    for (uint32_t s = blockIdx.x; s < n_segments; s += gridDim.x) {
        const uint32_t n = min(counts[s], seg_cap);
        const gss_report *seg = reports + (uint64_t)s * seg_cap;
        for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
            const uint64_t cell = ((uint64_t)seg[i].clause_id << w_log2) + seg[i].word;
            if (cell >= n_cells) continue;
            if constexpr (BITS)
                atomicOr(reinterpret_cast<uint32_t *>(cells) + (cell >> 5), 1u << (cell & 31));
            else
                reinterpret_cast<uint8_t *>(cells)[cell] = 1;
        }
    }
}

// Counts the marked cells, 64 a lane: the running count before each 64 within the
// workgroup's 65536, and the workgroup's total.  Byte cells are packed on the way, into
// (bits, bits, count, 0); bit cells stay as they are, with an array of counts beside
// them.  Four rounds of 256 words; the running count crosses rounds in a register
// every lane holds.
template <bool BITS>
__global__ __launch_bounds__(256) void k_rank_pack(const void *cells, uint32_t n_words, void *packed,
                                                   uint32_t *totals) {
    __shared__ uint32_t wave_sum[2][4];
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6;
    uint32_t run = 0;
#pragma unroll
    for (uint32_t r = 0; r < kRankBlock / 64 / 256; ++r) {
        const uint32_t w = blockIdx.x * (kRankBlock / 64) + 256 * r + t;
        uint32_t bits[2] = {0, 0};
        if (w < n_words) {
            if constexpr (BITS) {
                const uint2 c = reinterpret_cast<const uint2 *>(cells)[w];
                bits[0] = c.x;
                bits[1] = c.y;
            } else {
#pragma unroll
                for (uint32_t q = 0; q < 4; ++q) {
                    const uint4 c = reinterpret_cast<const uint4 *>(cells)[(uint64_t)w * 4 + q];
                    const uint32_t u[4] = {c.x, c.y, c.z, c.w};
                    // four cells (bytes 0 or 1) to four bits: byte i lands on bit 28 + i of the product
#pragma unroll
                    for (uint32_t k = 0; k < 4; ++k)
                        bits[q / 2] |= ((u[k] * 0x10204080u) >> 28) << (16 * (q % 2) + 4 * k);
                }
            }
        }
        const uint32_t mine = __builtin_popcount(bits[0]) + __builtin_popcount(bits[1]);
        uint32_t x = mine;
#pragma unroll
        for (uint32_t d = 1; d < 64; d <<= 1) {
            const uint32_t y = __shfl_up(x, d);
            if (lane >= d) x += y;
        }
        if (lane == 63) wave_sum[r & 1][wave] = x;
        __syncthreads();  // the other half of wave_sum is rewritten only behind the next round's barrier
        uint32_t before = run;
#pragma unroll
        for (uint32_t v = 0; v < 4; ++v) {
            before += v < wave ? wave_sum[r & 1][v] : 0u;
            run += wave_sum[r & 1][v];
        }
        if (w < n_words) {
            if constexpr (BITS)
                reinterpret_cast<uint32_t *>(packed)[w] = before + x - mine;
            else
                reinterpret_cast<uint4 *>(packed)[w] = make_uint4(bits[0], bits[1], before + x - mine, 0u);
        }
    }
    if (t == 0) totals[blockIdx.x] = run;
}

// Places R records a thread: records i0, i0 + blockDim, ... of a segment of n.
template <bool BITS, uint32_t R>
__device__ inline void rank_place(const uint4 *seg, uint32_t i0, uint32_t n, uint32_t w_log2, uint32_t n_cells,
                                  const void *cells, const void *packed, const uint32_t *base, uint64_t limit,
                                  gss_report *out) {
    uint4 rec[R], p[R];  // p: (bits, bits, count)
    uint32_t cell[R], first[R];
    bool ok[R];
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
        const uint32_t i = i0 + r * blockDim.x;
        rec[r] = seg[i < n ? i : i0];
    }
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
        const uint64_t at = ((uint64_t)rec[r].x << w_log2) + rec[r].y;
        ok[r] = at < n_cells && i0 + r * blockDim.x < n;
        cell[r] = ok[r] ? (uint32_t)at : 0u;
        if constexpr (BITS) {
            const uint2 c = reinterpret_cast<const uint2 *>(cells)[cell[r] >> 6];
            p[r] = make_uint4(c.x, c.y, reinterpret_cast<const uint32_t *>(packed)[cell[r] >> 6], 0u);
        } else {
            p[r] = reinterpret_cast<const uint4 *>(packed)[cell[r] >> 6];
        }
        first[r] = base[cell[r] / kRankBlock];
    }
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
        const uint64_t below = (((uint64_t)p[r].y << 32) | p[r].x) & ((1ull << (cell[r] & 63)) - 1);
        const uint64_t pos = (uint64_t)first[r] + p[r].z + __builtin_popcountll(below);
        if (ok[r] && pos < limit) reinterpret_cast<uint4 *>(out)[pos] = rec[r];
    }
}

// Stores every kept record at its place; places at or beyond `limit` are left out.
// Bound by memory: the records' lines in and out (10.1 M records, 0.32 GB: 115 us, 2.8
// TB/s), reached through a chain of three loads.  A thread of a segment that gives all
// threads one has four records in flight: with one 126 us, two 120, eight 107, but 0.4 M
// records in short segments took 22 us with four and 27 with eight.  Non-temporal
// stores: 154.
template <bool BITS>
__global__ __launch_bounds__(256) void k_rank_place(const gss_report *reports, const uint32_t *counts, uint32_t seg_cap,
                                                    uint32_t n_segments, uint32_t w_log2, uint32_t n_cells,
                                                    const void *cells, const void *packed, const uint32_t *base,
                                                    uint64_t limit, gss_report *out) {
    for (uint32_t s = blockIdx.x; s < n_segments; s += gridDim.x) {
        const uint32_t n = min(counts[s], seg_cap);
        const uint4 *seg = reinterpret_cast<const uint4 *>(reports) + (uint64_t)s * seg_cap;
        uint32_t i = threadIdx.x;
        if (n > blockDim.x) {
            for (; i < n; i += 4 * blockDim.x)
                rank_place<BITS, 4>(seg, i, n, w_log2, n_cells, cells, packed, base, limit, out);
        } else if (i < n) {
            rank_place<BITS, 1>(seg, i, n, w_log2, n_cells, cells, packed, base, limit, out);
        }
    }
}

// The whole ranked order of a small result by one workgroup, its bit cells and counts
// in LDS: one launch instead of five, 40 us of a 90 us pass of 20 K clauses x 64 slots.
// 2^lanes_log2 lanes take a segment, about as many as it has records.
__global__ __launch_bounds__(1024) void k_rank_small(const gss_report *reports, const uint32_t *counts, uint32_t seg_cap,
                                                     uint32_t n_segments, uint32_t lanes_log2, uint32_t w_log2,
                                                     uint32_t n_cells, uint64_t limit, gss_report *out) {
    __shared__ uint2 marks[kSmallCells / 64];
    __shared__ uint32_t before[kSmallCells / 64];
    __shared__ uint32_t wave_sum[16];
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const uint32_t words = (n_cells + 63) / 64;
    for (uint32_t w = t; w < words; w += 1024) marks[w] = make_uint2(0, 0);
    __syncthreads();
    const uint32_t first = t & ((1u << lanes_log2) - 1), step = 1u << lanes_log2;
    for (uint32_t s = t >> lanes_log2; s < n_segments; s += 1024u >> lanes_log2) {
        const uint32_t n = min(counts[s], seg_cap);
        for (uint32_t i = first; i < n; i += step) {
            const gss_report &r = reports[(uint64_t)s * seg_cap + i];
            const uint64_t cell = ((uint64_t)r.clause_id << w_log2) + r.word;
            if (cell < n_cells) atomicOr(reinterpret_cast<uint32_t *>(marks) + (cell >> 5), 1u << (cell & 31));
        }
    }
    __syncthreads();
    // a thread counts kSmallCells / 64 / 1024 consecutive words
    constexpr uint32_t kPer = kSmallCells / 64 / 1024;
    uint32_t mine = 0;
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k) {
        const uint32_t w = t * kPer + k;
        if (w < words) {
            before[w] = mine;
            mine += __builtin_popcount(marks[w].x) + __builtin_popcount(marks[w].y);
        }
    }
    uint32_t x = mine;
#pragma unroll
    for (uint32_t d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d);
        if (lane >= d) x += y;
    }
    if (lane == 63) wave_sum[wave] = x;
    __syncthreads();
    uint32_t base = x - mine;
    for (uint32_t w = 0; w < wave; ++w) base += wave_sum[w];
#pragma unroll
    for (uint32_t k = 0; k < kPer; ++k)
        if (t * kPer + k < words) before[t * kPer + k] += base;
    __syncthreads();
    for (uint32_t s = t >> lanes_log2; s < n_segments; s += 1024u >> lanes_log2) {
        const uint32_t n = min(counts[s], seg_cap);
        for (uint32_t i = first; i < n; i += step) {
            const uint4 rec = reinterpret_cast<const uint4 *>(reports)[(uint64_t)s * seg_cap + i];
            const uint64_t cell = ((uint64_t)rec.x << w_log2) + rec.y;
            if (cell >= n_cells) continue;
            const uint2 m = marks[cell >> 6];
            const uint64_t below = (((uint64_t)m.y << 32) | m.x) & ((1ull << (cell & 63)) - 1);
            const uint64_t pos = before[cell >> 6] + __builtin_popcountll(below);
            if (pos < limit) reinterpret_cast<uint4 *>(out)[pos] = rec;
        }
    }
}

unsigned grid_of(uint64_t n) { return (unsigned)std::max<uint64_t>(1, std::min<uint64_t>((n + 255) / 256, 16384)); }

}  // namespace

void launch_scan_u32(Ctx &c, uint32_t *x, uint64_t m) {
    if (m == 0) return;
    hipLaunchKernelGGL(k_sort_scan, dim3(1), dim3(1024), 0, c.stream, x, m);
    GSS_HIP(hipGetLastError());
}

RankPlan rank_plan(const Ctx &c) {
    return RankPlan(c.id_loc.size(), c.W, c.RWc, c.n_kept, c.hits_valid, c.hits_ids);
}

template <bool BITS>
static void launch_rank(Ctx &c, const RankPlan &p, char *ws, gss_report *dst, uint64_t limit) {
    void *marks = p.hits ? c.hits : ws, *packed = ws + p.marks;
    uint32_t *totals = (uint32_t *)(ws + p.marks + p.packed);
    const dim3 grid(std::max<uint32_t>(1, std::min<uint32_t>(c.last_waves, 65535)));
    if (!p.hits) {
        launch_fill_u64(c, (uint64_t *)marks, p.marks / 8, 0);
        hipLaunchKernelGGL(k_rank_mark<BITS>, grid, dim3(256), 0, c.stream, c.reports, c.seg_counts, c.seg_cap,
                           c.last_waves, p.w_log2, (uint32_t)p.cells, marks);
        GSS_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(k_rank_pack<BITS>, dim3((unsigned)p.blocks), dim3(256), 0, c.stream, marks, (uint32_t)p.words,
                       packed, totals);
    GSS_HIP(hipGetLastError());
    launch_scan_u32(c, totals, p.blocks);
    hipLaunchKernelGGL(k_rank_place<BITS>, grid, dim3(256), 0, c.stream, c.reports, c.seg_counts, c.seg_cap, c.last_waves,
                       p.w_log2, (uint32_t)p.cells, marks, packed, totals, limit, dst);
    GSS_HIP(hipGetLastError());
}

// Queues the ranked order of the last test's kept records, the first `limit` of it,
// into dst (device); ws: `bytes` of device memory, 256-byte aligned, that the plan fits in.
void rank_records(Ctx &c, char *ws, uint64_t bytes, gss_report *dst, uint64_t limit) {
    const RankPlan p = rank_plan(c);
    GSS_REQUIRE(p.fits_in(ws ? bytes : 0), GSS_ERR_DEVICE, "the ranked order does not fit its workspace");
    if (p.small) {
        uint32_t lanes_log2 = 0;
        while (lanes_log2 < 6 && ((uint64_t)c.last_waves << lanes_log2) < c.n_kept) ++lanes_log2;
        hipLaunchKernelGGL(k_rank_small, dim3(1), dim3(1024), 0, c.stream, c.reports, c.seg_counts, c.seg_cap, c.last_waves,
                           lanes_log2, p.w_log2, (uint32_t)p.cells, limit, dst);
        GSS_HIP(hipGetLastError());
    } else if (p.bits)
        launch_rank<true>(c, p, ws, dst, limit);
    else
        launch_rank<false>(c, p, ws, dst, limit);
}

void sort_records(Ctx &c, gss_report *src, uint64_t n, gss_report *dst) {
    if (n == 0) return;
    GSS_REQUIRE(n < (1ull << 32) - kSortTile, GSS_ERR_CAPACITY, "too many records to sort");
    uint32_t word_bits = 1;
    while ((1u << word_bits) < c.W) ++word_bits;
    const uint32_t n_passes = (32 + word_bits + 7) / 8;
    const uint32_t n_tiles = (uint32_t)((n + kSortTile - 1) / kSortTile);
    const uint64_t hist_n = (uint64_t)kRadix * n_tiles;
    const size_t counts_bytes = kMaxPasses * kRadix * sizeof(unsigned long long);
    const uint32_t chunks = (uint32_t)((hist_n + kScanChunk - 1) / kScanChunk);
    char *buf = (char *)c.dalloc(counts_bytes + (hist_n + chunks) * 4);
    unsigned long long *counts = (unsigned long long *)buf;
    uint32_t *hist = (uint32_t *)(buf + counts_bytes);
    try {
        launch_fill_u64(c, (uint64_t *)counts, kMaxPasses * kRadix, 0);
        hipLaunchKernelGGL(k_sort_digits, dim3(std::min<unsigned>(grid_of(n), 1024)), dim3(kSortThreads), 0, c.stream,
                           src, n, word_bits, n_passes, counts);
        GSS_HIP(hipGetLastError());
        std::vector<unsigned long long> h(kMaxPasses * kRadix);
        GSS_HIP(hipMemcpyAsync(h.data(), counts, counts_bytes, hipMemcpyDeviceToHost, c.stream));
        c.sync();
        // every non-trivial digit, least significant first; src and dst take turns
        gss_report *from = src, *to = dst;
        for (uint32_t p = 0; p < n_passes; ++p) {
            if (*std::max_element(h.begin() + p * kRadix, h.begin() + (p + 1) * kRadix) == n) continue;
            const uint32_t shift = 8 * p;
            hipLaunchKernelGGL(k_sort_tile_counts, dim3(n_tiles), dim3(kSortThreads), 0, c.stream, from, n, word_bits,
                               shift, hist, n_tiles);
            GSS_HIP(hipGetLastError());
            if (chunks <= 2) {  // up to 32 tiles: one launch
                launch_scan_u32(c, hist, hist_n);
            } else {
                uint32_t *sums = hist + hist_n;
                hipLaunchKernelGGL(k_scan_sums, dim3(chunks), dim3(256), 0, c.stream, hist, hist_n, sums);
                GSS_HIP(hipGetLastError());
                launch_scan_u32(c, sums, chunks);
                hipLaunchKernelGGL(k_scan_apply, dim3(chunks), dim3(256), 0, c.stream, hist, hist_n, sums);
                GSS_HIP(hipGetLastError());
            }
            hipLaunchKernelGGL(k_sort_scatter, dim3(n_tiles), dim3(kSortThreads), 0, c.stream, from, to, n, word_bits,
                               shift, hist, n_tiles);
            GSS_HIP(hipGetLastError());
            std::swap(from, to);
        }
        if (from != dst)
            GSS_HIP(hipMemcpyAsync(dst, from, n * sizeof(gss_report), hipMemcpyDeviceToDevice, c.stream));
        c.sync();
    } catch (...) {
        (void)hipStreamSynchronize(c.stream);
        c.dfree(buf);
        throw;
    }
    c.dfree(buf);
}

}  // namespace gss

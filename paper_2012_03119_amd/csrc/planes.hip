// Assignment bitplanes (Section 3.4): N assignments of a variable as two N-bit
// words.  The paper keeps (isTrue, isSet); this library keeps, per literal code,
// the word of slots where that literal is F:
//   row 2v   = slots where v = F   (isSet & ~isTrue)
//   row 2v+1 = slots where v = T   (isSet &  isTrue)
// so a clause's falsified mask is the AND of one gathered row per literal, and
// the Undef slots of v are the complement of (row 2v | row 2v+1).  The value of
// the isTrue bit for an Undef slot, which the paper leaves open, never enters.
//
// One 64-bit word holds 64 slots, one per lane of a wavefront.
#include "gss_internal.h"

#include <algorithm>
#include <cstring>

namespace gss {

// ---- aggregate bits (Section 4): per row and chunk, bit w = some slot of word
//      w of the chunk has the row's literal F (element g * n_rows + row).  Packed
//      word deltas keep them in step; bulk updates (full sets, large var-major deltas,
//      cleared slots) mark them stale, and the next aggregate test rebuilds them.
//      Above them, with more than one chunk, one bit per row and chunk (the
//      super-group: the aggregate of the chunk's word aggregates), rebuilt from
//      the word bits before an aggregate test when they changed.  Var-major deltas
//      recompute the listed variables' bits once a test has used them.

__device__ inline uint64_t agg_get(const void *agg, uint32_t RWc, uint64_t i) {
    if (RWc <= 16) return reinterpret_cast<const uint16_t *>(agg)[i];
    if (RWc <= 32) return reinterpret_cast<const uint32_t *>(agg)[i];
    return reinterpret_cast<const uint64_t *>(agg)[i];
}

__device__ inline void agg_put(void *agg, uint32_t RWc, uint64_t i, uint64_t bits) {
    if (RWc <= 16)
        reinterpret_cast<uint16_t *>(agg)[i] = (uint16_t)bits;
    else if (RWc <= 32)
        reinterpret_cast<uint32_t *>(agg)[i] = (uint32_t)bits;
    else
        reinterpret_cast<uint64_t *>(agg)[i] = bits;
}

// The elements of rows 2 v and 2 v + 1, one after the other, in one store.
__device__ inline void agg_put2(void *agg, uint32_t RWc, uint64_t i, uint64_t b0, uint64_t b1) {
    if (RWc <= 16)
        *reinterpret_cast<uint32_t *>(reinterpret_cast<uint16_t *>(agg) + i) = (uint32_t)b0 | ((uint32_t)b1 << 16);
    else if (RWc <= 32)
        *reinterpret_cast<uint2 *>(reinterpret_cast<uint32_t *>(agg) + i) = make_uint2((uint32_t)b0, (uint32_t)b1);
    else
        *reinterpret_cast<ulonglong2 *>(reinterpret_cast<uint64_t *>(agg) + i) = make_ulonglong2(b0, b1);
}

// The aggregates of one chunk of a variable's row pair, a lane per word (RWc lanes a
// variable): bit w of the results is the ballot of word w.
struct AggWords {
    uint64_t f, t, u;  // words with an F slot, with a T slot, with an active U slot
};

__device__ inline AggWords agg_words(uint64_t f, uint64_t t, uint64_t act, uint32_t RWc, uint32_t lane) {
    const uint32_t at = lane / RWc * RWc;
    const uint64_t m = RWc == 64 ? ~0ull : (1ull << RWc) - 1;
    return AggWords{(__ballot(f != 0) >> at) & m, (__ballot(t != 0) >> at) & m,
                    (__ballot(((f | t) & act) != act) >> at) & m};
}

// Aggregates of every variable below n_vars, [G][2 n_vars] and (aggu != null) their U
// bits [G][n_vars], in one pass over the planes.  A wavefront takes 64 / RWc variables
// a step, a lane a word of both rows, kAggSteps steps in flight.  Bound by the planes'
// reads: 25 K variables x 256 words (102 MB) in 18 us and 1 M x 16 words
// (256 MB) in 38 us with the U bits (a thread a row, its words strided over the lanes:
// 60 and 490 us for the U bits alone, the rows' own as much again).
constexpr uint32_t kAggSteps = 8;

__global__ __launch_bounds__(256) void k_agg_rows(const uint64_t *planes, uint32_t RWc, uint64_t chunk, uint64_t n_rows,
                                                  const uint64_t *active, uint32_t W, void *agg, void *aggu,
                                                  uint64_t n_vars) {
    const uint32_t lane = threadIdx.x & 63, g = blockIdx.y, per = 64 / RWc, w = lane % RWc;
    const uint64_t act = g * RWc + w < W ? active[g * RWc + w] : 0ull;
    const uint64_t v0 = ((uint64_t)blockIdx.x * 4 + threadIdx.x / 64) * kAggSteps * per + lane / RWc;
    uint64_t f[kAggSteps], t[kAggSteps];
#pragma unroll
    for (uint32_t k = 0; k < kAggSteps; ++k) {  // past the end: the last variable, not stored
        const uint64_t *p = planes + g * chunk + 2 * min(v0 + k * per, n_vars - 1) * RWc + w;
        f[k] = p[0];
        t[k] = p[RWc];
    }
#pragma unroll
    for (uint32_t k = 0; k < kAggSteps; ++k) {
        const uint64_t v = v0 + k * per;
        const AggWords a = agg_words(f[k], t[k], act, RWc, lane);
        if (w == 0 && v < n_vars) {
            agg_put2(agg, RWc, g * n_rows + 2 * v, a.f, a.t);
            if (aggu) agg_put(aggu, RWc, g * n_vars + v, a.u);
        }
    }
}

// The same for the listed variables only, after a delta, with their super-group bits
// (G > 1): the aggregates stay valid at the cost of the delta's rows.
__global__ __launch_bounds__(256) void k_agg_vars(const uint64_t *planes, uint32_t RWc, uint64_t chunk, uint32_t G,
                                                  uint64_t n_rows, const uint64_t *active, uint32_t W, void *agg,
                                                  void *aggu, uint64_t *sagg, uint64_t *saggu, const uint32_t *vars,
                                                  uint32_t n, const uint32_t *perm) {
    const uint32_t lane = threadIdx.x & 63, per = 64 / RWc, w = lane % RWc;
    const uint64_t i = ((uint64_t)blockIdx.x * 4 + threadIdx.x / 64) * per + lane / RWc;
    const uint64_t v = internal_var(perm, vars[min(i, (uint64_t)n - 1)]);
    const bool writes = w == 0 && i < n;
    uint64_t sf = 0, st = 0, su = 0;
    for (uint32_t g = 0; g < G; ++g) {
        const uint64_t act = g * RWc + w < W ? active[g * RWc + w] : 0ull;
        const uint64_t *p = planes + g * chunk + 2 * v * RWc + w;
        const AggWords a = agg_words(p[0], p[RWc], act, RWc, lane);
        sf |= (uint64_t)(a.f != 0) << g;
        st |= (uint64_t)(a.t != 0) << g;
        su |= (uint64_t)(a.u != 0) << g;
        if (writes) {
            agg_put2(agg, RWc, g * n_rows + 2 * v, a.f, a.t);
            if (aggu) agg_put(aggu, RWc, g * (n_rows / 2) + v, a.u);
        }
    }
    if (writes && sagg) *reinterpret_cast<ulonglong2 *>(sagg + 2 * v) = make_ulonglong2(sf, st);
    if (writes && saggu) saggu[v] = su;
}

// Super-group bits (G > 1): bit g of out[i] = the 64-word aggregate in[g][i] is nonzero.
__global__ void k_super_bits(const uint64_t *in, uint32_t G, uint64_t n, uint64_t *out) {
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
        uint64_t bits = 0;
        for (uint32_t g = 0; g < G; ++g) bits |= (uint64_t)(in[g * n + i] != 0) << g;
        out[i] = bits;
    }
}

static void launch_agg_rows(Ctx &c, bool with_u, uint64_t n_vars) {
    const uint64_t per_block = 4ull * kAggSteps * (64 / c.RWc);
    hipLaunchKernelGGL(k_agg_rows, dim3((unsigned)((n_vars + per_block - 1) / per_block), c.G), dim3(256), 0, c.stream,
                       c.planes, c.RWc, c.chunk_elems, c.n_rows, c.active, c.W, c.agg, with_u ? c.aggu : nullptr, n_vars);
    GSS_HIP(hipGetLastError());
}

void agg_init(Ctx &c) { launch_agg_rows(c, false, 1); }

// Recomputes what is stale of the aggregates, the U bits with them when wanted.
bool agg_refresh(Ctx &c, bool with_u) {
    c.agg_used = true;
    const uint64_t n = (uint64_t)c.cfg.num_vars + 1;
    bool moved = false;
    if (with_u && !c.aggu) {
        c.aggu = c.dalloc((uint64_t)c.G * n * agg_elem_bytes(c.RWc));
        moved = true;
    }
    if (c.agg_valid && (!with_u || c.aggu_valid)) return moved;
    launch_agg_rows(c, with_u, n);
    if (!c.agg_valid) c.sagg_valid = false;
    c.agg_valid = true;
    if (with_u) {
        c.aggu_valid = true;
        c.saggu_valid = false;
    } else {
        c.aggu_valid = false;
    }
    return moved;
}

// After a delta of n listed variables (device list): keeps valid aggregates valid when
// the context uses them, at the cost of the listed rows; a delta of more than half the
// variables, or aggregates that no test has asked for, are left to the next refresh.
static void agg_after_delta(Ctx &c, const uint32_t *d_vars, uint32_t n) {
    if (!c.agg_used || !c.agg_valid || n > c.cfg.num_vars / 2) {
        c.agg_valid = false;
        c.aggu_valid = false;
        return;
    }
    const bool with_u = c.aggu_valid, super = c.G > 1 && c.sagg_valid, super_u = with_u && c.G > 1 && c.saggu_valid;
    const uint32_t per_block = 4 * (64 / c.RWc);
    hipLaunchKernelGGL(k_agg_vars, dim3((n + per_block - 1) / per_block), dim3(256), 0, c.stream, c.planes, c.RWc,
                       c.chunk_elems, c.G, c.n_rows, c.active, c.W, c.agg, with_u ? c.aggu : nullptr,
                       super ? c.sagg : nullptr, super_u ? c.saggu : nullptr, d_vars, n, c.d_perm);
    GSS_HIP(hipGetLastError());
}

void super_rebuild(Ctx &c, bool with_u) {
    if (c.G == 1) return;
    if (!c.sagg_valid) {
        hipLaunchKernelGGL(k_super_bits, dim3(fill_grid(c.n_rows)), dim3(256), 0, c.stream,
                           (const uint64_t *)c.agg, c.G, c.n_rows, c.sagg);
        GSS_HIP(hipGetLastError());
        c.sagg_valid = true;
    }
    if (with_u && !c.saggu_valid) {
        const uint64_t n = (uint64_t)c.cfg.num_vars + 1;
        if (!c.saggu) c.saggu = (uint64_t *)c.dalloc(n * 8);
        hipLaunchKernelGGL(k_super_bits, dim3(fill_grid(n)), dim3(256), 0, c.stream, (const uint64_t *)c.aggu, c.G, n,
                           c.saggu);
        GSS_HIP(hipGetLastError());
        c.saggu_valid = true;
    }
}

// Packs slot-major values into plane words.  A wavefront takes one 64-slot word of 256
// variables, a lane four of them: each slot's row is read as one run of 256 bytes (at
// any alignment), and a dword's four sign bits and four "T" bits are shifted into four
// byte-wide accumulators, so that a value costs about a fortieth of an instruction
// (a ballot per variable and truth value, with the lanes on the slots, took 10
// instructions per variable and read 64-byte runs).  The up to 16 wavefronts of a
// workgroup take consecutive words of the same variables and, from four words on,
// turn them in LDS so that the rows are written as runs (stored 8 bytes a lane, the
// same kernel took 133 us on the figure below).
//
// vals: row r holds slot first + r, `pitch` bytes a row, byte v - 1 = variable v; words
// w_first .. w_first + nw - 1; a word only partly inside [first, first + n_slots) keeps
// its other slots.  Bound by the reads and writes: 1024 slots x
// 250 K variables (256 MB in, 64 MB out) in 64 us, 5.0 TB/s, where sixteen launches
// with a staging copy before each took 390 us.
constexpr uint32_t kPackWords = 16;

constexpr uint32_t kTurnWords = 4;  // words of a workgroup from which its rows are turned in LDS

typedef uint32_t u32_any __attribute__((aligned(1)));

// LDS entry of word `word` of row r (of 512, two a variable), `p` a power of two of
// words a row: the words of every eighth row, which one store of a wavefront writes,
// are spread over the banks.
__device__ inline uint32_t turn_index(uint32_t r, uint32_t word, uint32_t p) {
    return r * p + (word ^ ((r >> 3) & (p - 1)));
}

__host__ __device__ inline uint32_t turn_words(uint32_t wb) { return wb <= 4 ? 4 : wb <= 8 ? 8 : 16; }

// The workgroup's rows out of LDS, 16 lanes a row: words w0 .. w0 + wb - 1 of both rows
// of the variables from `tile` on (from 0).
__device__ inline void store_turned(const uint64_t *turn, uint64_t *planes, uint32_t RWc, uint64_t chunk,
                                    uint32_t num_vars, uint64_t tile, uint32_t w0, uint32_t wb, const uint32_t *perm) {
    const uint32_t word = threadIdx.x % kPackWords;
    for (uint32_t r = threadIdx.x / kPackWords; r < 512; r += blockDim.x / kPackWords) {
        const uint64_t v = tile + r / 2;
        if (v < num_vars && word < wb)
            planes[plane_index(2ull * internal_var(perm, (uint32_t)v + 1) + (r & 1), w0 + word, RWc, chunk)] =
                turn[turn_index(r, word, turn_words(wb))];
    }
}

__global__ __launch_bounds__(64 * kPackWords) void k_pack_rows(uint64_t *planes, uint32_t RWc, uint64_t chunk,
                                                               uint32_t num_vars, const int8_t *vals, uint64_t pitch,
                                                               uint32_t first, uint32_t n_slots, uint32_t w_first,
                                                               uint32_t nw, const uint32_t *bad,
                                                               const uint32_t *perm) {
    extern __shared__ uint64_t turn[];  // [512 rows of 256 variables][turn_words], see turn_index
    if (*bad) return;                   // the inputs failed validation: apply nothing
    const uint32_t wb = min(kPackWords, nw - blockIdx.y * kPackWords);  // words of this workgroup
    const uint32_t wave = threadIdx.x / 64, lane = threadIdx.x & 63;
    const uint64_t tile = 256ull * blockIdx.x, v0 = tile + 4 * lane;  // the lane's first variable, from 0
    const bool turns = wb >= kTurnWords;
    const uint32_t w = w_first + blockIdx.y * kPackWords + min(wave, wb - 1);
    const uint32_t lo = max(first, 64 * w), hi = min(first + n_slots, 64 * w + 64);
    const int8_t *src = vals + (uint64_t)(lo - first) * pitch + v0;
    // variables of this lane; none in a wavefront or lane past the end, which waits at the barrier below
    const uint32_t mine = wave < wb && v0 < num_vars ? (uint32_t)min((uint64_t)4, num_vars - v0) : 0u;
    uint64_t f[4] = {0, 0, 0, 0}, t[4] = {0, 0, 0, 0};
    // F = 0xFF has its sign bit set; T = 0x01 its lowest bit and not the sign bit
    auto f_bits = [](uint32_t d) { return (d >> 7) & 0x01010101u; };
    auto t_bits = [](uint32_t d) { return d & ~(d >> 7) & 0x01010101u; };
    if (hi - lo == 64 && mine == 4) {
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {  // 16 slots' rows in flight together
            uint32_t d[16];
#pragma unroll
            for (uint32_t s = 0; s < 16; ++s) d[s] = *reinterpret_cast<const u32_any *>(src + (16 * q + s) * pitch);
#pragma unroll
            for (uint32_t h = 0; h < 2; ++h) {  // 8 slots: byte k collects variable k's bits
                uint32_t fa = 0, ta = 0;
#pragma unroll
                for (uint32_t s = 8; s-- > 0;) {
                    fa = (fa << 1) | f_bits(d[8 * h + s]);
                    ta = (ta << 1) | t_bits(d[8 * h + s]);
                }
#pragma unroll
                for (uint32_t k = 0; k < 4; ++k) {
                    f[k] |= (uint64_t)((fa >> (8 * k)) & 0xFFu) << (16 * q + 8 * h);
                    t[k] |= (uint64_t)((ta >> (8 * k)) & 0xFFu) << (16 * q + 8 * h);
                }
            }
        }
    } else if (mine) {
        for (uint32_t s = lo; s < hi; ++s, src += pitch)
#pragma unroll
            for (uint32_t k = 0; k < 4; ++k) {
                const int8_t x = k < mine ? src[k] : 0;
                f[k] |= (uint64_t)(x == -1) << (s - 64 * w);
                t[k] |= (uint64_t)(x == 1) << (s - 64 * w);
            }
    }
    const uint64_t keep = hi - lo == 64 ? 0 : ~(((1ull << (hi - lo)) - 1) << (lo - 64 * w));
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
        if (k >= mine) break;
        const uint64_t r0 = plane_index(2ull * internal_var(perm, (uint32_t)v0 + k + 1), w, RWc, chunk), r1 = r0 + RWc;
        if (keep) {
            f[k] |= planes[r0] & keep;
            t[k] |= planes[r1] & keep;
        }
        if (turns) {
            turn[turn_index(2 * (4 * lane + k), wave, turn_words(wb))] = f[k];
            turn[turn_index(2 * (4 * lane + k) + 1, wave, turn_words(wb))] = t[k];
        } else {
            planes[r0] = f[k];
            planes[r1] = t[k];
        }
    }
    if (turns) {  // uniform over the workgroup
        __syncthreads();
        store_turned(turn, planes, RWc, chunk, num_vars, tile, w_first + blockIdx.y * kPackWords, wb, perm);
    }
}

// Delta update: thread per (variable, 64-slot word), the words of one variable
// on neighbouring lanes, so that a variable's plane rows are written as whole
// lines and its values read as one contiguous run.  The thread reads the word's
// 64 values of its variable (four 16-byte loads when the word is whole and
// aligned) and builds the F and T words; a word only partly inside
// [first, first + n_slots) keeps its other slots.  vals is var-major
// [n_vars][n_slots]; nw = words touched.
// With clear_bits != null, the thread of each variable's first word also clears
// the variable's word of the duplicate bitmap (left zero for the next check).
__global__ __launch_bounds__(256) void k_set_vars(uint64_t *planes, uint32_t RWc, uint64_t chunk, const uint32_t *vars,
                                                  uint32_t n_vars,
                                                  const int8_t *vals, uint32_t first, uint32_t n_slots, uint32_t nw,
                                                  const uint32_t *bad, uint32_t *clear_bits, const uint32_t *perm) {
    const uint64_t x = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    if (x >= (uint64_t)n_vars * nw) return;
    const uint32_t i = (uint32_t)(x / nw);
    const uint32_t wi = (uint32_t)(x - (uint64_t)i * nw);
    if (clear_bits && wi == 0) clear_bits[vars[i] >> 5] = 0;
    if (*bad) return;  // the inputs failed validation: apply nothing
    const uint32_t w = first / 64 + wi;
    const uint32_t lo = max(first, 64 * w), hi = min(first + n_slots, 64 * w + 64);
    const int8_t *src = vals + (uint64_t)i * n_slots + (lo - first);
    uint64_t f = 0, t = 0;
    if (hi - lo == 64 && (reinterpret_cast<uintptr_t>(src) & 15) == 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint4 v = reinterpret_cast<const uint4 *>(src)[q];
            const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const uint32_t b = (u[k >> 2] >> (8 * (k & 3))) & 0xFFu;
                f |= (uint64_t)(b == 0xFFu) << (16 * q + k);
                t |= (uint64_t)(b == 0x01u) << (16 * q + k);
            }
        }
    } else {
        for (uint32_t s = lo; s < hi; ++s) {
            const int8_t x = src[s - lo];
            f |= (uint64_t)(x == -1) << (s - 64 * w);
            t |= (uint64_t)(x == 1) << (s - 64 * w);
        }
    }
    const uint64_t r0 = plane_index(2ull * internal_var(perm, vars[i]), w, RWc, chunk), r1 = r0 + RWc;
    if (hi - lo != 64) {
        const uint64_t sm = ((1ull << (hi - lo)) - 1) << (lo - 64 * w);  // hi - lo < 64 here
        f = (planes[r0] & ~sm) | (f & sm);
        t = (planes[r1] & ~sm) | (t & sm);
    }
    planes[r0] = f;
    planes[r1] = t;
}

// Packed delta: new plane words of listed variables in one 64-slot word.  Thread
// per variable; f = slots where the variable is F, t = slots where it is T.
// The variables of one launch are distinct, so each thread owns its two rows'
// aggregate bits (bit `word` of the word's chunk), updated in place, and, with aggu
// != null, its variable's U bit.
__global__ void k_set_words(uint64_t *planes, uint32_t RWc, uint64_t chunk, uint64_t n_rows, uint32_t word,
                            const uint32_t *vars, const uint64_t *f, const uint64_t *t, uint32_t n, void *agg,
                            void *aggu, const uint64_t *active, const uint32_t *perm) {
    const uint64_t act = aggu ? active[word] : 0ull;
    const uint64_t a_base = (uint64_t)(word / kChunkWords) * n_rows;
    const uint64_t bit = 1ull << (word % kChunkWords);
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const uint64_t row = 2ull * internal_var(perm, vars[i]);
        const uint64_t r0 = plane_index(row, word, RWc, chunk);
        planes[r0] = f[i];
        planes[r0 + RWc] = t[i];
        const uint64_t a0 = agg_get(agg, RWc, a_base + row), a1 = agg_get(agg, RWc, a_base + row + 1);
        agg_put(agg, RWc, a_base + row, f[i] ? (a0 | bit) : (a0 & ~bit));
        agg_put(agg, RWc, a_base + row + 1, t[i] ? (a1 | bit) : (a1 & ~bit));
        if (aggu) {
            const uint64_t u0 = agg_get(aggu, RWc, (a_base + row) / 2);
            agg_put(aggu, RWc, (a_base + row) / 2, ((f[i] | t[i]) & act) != act ? (u0 | bit) : (u0 & ~bit));
        }
    }
}

// Clears slots [first, first+n) in every row of real variables (rows >= 2).
__global__ void k_clear_slots(uint64_t *planes, uint32_t RWc, uint64_t chunk, uint64_t n_rows, uint32_t first,
                              uint32_t n_slots) {
    const uint32_t w_lo = first / 64, w_hi = (first + n_slots - 1) / 64, nw = w_hi - w_lo + 1;
    const uint64_t total = (n_rows - 2) * nw;
    for (uint64_t x = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; x < total; x += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t row = 2 + x / nw;
        const uint32_t w = w_lo + (uint32_t)(x % nw);
        const uint32_t a = std::max(first, 64 * w), b = std::min(first + n_slots, 64 * w + 64);
        const uint64_t sm = (b - a == 64) ? ~0ull : (((1ull << (b - a)) - 1) << (a - 64 * w));
        planes[plane_index(row, w, RWc, chunk)] &= ~sm;
    }
}

void launch_set_words(Ctx &c, uint32_t word, const uint32_t *vars, const uint64_t *f, const uint64_t *t, uint32_t n) {
    if (n == 0) return;
    c.sagg_valid = false;
    c.saggu_valid = false;
    const unsigned grid = std::max<uint32_t>(1, std::min<uint32_t>((n + 255) / 256, 4096));
    hipLaunchKernelGGL(k_set_words, dim3(grid), dim3(256), 0, c.stream, c.planes, c.RWc, c.chunk_elems, c.n_rows, word,
                       vars, f, t, n, c.agg, c.aggu_valid ? c.aggu : nullptr, c.active, c.d_perm);
    GSS_HIP(hipGetLastError());
    c.mutations++;
}

static uint64_t slot_mask(uint32_t first, uint32_t n, uint32_t w) {
    const uint32_t a = std::max(first, 64 * w), b = std::min(first + n, 64 * w + 64);
    if (b <= a) return 0;
    return (b - a == 64) ? ~0ull : (((1ull << (b - a)) - 1) << (a - 64 * w));
}

__global__ void k_copy_words(const uint64_t *src, uint64_t *dst, uint32_t n) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

// The active words go up by a kernel reading the pinned ring slot: a queued DMA
// copy would start only after the test before it and then hold up the next one.
static void upload_active(Ctx &c) {
    c.aggu_valid = false;  // U counts active slots only
    const Ctx::Staged st = c.stage_upload(c.W * 8);
    std::memcpy(st.h, c.h_active.data(), c.W * 8);
    hipLaunchKernelGGL(k_copy_words, dim3((c.W + 255) / 256), dim3(256), 0, c.stream, (const uint64_t *)st.hd, c.active,
                       c.W);
    GSS_HIP(hipGetLastError());
    c.stage_done(st);
}

// Range and distinctness of a variable list: an increasing one (as a solver's trail
// sorted, or a run of variables) by its neighbours, any other in O(n) with a bitmap
// that is cleared again afterwards.
static void check_vars(Ctx &c, const uint32_t *vars, uint32_t n_vars) {
    uint32_t unordered = vars[0] < 1 || vars[n_vars - 1] > c.cfg.num_vars;
    for (uint32_t i = 1; i < n_vars; ++i) unordered |= vars[i] <= vars[i - 1];
    if (!unordered) return;
    std::vector<uint64_t> &seen = c.var_seen;
    if (seen.size() < (uint64_t)c.cfg.num_vars / 64 + 1) seen.assign((uint64_t)c.cfg.num_vars / 64 + 1, 0);
    uint32_t bad = 0;  // 1: out of range, 2: repeated
    uint32_t i = 0;
    for (; i < n_vars; ++i) {
        const uint32_t v = vars[i];
        if (v < 1 || v > c.cfg.num_vars) { bad = 1; break; }
        uint64_t &word = seen[v >> 6];
        const uint64_t bit = 1ull << (v & 63);
        if (word & bit) { bad = 2; break; }
        word |= bit;
    }
    for (uint32_t k = 0; k < i; ++k) seen[vars[k] >> 6] = 0;
    GSS_REQUIRE(bad != 1, GSS_ERR_BAD_LITERAL, "variable out of range");
    GSS_REQUIRE(bad != 2, GSS_ERR_INVALID_ARG, "variable listed twice");
}

// Every listed variable in 1..num_vars (the cheap half of check_vars).
static void check_var_range(const Ctx &c, const uint32_t *vars, uint32_t n_vars) {
    uint32_t bad = 0;
    const uint32_t V = c.cfg.num_vars;
    for (uint32_t i = 0; i < n_vars; ++i) bad |= (uint32_t)(vars[i] - 1u >= V);
    GSS_REQUIRE(!bad, GSS_ERR_BAD_LITERAL, "variable out of range");
}

// Device half of the variable check: a variable listed twice sets bit 2 of
// *bad (one bitmap bit per variable, cleared again by k_set_vars).
__global__ void k_check_vars(const uint32_t *vars, uint32_t n, uint32_t *bits, uint32_t *bad) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t v = vars[i], m = 1u << (v & 31);
    if (atomicOr(&bits[v >> 5], m) & m) atomicOr(bad, 2u);
}

// Both checks of a queued delta in one launch: the first var_blocks workgroups
// take the variable list, marking repeats (bit 2 of *bad); the others check the truth
// values (bit 1).  The list is already on the device, or (list != null) read here
// from pinned host memory and stored to vars.
__global__ __launch_bounds__(256) void k_check_delta(const int8_t *vals, uint64_t n_vals, uint32_t var_blocks,
                                                     const uint32_t *list, uint32_t *vars, uint32_t n, uint32_t *bits,
                                                     uint32_t *bad) {
    if (blockIdx.x >= var_blocks) {
        const uint32_t b = blockIdx.x - var_blocks, value_blocks = gridDim.x - var_blocks;
        if (values_invalid(vals, n_vals, b * (uint64_t)blockDim.x + threadIdx.x, (uint64_t)value_blocks * blockDim.x))
            atomicOr(bad, 1u);
        return;
    }
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t v = list ? list[i] : vars[i], m = 1u << (v & 31);
    if (list) vars[i] = v;
    if (atomicOr(&bits[v >> 5], m) & m) atomicOr(bad, 2u);
}


static void launch_set_vars(Ctx &c, const uint32_t *d_vars, uint32_t n_vars, const int8_t *d_vals, uint32_t first_slot,
                            uint32_t n_slots, const uint32_t *bad, uint32_t *clear_bits) {
    const uint32_t nw = (first_slot + n_slots - 1) / 64 - first_slot / 64 + 1;
    const uint64_t threads = (uint64_t)n_vars * nw;
    hipLaunchKernelGGL(k_set_vars, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, c.stream, c.planes, c.RWc,
                       c.chunk_elems, d_vars, n_vars, d_vals, first_slot, n_slots, nw, bad, clear_bits, c.d_perm);
    GSS_HIP(hipGetLastError());
}

// Checks shared by both forms of gss_set_var_values: the slot range and its activity.
static void check_delta_slots(const Ctx &c, uint32_t first_slot, uint32_t n_slots) {
    GSS_REQUIRE((uint64_t)first_slot + n_slots <= c.cfg.max_slots, GSS_ERR_CAPACITY, "slot range beyond max_slots");
    for (uint32_t w = first_slot / 64; w <= (first_slot + n_slots - 1) / 64; ++w) {
        const uint64_t sm = slot_mask(first_slot, n_slots, w);
        GSS_REQUIRE((c.h_active[w] & sm) == sm, GSS_ERR_INVALID_ARG, "slot range includes inactive slots");
    }
}

// Uploads up to these sizes are read by their kernels from the pinned ring slot, with
// no copy queued before them: a variable list of a queued delta; a host delta's list
// and values, or a packed delta, each byte read once (a kernel reads pinned memory at
// 44 GB/s, as fast as a copy).
constexpr size_t kDirectList = 64u << 10, kDirectDelta = 1u << 20;

static void check_values_host(const int8_t *v, uint64_t n) {
    uint8_t bad = 0;
    for (uint64_t i = 0; i < n; ++i) bad |= (uint8_t)((uint8_t)(v[i] + 1) > 2);
    GSS_REQUIRE(!bad, GSS_ERR_INVALID_ARG, "truth values must be -1, 0 or +1");
}

}  // namespace gss

using namespace gss;

extern "C" gss_status gss_set_assignments(gss_ctx *ctx, uint32_t first_slot, uint32_t n_slots, const int8_t *values) {
    GSS_API_BEGIN(ctx)
    c_->mutations++;  // a test in flight no longer sees the current state
    Ctx &c = *c_;
    if (n_slots == 0) return GSS_OK;
    GSS_REQUIRE(values != nullptr, GSS_ERR_INVALID_ARG, "null argument");
    GSS_REQUIRE((uint64_t)first_slot + n_slots <= c.cfg.max_slots, GSS_ERR_CAPACITY, "slot range beyond max_slots");
    const uint64_t V = c.cfg.num_vars;
    const bool dev = is_device_pointer(values);
    const uint32_t *bad = c.dsmall + 1;  // always zero
    if (dev)
        bad = queue_value_check(c, values, (uint64_t)n_slots * V);
    else
        check_values_host(values, (uint64_t)n_slots * V);

    const uint32_t last = first_slot + n_slots, w_lo = first_slot / 64, w_hi = (last - 1) / 64;
    auto pack = [&](const int8_t *vals, uint32_t first, uint32_t n, uint32_t w, uint32_t nw) {
        const uint32_t waves = std::min(nw, kPackWords);
        hipLaunchKernelGGL(k_pack_rows, dim3((unsigned)((V + 255) / 256), (nw + kPackWords - 1) / kPackWords),
                           dim3(64 * waves), waves >= kTurnWords ? 512 * turn_words(waves) * 8 : 0, c.stream, c.planes, c.RWc,
                           c.chunk_elems, (uint32_t)V, vals, V, first, n, w, nw, bad, c.d_perm);
        GSS_HIP(hipGetLastError());
    };
    if (dev) {
        pack(values, first_slot, n_slots, w_lo, w_hi - w_lo + 1);
    } else {  // host values go up a word's slots at a time
        int8_t *stage = (int8_t *)c.device_stage(64 * V);
        for (uint32_t w = w_lo; w <= w_hi; ++w) {
            const uint32_t s_lo = std::max(first_slot, 64 * w), s_hi = std::min(last, 64 * w + 64);
            GSS_HIP(hipMemcpyAsync(stage, values + (uint64_t)(s_lo - first_slot) * V, (uint64_t)(s_hi - s_lo) * V,
                                   hipMemcpyHostToDevice, c.stream));
            pack(stage, s_lo, s_hi - s_lo, w, 1);
        }
    }
    if (dev) check_flag(c);  // throws, having applied nothing, if a value was invalid
    c.agg_valid = false;
    c.aggu_valid = false;
    for (uint32_t w = first_slot / 64; w <= (last - 1) / 64; ++w) c.h_active[w] |= slot_mask(first_slot, n_slots, w);
    upload_active(c);
    c.sync();  // host inputs are read by the copies above: done before returning
    GSS_API_END
}

extern "C" gss_status gss_set_var_values(gss_ctx *ctx, uint32_t first_slot, uint32_t n_slots, uint32_t n_vars,
                                         const uint32_t *vars, const int8_t *values) {
    GSS_API_BEGIN(ctx)
    c_->mutations++;  // a test in flight no longer sees the current state
    Ctx &c = *c_;
    if (n_slots == 0 || n_vars == 0) return GSS_OK;
    GSS_REQUIRE(vars && values, GSS_ERR_INVALID_ARG, "null argument");
    check_delta_slots(c, first_slot, n_slots);
    const uint64_t nv = (uint64_t)n_vars * n_slots;
    const bool dev = is_device_pointer(values);
    const uint32_t *bad = c.dsmall + 1;  // always zero
    if (dev) {
        // device values are checked on the device, and so are repeated variables:
        // one synchronisation at the end reports either
        check_var_range(c, vars, n_vars);
        bad = queue_value_check(c, values, nv);
        if (!c.var_bits) {
            c.var_bits = (uint32_t *)c.dalloc(((uint64_t)c.cfg.num_vars / 32 + 1) * 4);
            launch_fill_u32(c, c.var_bits, (uint64_t)c.cfg.num_vars / 32 + 1, 0);
        }
    } else {
        check_vars(c, vars, n_vars);
        check_values_host(values, nv);
    }

    const size_t vars_bytes = ((size_t)n_vars * 4 + 255) / 256 * 256;
    const size_t bytes = vars_bytes + (dev ? 0 : nv);
    const bool direct = !dev && bytes <= kDirectList;
    const Ctx::Staged st = c.stage_upload(bytes, direct);
    char *h = st.h, *d = direct ? const_cast<char *>(st.hd) : st.d;
    std::memcpy(h, vars, (size_t)n_vars * 4);
    if (!dev) std::memcpy(h + vars_bytes, values, nv);
    if (!direct) GSS_HIP(hipMemcpyAsync(d, h, bytes, hipMemcpyHostToDevice, c.stream));
    const int8_t *dvals = dev ? values : (const int8_t *)(d + vars_bytes);
    if (dev) {
        hipLaunchKernelGGL(k_check_vars, dim3((n_vars + 255) / 256), dim3(256), 0, c.stream, (const uint32_t *)d, n_vars,
                           c.var_bits, c.dsmall);
        GSS_HIP(hipGetLastError());
    }
    launch_set_vars(c, (const uint32_t *)d, n_vars, dvals, first_slot, n_slots, bad, dev ? c.var_bits : nullptr);
    agg_after_delta(c, (const uint32_t *)d, n_vars);
    c.stage_done(st);
    if (dev) check_flag(c);  // one synchronisation: device inputs are fully read when the call returns
    GSS_API_END
}

extern "C" gss_status gss_set_var_values_async(gss_ctx *ctx, uint32_t first_slot, uint32_t n_slots, uint32_t n_vars,
                                               const uint32_t *vars, const int8_t *values) {
    GSS_API_BEGIN(ctx)
    c_->mutations++;  // a test in flight no longer sees the current state
    Ctx &c = *c_;
    if (n_slots == 0 || n_vars == 0) return GSS_OK;
    GSS_REQUIRE(vars && values, GSS_ERR_INVALID_ARG, "null argument");
    GSS_REQUIRE(is_device_pointer(values), GSS_ERR_INVALID_ARG, "values must be device memory");
    check_delta_slots(c, first_slot, n_slots);
    check_var_range(c, vars, n_vars);
    if (!c.var_bits) {
        c.var_bits = (uint32_t *)c.dalloc(((uint64_t)c.cfg.num_vars / 32 + 1) * 4);
        launch_fill_u32(c, c.var_bits, (uint64_t)c.cfg.num_vars / 32 + 1, 0);
    }
    // A short list is read from its pinned ring slot by the checking kernel.  A longer
    // one goes up on the copy stream, which runs while the test ahead of it executes
    // (on the context stream, a copy would start only when that test ends); the
    // checking kernel waits for it.  The copy's three calls take about 20 us of host
    // time, and its wait leaves the stream idle for 5 us; 64 KiB over the bus take the
    // kernel 2 us.
    const size_t bytes = (size_t)n_vars * 4;
    const bool direct = bytes <= kDirectList;
    const Ctx::Staged st = c.stage_upload(bytes);
    std::memcpy(st.h, vars, bytes);
    uint32_t *dv = (uint32_t *)st.d;
    if (!direct) {
        if (!c.copy_stream) {
            GSS_HIP(hipStreamCreateWithFlags(&c.copy_stream, hipStreamNonBlocking));
            GSS_HIP(hipEventCreateWithFlags(&c.ev_copy, hipEventDisableTiming));
        }
        GSS_HIP(hipMemcpyAsync(dv, st.h, bytes, hipMemcpyHostToDevice, c.copy_stream));
        GSS_HIP(hipEventRecord(c.ev_copy, c.copy_stream));
        GSS_HIP(hipStreamWaitEvent(c.stream, c.ev_copy, 0));
    }
    uint32_t *bad = deferred_flag(c);  // sticky: set by this check or an earlier one not yet reported
    const uint64_t nv = (uint64_t)n_vars * n_slots;
    const uint32_t var_blocks = (n_vars + 255) / 256;
    hipLaunchKernelGGL(k_check_delta, dim3(var_blocks + fill_grid((nv + 15) / 16)), dim3(256), 0, c.stream, values, nv,
                       var_blocks, direct ? (const uint32_t *)st.hd : nullptr, dv, n_vars, c.var_bits, bad);
    GSS_HIP(hipGetLastError());
    launch_set_vars(c, dv, n_vars, values, first_slot, n_slots, bad, c.var_bits);
    agg_after_delta(c, dv, n_vars);
    c.stage_done(st);
    GSS_API_END
}

extern "C" gss_status gss_clear_slots(gss_ctx *ctx, uint32_t first_slot, uint32_t n_slots) {
    GSS_API_BEGIN(ctx)
    c_->mutations++;  // a test in flight no longer sees the current state
    Ctx &c = *c_;
    if (n_slots == 0) return GSS_OK;
    GSS_REQUIRE((uint64_t)first_slot + n_slots <= c.cfg.max_slots, GSS_ERR_CAPACITY, "slot range beyond max_slots");
    const uint64_t n_rows = 2ull * ((uint64_t)c.cfg.num_vars + 1);
    const uint64_t nw = (first_slot + n_slots - 1) / 64 - first_slot / 64 + 1;
    const uint64_t total = (n_rows - 2) * nw;
    const unsigned grid = (unsigned)std::max<uint64_t>(1, std::min<uint64_t>((total + 255) / 256, 16384));
    hipLaunchKernelGGL(k_clear_slots, dim3(grid), dim3(256), 0, c.stream, c.planes, c.RWc, c.chunk_elems, n_rows,
                       first_slot, n_slots);
    GSS_HIP(hipGetLastError());
    c.agg_valid = false;
    c.aggu_valid = false;
    for (uint32_t w = first_slot / 64; w <= (first_slot + n_slots - 1) / 64; ++w)
        c.h_active[w] &= ~slot_mask(first_slot, n_slots, w);
    upload_active(c);
    GSS_API_END
}

extern "C" gss_status gss_update_words(gss_ctx *ctx, uint32_t word, uint32_t n_vars, const uint32_t *vars,
                                       const uint64_t *f_words, const uint64_t *t_words) {
    GSS_API_BEGIN(ctx)
    c_->mutations++;  // a test in flight no longer sees the current state
    Ctx &c = *c_;
    if (n_vars == 0) return GSS_OK;
    GSS_REQUIRE(vars && f_words && t_words, GSS_ERR_INVALID_ARG, "null argument");
    GSS_REQUIRE(word < c.W, GSS_ERR_CAPACITY, "word beyond max_slots / 64");
    check_vars(c, vars, n_vars);
    uint64_t both = 0;
    for (uint32_t i = 0; i < n_vars; ++i) both |= f_words[i] & t_words[i];
    GSS_REQUIRE(both == 0, GSS_ERR_INVALID_ARG, "a slot cannot be both F and T");
    const size_t vb = ((size_t)n_vars * 4 + 255) / 256 * 256, wb = ((size_t)n_vars * 8 + 255) / 256 * 256;
    const bool direct = vb + 2 * wb <= kDirectDelta;
    const Ctx::Staged st = c.stage_upload(vb + 2 * wb, direct);
    char *h = st.h, *d = direct ? const_cast<char *>(st.hd) : st.d;
    std::memcpy(h, vars, (size_t)n_vars * 4);
    std::memcpy(h + vb, f_words, (size_t)n_vars * 8);
    std::memcpy(h + vb + wb, t_words, (size_t)n_vars * 8);
    if (!direct) GSS_HIP(hipMemcpyAsync(d, h, vb + 2 * wb, hipMemcpyHostToDevice, c.stream));
    launch_set_words(c, word, (const uint32_t *)d, (const uint64_t *)(d + vb), (const uint64_t *)(d + vb + wb), n_vars);
    c.stage_done(st);
    GSS_API_END
}

extern "C" gss_status gss_set_active(gss_ctx *ctx, const uint64_t *active) {
    GSS_API_BEGIN(ctx)
    c_->mutations++;  // a test in flight no longer sees the current state
    Ctx &c = *c_;
    GSS_REQUIRE(active != nullptr, GSS_ERR_INVALID_ARG, "null argument");
    std::memcpy(c.h_active.data(), active, c.W * 8);
    upload_active(c);
    GSS_API_END
}

extern "C" gss_status gss_update_vars(gss_ctx *ctx, uint32_t word, uint32_t n_vars, const uint32_t *vars,
                                      const uint64_t *fp_words, const uint64_t *fn_words) {
    return gss_update_words(ctx, word, n_vars, vars, fp_words, fn_words);
}

// Kernels of the tlookup prover (Section 4 of the paper, Protocol 1): table
// hashing and multiplicity counting, the leaf digests of m, pooled eq tables,
// and the sumcheck round kernels for the data side (A, S) and the table side
// (B, T, m) of the tlookup identity.
#pragma once
#include "common.h"
#include "reduce_dev.h"
#include "fr29_dev.h"
#include "mle_dev.h"
#include "sha256_dev.h"
#include "small_dev.h"

namespace zkmi {

// ---- table rows by value: open-addressing hash of T -----------------------------

static const uint32_t kEmptySlot = 0xffffffffu;

__device__ __forceinline__ uint32_t fr_hash(const Fr& a) {
    uint32_t h = a.l[0] * 0x9e3779b1u;
    h = (h ^ a.l[1]) * 0x85ebca77u;
    h = (h ^ a.l[2]) * 0xc2b2ae3du;
    h = (h ^ a.l[3]) * 0x27d4eb2fu;
    h = (h ^ a.l[4]) * 0x165667b1u;
    h = (h ^ a.l[5]) * 0x9e3779b1u;
    h = (h ^ a.l[6]) * 0x85ebca77u;
    h = (h ^ a.l[7]) * 0xc2b2ae3du;
    return h ^ (h >> 15);
}

// What the kernels that work on tables need of each; blockIdx.y is the table.  The tables of
// a call share launches: short ones took as long one after the other as launches do (three
// tables of 2^10 to 2^16 rows: counting 262 -> 142 us, inversions 160 -> 115, with the trips).
struct TableJob {
    const uint32_t* T;
    size_t ts;
    uint32_t N;
    uint32_t* slots;    // hash of T
    uint32_t cap_mask;
    uint32_t* flags;
    uint32_t* canon;
    uint4* rows;
    uint32_t* m;        // counts
    const uint32_t* hist;  // the workgroups' histograms
    uint32_t hist_parts;   // (none: zero)
    uint32_t* M;        // counts as field elements
    const uint32_t* B;
    uint4* rows_b;      // null: B's rows are not asked for
    uint4* rows_hash;   // not null: B's canonical values by themselves, and what the rounds read by row:
    uint4* rows_pair;   // (tlookup_rows.h)
};
// (Calls with one table pass one, whose pointers the compiler can see to be global: through
// an array they are flat, and flat loads share a counter with the LDS; the counts' leaves
// took 28 instead of 25 us.)
static const int kMaxTables = 8;
template <int NT>
struct TableJobs {
    TableJob job[NT];
};

// How far apart the slots are that a value looks at one after the other: odd, so that it comes
// to all of them.  (Next to each other, full stretches of the half full table grow, and
// wavefronts wait for the longest.)
__device__ __forceinline__ uint32_t hash_step(uint32_t hash) { return (hash >> 12) | 1u; }

// Every row j claims the first slot of its probe sequence that is empty or holds
// a row with the same value; equal values meet in one slot and the lowest row
// wins.  Slots never empty again and the value class of a slot never changes, so
// all rows of one value walk the same sequence to the same slot.
template <int NT>
static __global__ void __launch_bounds__(kBlock) k_hash_build(TableJobs<NT> tables) {
    const TableJob& g = tables.job[NT == 1 ? 0 : blockIdx.y];
    uint32_t* const slots = g.slots;
    const uint32_t* __restrict__ const T = g.T;
    uint32_t* const dup_flag = g.flags;
    const uint32_t cap_mask = g.cap_mask, N = g.N;
    const size_t ts = g.ts;
    for (uint32_t j = blockIdx.x * kBlock + threadIdx.x; j < N; j += gridDim.x * kBlock) {
        Fr v = fr_load(T, ts, j);
        const uint32_t hash = fr_hash(v), by = hash_step(hash);
        uint32_t pos = hash & cap_mask;
        for (uint32_t step = 0; step <= cap_mask; ++step) {
            uint32_t cur = atomicCAS(&slots[pos], kEmptySlot, j);
            if (cur == kEmptySlot) break;  // claimed
            if (fr_equal(fr_load(T, ts, cur), v)) {
                atomicMin(&slots[pos], j);
                atomicOr(dup_flag, 1u);
                break;
            }
            pos = (pos + by) & cap_mask;
        }
    }
}

// Row of the table holding value v (lowest row of equal ones), or kEmptySlot.
__device__ __forceinline__ uint32_t hash_find(const uint32_t* __restrict__ slots, uint32_t cap_mask,
                                              const uint32_t* __restrict__ T, size_t ts, const Fr& v) {
    const uint32_t hash = fr_hash(v), by = hash_step(hash);
    uint32_t pos = hash & cap_mask;
    for (uint32_t step = 0; step <= cap_mask; ++step) {
        uint32_t cur = slots[pos];
        if (cur == kEmptySlot) return kEmptySlot;
        if (fr_equal(fr_load(T, ts, cur), v)) return cur;
        pos = (pos + by) & cap_mask;
    }
    return kEmptySlot;
}

// The same through the row-major copy of the table (k_canon_rows): a candidate row
// is one 32-byte access instead of eight words from eight limb planes.
__device__ __forceinline__ uint32_t hash_find_rows(const uint32_t* __restrict__ slots, uint32_t cap_mask,
                                                   const uint4* __restrict__ rows, const Fr& v) {
    const uint32_t hash = fr_hash(v), by = hash_step(hash);
    uint32_t pos = hash & cap_mask;
    for (uint32_t step = 0; step <= cap_mask; ++step) {
        uint32_t cur = slots[pos];
        if (cur == kEmptySlot) return kEmptySlot;
        const uint4 lo = rows[2 * (size_t)cur], hi = rows[2 * (size_t)cur + 1];
        const uint32_t diff = (lo.x ^ v.l[0]) | (lo.y ^ v.l[1]) | (lo.z ^ v.l[2]) | (lo.w ^ v.l[3]) |
                              (hi.x ^ v.l[4]) | (hi.y ^ v.l[5]) | (hi.z ^ v.l[6]) | (hi.w ^ v.l[7]);
        if (diff == 0) return cur;
        pos = (pos + by) & cap_mask;
    }
    return kEmptySlot;
}

// canon[j] = lowest row with the value of row j; rows[j] = row j of T as eight
// consecutive words, so that a lookup by row number is one 32-byte access
// instead of eight accesses to eight limb planes.
template <int NT>
static __global__ void __launch_bounds__(kBlock) k_canon_rows(TableJobs<NT> tables) {
    const TableJob& g = tables.job[NT == 1 ? 0 : blockIdx.y];
    uint32_t* __restrict__ const canon = g.canon;
    uint4* __restrict__ const rows = g.rows;
    const uint32_t* __restrict__ const slots = g.slots;
    const uint32_t* __restrict__ const T = g.T;
    const uint32_t cap_mask = g.cap_mask, N = g.N;
    const size_t ts = g.ts;
    for (uint32_t j = blockIdx.x * kBlock + threadIdx.x; j < N; j += gridDim.x * kBlock) {
        Fr v = fr_load(T, ts, j);
        canon[j] = hash_find(slots, cap_mask, T, ts, v);
        rows[2 * j] = make_uint4(v.l[0], v.l[1], v.l[2], v.l[3]);
        rows[2 * j + 1] = make_uint4(v.l[4], v.l[5], v.l[6], v.l[7]);
    }
}

// All that counting starts from (k_count_init, k_hash_build, k_canon_rows) for tables of few
// rows, a workgroup each, the hash in LDS until it is done: kernel time of 2^8 rows 10.8 us in
// three launches, 4.3 in this one (2^11: 16.9 and 9.7), a proof of 2^10 entries in 2^8 rows 257
// -> 250 us, of 2^14 in 2^11 rows 422 -> 413.
static const size_t kSmallTable = 2048;
template <int NT>
static __global__ void __launch_bounds__(1024) k_table_small(TableJobs<NT> tables) {
    __shared__ uint32_t slots[2 * kSmallTable];
    __shared__ uint32_t dup;
    const TableJob& g = tables.job[NT == 1 ? 0 : blockIdx.y];
    const uint32_t cap_mask = g.cap_mask, N = g.N;  // at most kSmallTable rows, twice as many slots
    const uint32_t* __restrict__ const T = g.T;
    for (uint32_t i = threadIdx.x; i <= cap_mask; i += 1024) slots[i] = kEmptySlot;
    for (uint32_t j = threadIdx.x; j < N; j += 1024) g.m[j] = 0;
    if (threadIdx.x == 0) dup = 0;
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < N; j += 1024) {
        const Fr v = fr_load(T, g.ts, j);
        g.rows[2 * j] = make_uint4(v.l[0], v.l[1], v.l[2], v.l[3]);
        g.rows[2 * j + 1] = make_uint4(v.l[4], v.l[5], v.l[6], v.l[7]);
        const uint32_t hash = fr_hash(v), by = hash_step(hash);
        uint32_t pos = hash & cap_mask;
        for (uint32_t step = 0; step <= cap_mask; ++step) {
            const uint32_t cur = atomicCAS(&slots[pos], kEmptySlot, j);
            if (cur == kEmptySlot) break;  // claimed
            if (fr_equal(fr_load(T, g.ts, cur), v)) {
                atomicMin(&slots[pos], j);
                dup = 1;
                break;
            }
            pos = (pos + by) & cap_mask;
        }
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i <= cap_mask; i += 1024) g.slots[i] = slots[i];
    if (threadIdx.x < 4) g.flags[threadIdx.x] = threadIdx.x == 0 ? dup : threadIdx.x == 1 ? 0u : 0xffffffffu;
    // without duplicates every row is its value's lowest
    for (uint32_t j = threadIdx.x; j < N; j += 1024) g.canon[j] = dup ? hash_find(slots, cap_mask, T, g.ts, fr_load(T, g.ts, j)) : j;
}

// The row of every S_i, for calls without hints (the smallest i that has none ends up in
// *bad, its row is the table's length).  A kernel of its own: four dependent accesses
// per element want wavefronts, and the counting's 128 KiB of LDS per workgroup leaves
// four per SIMD (2^25 elements in 2^16 rows: 0.98 ms when the counting looked them up,
// 0.87 ms here and there together).
static __global__ void __launch_bounds__(kBlock) k_find_rows(uint32_t* __restrict__ found, const uint32_t* __restrict__ S, size_t ss,
                                                      size_t D, const uint4* __restrict__ rows, uint32_t N,
                                                      const uint32_t* __restrict__ slots, uint32_t cap_mask,
                                                      unsigned long long* bad) {
    const size_t i = blockIdx.x * (size_t)kBlock + threadIdx.x;
    if (i >= D) return;
    const uint32_t row = hash_find_rows(slots, cap_mask, rows, fr_load(S, ss, i));
    found[i] = row == kEmptySlot ? N : row;
    if (row == kEmptySlot) atomicMin(bad, (unsigned long long)i);
}

// A wavefront's running total for the row it keeps meeting (wave-uniform).
// Long runs of one row (padding, saturated activations) would otherwise become
// a stream of atomics to a single address, which the memory system serialises.
struct HotRun {
    uint32_t row = kEmptySlot;
    uint32_t count = 0;
    __device__ __forceinline__ void add(uint32_t* m, uint32_t r, uint32_t c) {
        if (r == row) {
            count += c;
        } else {
            flush(m);
            row = r;
            count = c;
        }
    }
    __device__ __forceinline__ void flush(uint32_t* m) {
        if (count && (threadIdx.x & 63) == 0) atomicAdd(&m[row], count);
        count = 0;
    }
};

// Adds one to m[row] for every active lane with a valid row.  Lanes of a
// wavefront that hit the same row are merged first: a few rounds of "take the
// first pending lane's row, count the lanes that share it", runs of half a
// wavefront or more going to the wavefront's running total and shorter ones to
// one atomic each, then plain atomics for whatever rows are left.
__device__ __forceinline__ void count_merged(uint32_t* m, uint32_t row, bool valid, HotRun& hot) {
    bool pending = valid;
#pragma unroll 1
    for (int round = 0; round < 8; ++round) {
        unsigned long long todo = __ballot(pending);
        if (todo == 0) return;
        int leader = __ffsll((long long)todo) - 1;
        uint32_t lead_row = (uint32_t)__builtin_amdgcn_readlane((int)row, leader);  // leader is wave-uniform: no trip through LDS
        bool mine = pending && row == lead_row;
        uint32_t run = (uint32_t)__popcll(__ballot(mine));
        if (run >= 32) hot.add(m, lead_row, run);
        else if ((int)(threadIdx.x & 63) == leader) atomicAdd(&m[lead_row], run);
        pending = pending && !mine;
    }
    if (pending) atomicAdd(&m[row], 1u);
}

// m[row(S_i)] += 1.  With idx the row is given and only checked; without, it is
// found through the hash.  The smallest offending i ends up in *bad.
static __global__ void __launch_bounds__(kBlock) k_count(uint32_t* m, const uint32_t* __restrict__ S, size_t ss, size_t D,
                                                  const uint32_t* __restrict__ idx, const uint32_t* __restrict__ T,
                                                  size_t ts, const uint4* __restrict__ rows, uint32_t N,
                                                  const uint32_t* __restrict__ slots,
                                                  uint32_t cap_mask, const uint32_t* __restrict__ canon,
                                                  const uint32_t* __restrict__ dup_flag, unsigned long long* bad) {
    const bool dups = *dup_flag != 0;
    // every lane of a wavefront runs the same number of iterations, so the
    // cross-lane steps in count_merged see whole wavefronts
    const size_t per_pass = (size_t)gridDim.x * kBlock;
    const size_t passes = (D + per_pass - 1) / per_pass;
    HotRun hot;
    for (size_t pass = 0; pass < passes; ++pass) {
        size_t i = pass * per_pass + blockIdx.x * (size_t)kBlock + threadIdx.x;
        bool in_range = i < D;
        uint32_t row = kEmptySlot;
        if (in_range) {
            Fr v = fr_load(S, ss, i);
            if (idx) {
                row = idx[i];
                if (row < N) {
                    uint4 lo = rows[2 * (size_t)row], hi = rows[2 * (size_t)row + 1];
                    uint32_t diff = (lo.x ^ v.l[0]) | (lo.y ^ v.l[1]) | (lo.z ^ v.l[2]) | (lo.w ^ v.l[3]) |
                                    (hi.x ^ v.l[4]) | (hi.y ^ v.l[5]) | (hi.z ^ v.l[6]) | (hi.w ^ v.l[7]);
                    if (diff) row = kEmptySlot;
                    else if (dups) row = canon[row];
                } else {
                    row = kEmptySlot;
                }
            } else {
                row = hash_find_rows(slots, cap_mask, rows, v);
            }
            if (row == kEmptySlot) atomicMin(bad, (unsigned long long)i);
        }
        count_merged(m, row, in_range && row != kEmptySlot, hot);
    }
    hot.flush(m);
}

// ---- multiplicities through workgroup-private histograms in LDS ---------------------
//
// For tables of up to 2^16 rows the counters of a workgroup fit in LDS as packed
// 16-bit pairs (128 KiB at 2^16 rows, of the 160 KiB a gfx950 compute unit has),
// which takes the counting off the device-wide atomics.  A workgroup walks its
// share of S in passes (chunks of at most kHistPass elements, handed out round
// robin) short enough that no 16-bit counter can overflow, and
// after each pass adds its counters into a 32-bit histogram of its own in HBM
// (plain loads and stores, nobody else touches it); a second kernel adds the
// workgroups' histograms up.  Runs of one row that fill half a wavefront or more
// (padding, saturated activations) are kept in a per-wavefront running total and
// go straight to the result, so they do not eat into the 16-bit budget.
static const int kHistThreads = 1024;
static const uint32_t kHistPass = 60 * 1024;  // elements per pass, < 2^16

// CHECK_S = false: rows are taken from the hints unchecked (an out-of-range hint
// is not counted); the comparison of every S_i with its row is then the caller's
// business (it rides on what reads the rows: see LeafGather).
template <bool CHECK_S>
static __global__ void __launch_bounds__(kHistThreads)
k_count_lds(uint32_t* m, uint32_t* __restrict__ part, const uint32_t* __restrict__ S, size_t ss, size_t D,
            size_t chunk, const uint32_t* __restrict__ idx, const uint32_t* __restrict__ T, size_t ts,
            const uint4* __restrict__ rows, uint32_t N, const uint32_t* __restrict__ slots, uint32_t cap_mask,
            const uint32_t* __restrict__ canon, const uint32_t* __restrict__ dup_flag, unsigned long long* bad) {
    extern __shared__ uint32_t hist[];  // (N+1)/2 words, two 16-bit counters each
    const uint32_t words = (N + 1) / 2;
    const bool dups = *dup_flag != 0;
    uint32_t* mine_part = part + (size_t)blockIdx.x * N;
    bool first = true;
    HotRun hot;
    // pass p of this workgroup covers chunk p * gridDim.x + blockIdx.x of S: stretches
    // that are cheap to count (padding) are spread over all workgroups that way
    for (size_t pass_begin = blockIdx.x * chunk; pass_begin < D || first; pass_begin += (size_t)gridDim.x * chunk) {
        for (uint32_t w = threadIdx.x; w < words; w += kHistThreads) hist[w] = 0;
        __syncthreads();
        const size_t pass_end = pass_begin + chunk < D ? pass_begin + chunk : D;
        // whole wavefronts iterate together so that the cross-lane merge sees all 64
        // lanes; several elements per thread per trip keep more loads in flight
        constexpr int E = 8;
        for (size_t base = pass_begin; base < pass_end; base += E * kHistThreads) {
            size_t i[E];
            bool in_range[E];
            uint32_t row[E];
            Fr v[CHECK_S ? E : 1];
#pragma unroll
            for (int e = 0; e < E; ++e) {
                i[e] = base + (size_t)e * kHistThreads + threadIdx.x;
                in_range[e] = i[e] < pass_end;
                row[e] = kEmptySlot;
                if (in_range[e]) {
                    if (idx) row[e] = idx[i[e]];
                    if constexpr (CHECK_S) v[e] = fr_load(S, ss, i[e]);
                }
            }
#pragma unroll
            for (int e = 0; e < E; ++e) {
                if (!in_range[e]) continue;
                if (idx) {
                    uint32_t r = row[e];
                    if (r < N) {
                        uint32_t diff = 0;
                        if constexpr (CHECK_S) {
                            uint4 lo = rows[2 * (size_t)r], hi = rows[2 * (size_t)r + 1];
                            diff = (lo.x ^ v[e].l[0]) | (lo.y ^ v[e].l[1]) | (lo.z ^ v[e].l[2]) | (lo.w ^ v[e].l[3]) |
                                   (hi.x ^ v[e].l[4]) | (hi.y ^ v[e].l[5]) | (hi.z ^ v[e].l[6]) | (hi.w ^ v[e].l[7]);
                        }
                        if (diff) r = kEmptySlot;
                        else if (dups) r = canon[r];
                    } else {
                        r = kEmptySlot;
                    }
                    row[e] = r;
                } else {
                    if constexpr (CHECK_S) row[e] = hash_find_rows(slots, cap_mask, rows, v[e]);
                }
                // without the comparison a hint out of range is left for the caller's check to report
                if (CHECK_S && row[e] == kEmptySlot) atomicMin(bad, (unsigned long long)i[e]);
            }
#pragma unroll
            for (int e = 0; e < E; ++e) {
                bool pending = in_range[e] && row[e] != kEmptySlot;
#pragma unroll 1
                for (int round = 0; round < 4; ++round) {
                    unsigned long long todo = __ballot(pending);
                    if (todo == 0) break;
                    int leader = __ffsll((long long)todo) - 1;
                    uint32_t lead_row = (uint32_t)__builtin_amdgcn_readlane((int)row[e], leader);  // wave-uniform lane: no trip through LDS
                    bool same_row = pending && row[e] == lead_row;
                    uint32_t run = (uint32_t)__popcll(__ballot(same_row));
                    // A long run goes to the wavefront's running total and a run of a few
                    // lanes is added once by its first lane (lanes on one address are
                    // served one after the other).  A run of one to three lanes says that
                    // the wavefront's rows are mostly different: the remaining lanes then
                    // go in one instruction, because the LDS pipeline, which every
                    // instruction occupies for about as long whatever it carries, is what
                    // bounds this kernel.
                    if (run >= 32) hot.add(m, lead_row, run);
                    else if (run < 4) break;
                    else if ((int)(threadIdx.x & 63) == leader)
                        atomicAdd(&hist[lead_row >> 1], run << (16 * (lead_row & 1)));
                    pending = pending && !same_row;
                }
                if (pending) atomicAdd(&hist[row[e] >> 1], 1u << (16 * (row[e] & 1)));
            }
        }
        __syncthreads();
        // Flush into this workgroup's 32-bit histogram, eight words per thread at a
        // time so that the loads of a group are in flight together (one word after
        // the other this flush cost more than the counting).
        if ((N & 1u) == 0) {
            uint2* mine2 = reinterpret_cast<uint2*>(mine_part);
            for (uint32_t w0 = threadIdx.x; w0 < words; w0 += 8 * kHistThreads) {
                uint32_t v[8];
                uint2 old[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const uint32_t w = w0 + k * kHistThreads;
                    v[k] = w < words ? hist[w] : 0;
                    old[k] = make_uint2(0, 0);
                    if (!first && v[k]) old[k] = mine2[w];
                }
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const uint32_t w = w0 + k * kHistThreads;
                    if (w < words && (first || v[k])) mine2[w] = make_uint2(old[k].x + (v[k] & 0xffffu), old[k].y + (v[k] >> 16));
                }
            }
        } else {  // a table of one row
            for (uint32_t w = threadIdx.x; w < words; w += kHistThreads) {
                uint32_t v = hist[w];
                uint32_t c0 = v & 0xffffu, c1 = v >> 16;
                if (first) {
                    mine_part[2 * w] = c0;
                    if (2 * w + 1 < N) mine_part[2 * w + 1] = c1;
                } else if (v) {
                    mine_part[2 * w] += c0;
                    if (2 * w + 1 < N) mine_part[2 * w + 1] += c1;
                }
            }
        }
        __syncthreads();
        first = false;
    }
    hot.flush(m);
}

// m[j] += sum over workgroups of their histograms; blockIdx.y selects a group of
// `group` histograms, so that the additions of one row are spread over several
// threads.
template <int NT>
static __global__ void __launch_bounds__(kBlock) k_hist_reduce(TableJobs<NT> tables, uint32_t group) {
    const TableJob& g = tables.job[NT == 1 ? 0 : blockIdx.z];
    uint32_t* __restrict__ const m = g.m;
    const uint32_t* __restrict__ const part = g.hist;
    const uint32_t nparts = g.hist_parts, N = g.N;
    uint32_t j = blockIdx.x * kBlock + threadIdx.x;
    if (j >= N) return;
    uint32_t b0 = blockIdx.y * group, b1 = b0 + group < nparts ? b0 + group : nparts;
    uint32_t acc = 0;
    for (uint32_t b = b0; b < b1; ++b) acc += part[(size_t)b * N + j];
    if (acc) atomicAdd(&m[j], acc);
}

// Row j of B as sixteen consecutive words, so that reading it by number is one
// 64-byte access: the element, then its canonical value as the hash takes it
// (big-endian bytes of little-endian words).  Where A itself is not asked for, only its
// hash (rows_hash not null), the hash's values lie by themselves, 32 bytes each, and the
// rows are those the rounds read by row: T's balanced digits (outer_dev.h) and B's words
// for the first pass (rows_b), both elements' digits for the second (rows_pair).
__device__ __forceinline__ void row_digits(uint4* at, const Fr& v) {
    uint32_t d[8], carry = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        uint32_t co;
        d[k] = __builtin_addc(v.l[k], 0x80808080u, carry, &co) ^ 0x80808080u;
        carry = co;
    }
    at[0] = make_uint4(d[0], d[1], d[2], d[3]);
    at[1] = make_uint4(d[4], d[5], d[6], d[7]);
}
template <int NT>
static __global__ void __launch_bounds__(kBlock) k_rows_of(TableJobs<NT> tables) {
    const TableJob& g = tables.job[NT == 1 ? 0 : blockIdx.y];
    uint4* __restrict__ const rows = g.rows_b;
    const uint32_t* __restrict__ const B = g.B;
    const uint32_t N = rows ? g.N : 0;
    const size_t bs = g.N;
    for (uint32_t j = blockIdx.x * kBlock + threadIdx.x; j < N; j += gridDim.x * kBlock) {
        const Fr v = fr_load(B, bs, j);
        Fr c = fr_from_mont(v);
#pragma unroll
        for (int k = 0; k < 8; ++k) c.l[k] = __builtin_bswap32(c.l[k]);
        uint4 *words = rows + 4 * (size_t)j, *hash = words + 2;
        if (g.rows_hash) {
            const Fr t = fr_load(g.T, g.ts, j);
            row_digits(words, t);
            row_digits(g.rows_pair + 4 * (size_t)j, v);
            row_digits(g.rows_pair + 4 * (size_t)j + 2, t);
            words += 2;
            hash = g.rows_hash + 2 * (size_t)j;
        }
        words[0] = make_uint4(v.l[0], v.l[1], v.l[2], v.l[3]);
        words[1] = make_uint4(v.l[4], v.l[5], v.l[6], v.l[7]);
        hash[0] = make_uint4(c.l[0], c.l[1], c.l[2], c.l[3]);
        hash[1] = make_uint4(c.l[4], c.l[5], c.l[6], c.l[7]);
    }
}

// What counting starts from, in one launch: empty hash slots, zero counts, and the
// four flag words (duplicate flag and ticket zero, smallest bad index all ones).
template <int NT>
static __global__ void __launch_bounds__(kBlock) k_count_init(TableJobs<NT> tables) {
    const TableJob& g = tables.job[NT == 1 ? 0 : blockIdx.y];
    uint32_t* __restrict__ const slots = g.slots;
    uint32_t* __restrict__ const m = g.m;
    uint32_t* __restrict__ const flags = g.flags;
    const size_t cap = (size_t)g.cap_mask + 1, N = g.N;
    const size_t total = cap + N + 4;
    for (size_t i = blockIdx.x * (size_t)kBlock + threadIdx.x; i < total; i += (size_t)gridDim.x * kBlock) {
        if (i < cap) slots[i] = kEmptySlot;
        else if (i < cap + N) m[i - cap] = 0;
        else flags[i - cap - N] = i - cap - N < 2 ? 0u : 0xffffffffu;
    }
}

template <int NT>
static __global__ void __launch_bounds__(kBlock) k_counts_to_fr(TableJobs<NT> tables) {
    const TableJob& g = tables.job[NT == 1 ? 0 : blockIdx.y];
    for (size_t j = blockIdx.x * (size_t)kBlock + threadIdx.x; j < g.N; j += (size_t)gridDim.x * kBlock)
        fr_store(g.M, g.N, j, fr_from_u32(g.m[j]));
}

// The last step of counting where the host hashes m: the workgroups' histograms added up,
// the counts as they are and as field elements, and to pinned memory, behind the flags (in one
// launch what k_hist_reduce, k_leaf_digests and k_counts_to_fr do in three).  A workgroup takes
// 64 rows, sixteen threads each.
template <int NT>
struct CountsOutArgs {
    TableJobs<NT> tables;
    uint32_t* out[NT];  // four flag words, then the counts
    uint32_t* words;    // the mailbox
    uint32_t* ticket;
    uint32_t seq;
};
template <int NT>
static __global__ void __launch_bounds__(1024) k_counts_out(CountsOutArgs<NT> args) {
    __shared__ uint32_t sums[16][64];
    const int t = NT == 1 ? 0 : blockIdx.y;
    const TableJob& g = args.tables.job[t];
    const uint32_t lane = threadIdx.x & 63, group = threadIdx.x >> 6, j = blockIdx.x * 64 + lane;
    uint32_t acc = 0;
    if (j < g.N) {
#pragma unroll 8
        for (uint32_t b = group; b < g.hist_parts; b += 16) acc += g.hist[(size_t)b * g.N + j];
    }
    sums[group][lane] = acc;
    __syncthreads();
    if (threadIdx.x < 64 && j < g.N) {
        acc = g.m[j];  // long runs of one row
#pragma unroll
        for (int q = 0; q < 16; ++q) acc += sums[q][lane];
        g.m[j] = acc;
        fr_store(g.M, g.N, j, fr_from_u32(acc));
        args.out[t][4 + j] = acc;
        if (j < 4) args.out[t][j] = g.flags[j];
        if (g.N < 4 && j == 0)
            for (uint32_t q = g.N; q < 4; ++q) args.out[t][q] = g.flags[q];
        mailbox_written();
    }
    __syncthreads();
    if (threadIdx.x == 0 && atomicAdd(args.ticket, 1u) == gridDim.x * gridDim.y - 1) {
        *args.ticket = 0;
        mailbox_publish(args.words, args.seq);
    }
}

// ---- SHA-256 of the leaves of m ---------------------------------------------------

static const uint32_t kLeafCounts = 128;
// Up to this many leaves of a call the host hashes: 0.25 us each with SHA instructions, where the
// device takes 26 us for any number (and up to 27 for 512).
static const uint32_t kHostCountLeaves = 64;

// The rounds of a chain of blocks whose schedules (round constants added) another
// wavefront of the workgroup makes in LDS, one block ahead: kw[block & 1], four rounds
// per uint4 and lane.  Takes steps + 1 barriers, as the other does; blocks <= steps.
__device__ __forceinline__ void sha256_piped_rounds(uint32_t (&h)[8], const uint4 (*kw)[16][64], uint32_t blocks, uint32_t steps) {
    const int lane = threadIdx.x & 63;
    sha256_init(h);
    __syncthreads();
    for (uint32_t b = 0; b < steps; ++b) {
        if (b < blocks) {
            uint32_t s[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) s[i] = h[i];
#pragma unroll
            for (int g = 0; g < 16; ++g) {
                const uint4 q = kw[b & 1][g][lane];
                sha256_round(s, q.x);
                sha256_round(s, q.y);
                sha256_round(s, q.z);
                sha256_round(s, q.w);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) h[i] += s[i];
        }
        __syncthreads();
    }
}

// 64 leaves per workgroup, one lane each: SHA-256 of up to 128 counts as 4-byte
// little-endian words.  Digest bytes go out in order, 32 per leaf, straight to pinned
// host memory, and behind them the flag words of the counting (flags not null).  A leaf
// is nine dependent blocks and there are never many: one wavefront does the rounds,
// the other the schedules (42 us with one wavefront for both, 27 so).
struct LeafDigestJob {
    uint32_t* out;
    const uint32_t* m;
    uint32_t N, nleaves;
    const uint32_t* flags;  // four words
    uint32_t* out_flags;
};
template <int NT>
struct LeafDigestArgs {
    LeafDigestJob job[NT];  // by blockIdx.y
    uint32_t* words;        // the mailbox
    uint32_t* ticket;
    uint32_t seq;
};
// By two wavefronts, `rounds` the first: the 64 leaves from `first` on, of nblk blocks (0: none).
__device__ __forceinline__ void count_leaves(const LeafDigestJob& g, uint32_t first, uint32_t nblk, bool rounds, uint4 (*kw)[16][64]) {
    const int lane = threadIdx.x & 63;
    const uint32_t leaf = first + lane;
    const uint32_t base = (leaf < g.nleaves ? leaf : g.nleaves - 1) * kLeafCounts;
    const uint32_t cnt = g.N < kLeafCounts ? g.N : kLeafCounts;  // N is a power of two: all leaves are alike
    if (rounds) {
        uint32_t h[8];
        sha256_piped_rounds(h, kw, nblk, nblk);
        if (leaf < g.nleaves) {
#pragma unroll
            for (int i = 0; i < 8; ++i) g.out[leaf * 8 + i] = __builtin_bswap32(h[i]);
        }
        if (first == 0 && lane < 4 && g.flags) g.out_flags[lane] = g.flags[lane];
        mailbox_written();
    } else {
        for (uint32_t b = 0; b <= nblk; ++b) {
            if (b < nblk) {
                uint32_t w[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const uint32_t pos = b * 16 + i;
                    uint32_t v = 0;
                    if (pos < cnt) v = __builtin_bswap32(g.m[base + pos]);
                    else if (pos == cnt) v = 0x80000000u;
                    else if (pos == nblk * 16 - 1) v = cnt * 32;  // message length in bits
                    w[i] = v;
                }
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    if (q >= 4) sha256_schedule4(w, 4 * q);
                    const int i = (4 * q) & 15;
                    kw[b & 1][q][lane] = make_uint4(w[i] + kShaK[4 * q], w[i + 1] + kShaK[4 * q + 1], w[i + 2] + kShaK[4 * q + 2],
                                                    w[i + 3] + kShaK[4 * q + 3]);
                }
            }
            __syncthreads();
        }
    }
}
__device__ __forceinline__ uint32_t count_leaf_blocks(const LeafDigestJob& g) {
    return ((g.N < kLeafCounts ? g.N : kLeafCounts) + 3 + 15) / 16;
}
template <int NT>
static __global__ void __launch_bounds__(128) k_leaf_digests(LeafDigestArgs<NT> args) {
    __shared__ uint4 kw[2][16][64];
    const LeafDigestJob& g = args.job[NT == 1 ? 0 : blockIdx.y];
    count_leaves(g, blockIdx.x * 64, blockIdx.x * 64 < g.nleaves ? count_leaf_blocks(g) : 0, threadIdx.x < 64, kw);
    if (args.seq) {
        __syncthreads();
        if (threadIdx.x == 0 && atomicAdd(args.ticket, 1u) == gridDim.x * gridDim.y - 1) {
            *args.ticket = 0;
            mailbox_publish(args.words, args.seq);
        }
    }
}

// ---- digest of a vector of field elements (stand-in for its commitment) ----------
//
// A hash tree over the canonical bytes of the elements: with L = max(1, n/128)
// leaves, leaf i is the SHA-256 of elements i, i+L, i+2L, ... (so that lane i of a
// wavefront reads element i + tL in step t: one limb plane of 64 consecutive
// elements is 256 contiguous bytes); rows of digests are then hashed in
// consecutive fours (a last pair in twos) down to one.  Digests travel between
// the kernels as the eight state words of the hash (big-endian words of the
// digest's bytes).
static const uint32_t kVecLeaf = 128;

// The smallest indices found at fault while A was made: they go to the host with the digests.
struct BadWords {
    const unsigned long long* from[8];  // of each instance
    int count;
    uint32_t* to;                       // two words each
};
// By the thread that publishes, once all workgroups are done.
__device__ __forceinline__ void bad_words_publish(const BadWords& b) {
    for (int i = 0; i < b.count; ++i) {
        const unsigned long long v = __hip_atomic_load(b.from[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        b.to[2 * i] = (uint32_t)v;
        b.to[2 * i + 1] = (uint32_t)(v >> 32);
    }
}

// All vectors of a call are hashed by one launch (a leaf is a chain of 65 dependent
// blocks whatever the vector's length: one after the other, short vectors would
// cost as much as long ones).
//
// A lookup's A need not be there.  S_i is the table's row rho_i, so A_i = 1/(beta + S_i) is
// B[rho_i]: with a LeafGather the hash reads B's canonical values by row (kLeafRowsHash), and
// the inversion of D elements (three multiplications and 160 bytes per element) becomes one of
// N.  For tables of up to 2^16 rows, whose row-major copies the caches hold.  Measured at 2^25
// elements and 2^16 rows, inversion and leaves: 2.32 ms (1.21 and 1.11) -> 0.89 ms (0.06 and
// 0.83).  What else reads A by row, and compares S with T's rows: the long rounds
// (tlookup_rows.h), or, for shorter tensors (2^18 entries or fewer, kMadeApart), k_make_a, which
// writes A.  (While the hash wrote A and compared, its chain was the longer by it: 2^20 entries
// 153 us, now 126; 2^18 entries 155, now 126 and 8.)  Longer tables by row (tlookup_prove_by_rows)
// keep the hash that writes A (kLeafRows), where that rides under the hash's issue.
enum LeafMode {
    kLeafPlain = 0,      // the vector is there
    kLeafRows = 1,       // made by row and written, the rows known to be right
    kLeafRowsCheck = 2,  // made by row, S compared with T's rows (k_make_a, k_leaves_to_host)
    kLeafRowsInts = 3,   // the same with S_i from integers
    kLeafRowsHash = 4    // made by row, only hashed (LeafGather::hash_only)
};
struct LeafGather {
    const uint32_t* rows = nullptr;    // row numbers; null: the vector itself is hashed (hash_only: all rows in order)
    const uint32_t* S = nullptr;       // what kLeafRowsCheck compares
    size_t ss = 0;
    const uint4* T = nullptr;          // N rows, two uint4 each (k_canon_rows)
    const uint4* B = nullptr;          // N rows, four uint4 each (k_rows_of), or (hash_only) the words of the hash, two in
    uint32_t N = 0;                    // every hash_only uint4 (two or four)
    int hash_only = 0;
    unsigned long long* bad = nullptr; // smallest i with S_i != T[row_i] or row_i >= N
};
struct VecLeavesJob {
    uint32_t* v;           // read, or written with a LeafGather
    size_t stride, n, L;
    uint32_t* out;         // L digests; device memory, or pinned host memory if the host finishes the tree from here
    uint32_t first_group;  // of 64 leaves each
    LeafGather from;
    int to_host;           // out is pinned host memory: fenced here, whichever launch publishes
};
static const int kDigestMaxJobs = 16;  // A and B of eight instances
struct VecLeavesArgs {
    VecLeavesJob job[kDigestMaxJobs];
    int njobs;
    uint32_t groups;
    uint32_t* words;   // the mailbox, if this launch is the last to write results (seq != 0)
    uint32_t* ticket;
    uint32_t seq;
    SmallSource ints;  // k_leaves_to_host: of the job that asks for it
    BadWords bad;
};

// The pointers of a job come out of an array, so the compiler does not know that
// they are global memory; flat accesses would share a counter with the loads of the
// round constants and be waited for long before they are needed.  An element's words
// are addressed by a wave-uniform part (scalar registers) and the lane's byte offset:
// as sixteen 64-bit addresses per lane they took the registers that the elements on
// their way in need.
typedef __attribute__((address_space(1))) uint32_t GlobalWord;
typedef __attribute__((address_space(1))) char GlobalByte;
typedef uint32_t Vec4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) Vec4 GlobalVec4;

__device__ __forceinline__ GlobalWord* at_lane(const void* p, size_t uniform, uint32_t lane_bytes) {
    return (GlobalWord*)((GlobalByte*)((GlobalWord*)p + uniform) + lane_bytes);
}
__device__ __forceinline__ Fr fr_load_lane(const uint32_t* p, size_t stride, size_t uniform, uint32_t lane_bytes) {
    Fr a;
#pragma unroll
    for (int k = 0; k < 8; ++k) a.l[k] = *at_lane(p, uniform + k * stride, lane_bytes);
    return a;
}
template <int STEP, int AT>
__device__ __forceinline__ Fr fr_load_row(const uint4* table, uint32_t r) {
    const GlobalVec4* rows = (const GlobalVec4*)table;
    const Vec4 lo = rows[(size_t)STEP * r + AT], hi = rows[(size_t)STEP * r + AT + 1];
    return Fr{{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w}};
}

// The sixteen words of block b of one leaf, as the hash takes them.  Elements are
// asked for one block ahead, row numbers two: a block is some thousand instructions
// during which the loads can be on the way.
template <int MODE>
struct LeafBlocks {
    VecLeavesJob job;
    uint32_t lane_bytes;  // four times the leaf's number: there are at most 2^24 leaves
    uint32_t cnt;
    bool live;            // lanes past the last leaf read what the last one reads and write nothing
    uint32_t next0, next1;  // row numbers of the two elements after those held
    Fr x0, x1;              // with rows: in the words of the hash (y: the elements themselves)
    Fr y0, y1;

    __device__ __forceinline__ uint32_t row_number(uint32_t i) const {
        if (MODE == kLeafPlain) return 0u;
        if (MODE == kLeafRowsHash && !job.from.rows) return i * (uint32_t)job.L + lane_bytes / 4;  // the table's own rows
        return *at_lane(job.from.rows, i * job.L, lane_bytes);
    }
    __device__ __forceinline__ uint32_t in_table(uint32_t row) const { return row < job.from.N ? row : 0u; }
    __device__ __forceinline__ void fetch(Fr& x, Fr& y, uint32_t i, uint32_t row) {
        if constexpr (MODE == kLeafPlain) {
            x = fr_load_lane(job.v, job.stride, i * job.L, lane_bytes);
        } else if constexpr (MODE == kLeafRowsHash) {
            x = fr_load_row<1, 0>(job.from.B, in_table(row) * (uint32_t)job.from.hash_only);
        } else {
            y = fr_load_row<4, 0>(job.from.B, in_table(row));
            x = fr_load_row<4, 2>(job.from.B, in_table(row));
        }
    }
    // A's element on its way to memory
    __device__ __forceinline__ void write(const Fr& x, uint32_t i) {
        if (MODE == kLeafPlain || MODE == kLeafRowsHash || !live) return;
#pragma unroll
        for (int k = 0; k < 8; ++k) *at_lane(job.v, i * job.L + k * job.stride, lane_bytes) = x.l[k];
    }
    __device__ __forceinline__ void words(uint32_t* w, const Fr& el) {
        const Fr x = MODE == kLeafPlain ? fr_from_mont(el) : el;
#pragma unroll
        for (int k = 0; k < 8; ++k) w[k] = MODE == kLeafPlain ? __builtin_bswap32(x.l[k]) : x.l[k];
    }

    __device__ __forceinline__ void begin(const VecLeavesJob& j, size_t which) {
        job = j;
        live = which < j.L;
        lane_bytes = (uint32_t)(live ? which : j.L - 1) * 4;
        cnt = (uint32_t)(j.n / j.L);  // kVecLeaf, or all n (a power of two) when n < kVecLeaf
        const uint32_t last = cnt - 1;  // short vectors: places past the end read the last element again
        const uint32_t row0 = row_number(0), row1 = row_number(last < 1 ? last : 1);
        next0 = row_number(last < 2 ? last : 2);
        next1 = row_number(last < 3 ? last : 3);
        fetch(x0, y0, 0, row0);
        fetch(x1, y1, last < 1 ? last : 1, row1);
    }
    __device__ __forceinline__ uint32_t blocks() const { return cnt / 2 + 1; }  // the last holds the padding
    // The words of elements 2b and 2b+1; what follows is asked for before work() runs (the
    // block's rounds, or the making of its schedule).
    template <class Work>
    __device__ __forceinline__ void data_block(uint32_t (&w)[16], uint32_t b, Work&& work) {
        write(y0, 2 * b);
        write(y1, 2 * b + 1);
        words(w, x0);
        words(w + 8, x1);
        // past the end: the last two again
        const uint32_t end = cnt - 2, i = 2 * b + 2 < end ? 2 * b + 2 : end, ii = i + 2 < end ? i + 2 : end;
        fetch(x0, y0, i, next0);
        fetch(x1, y1, i + 1, next1);
        next0 = row_number(ii);
        next1 = row_number(ii + 1);
        __builtin_amdgcn_sched_barrier(0);  // asked for here, not where they are used
        work();
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ void last_block(uint32_t (&w)[16]) {
        if (cnt == 1) {  // a vector of one element shares its block with the padding
            write(y0, 0);
            words(w, x0);
        }
        const int pad = cnt == 1 ? 8 : 0;
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (k >= pad) w[k] = k == pad ? 0x80000000u : k == 15 ? cnt * 256u : 0u;
    }
};

__device__ __forceinline__ const VecLeavesJob& leaves_job(const VecLeavesArgs& args, uint32_t group) {
    int q = 0;
    while (q + 1 < args.njobs && group >= args.job[q + 1].first_group) ++q;
    return args.job[q];
}

__device__ __forceinline__ void leaves_done(const VecLeavesArgs& args) {
    if (args.seq == 0) return;
    __syncthreads();
    if (threadIdx.x == 0 && atomicAdd(args.ticket, 1u) == gridDim.x - 1) {
        *args.ticket = 0;
        bad_words_publish(args.bad);
        mailbox_publish(args.words, args.seq);
    }
}

// Many leaves: one lane does all of a leaf.  Bound by instruction issue.
template <int MODE>
__device__ __forceinline__ void leaf_by_lane(const VecLeavesJob& job, size_t leaf) {
    LeafBlocks<MODE> src;
    src.begin(job, leaf);
    uint32_t h[8];
    sha256_init(h);
    uint32_t w[16];
#pragma unroll 1
    for (uint32_t b = 0; b + 1 < src.blocks(); ++b) {
        uint32_t s[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) s[i] = h[i];
        src.data_block(w, b, [&] { sha256_rounds<0, 64>(s, w); });
#pragma unroll
        for (int i = 0; i < 8; ++i) h[i] += s[i];
    }
    src.last_block(w);
    sha256_compress(h, w);
#pragma unroll
    for (int k = 0; k < 8; ++k) job.out[leaf * 8 + k] = h[k];
    if (job.to_host) mailbox_written();
}

// MODE: of the jobs that have rows, but for those of which only the hash is asked for (kLeafRowsHash:
// there are no others).
template <int MODE>
static __global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4, 8))) k_vec_leaves(VecLeavesArgs args) {
    const VecLeavesJob& job = leaves_job(args, blockIdx.x);
    const size_t leaf = (size_t)(blockIdx.x - job.first_group) * 64 + threadIdx.x;
    if (leaf < job.L) {
        if (MODE != kLeafPlain && job.from.hash_only) leaf_by_lane<kLeafRowsHash>(job, leaf);
        else if (MODE != kLeafPlain && MODE != kLeafRowsHash && job.from.rows) leaf_by_lane<MODE>(job, leaf);
        else leaf_by_lane<kLeafPlain>(job, leaf);
    }
    leaves_done(args);
}

// Few leaves: what counts is the length of one leaf's chain, some 1750 instructions
// per block with conversion and message schedule.  Two wavefronts share it: the
// second makes the schedule of the next block (loads, conversion, expansion, round
// constants added) in LDS while the first does the rounds of the current one, so that
// a block costs the rounds' 900 instructions.  A workgroup is two such pairs, one
// wavefront per SIMD: two workgroups of one pair each were seen to share two SIMDs and
// leave two idle.  Measured at 2^20 elements (8192 leaves): 220 -> 140 us.  Above
// kPipedLeafGroups the wavefronts share SIMDs.  Where every element is converted first, whose long
// chain one wavefront per SIMD waits out, the pairs are still ahead at 1032 groups (520 groups without
// rows: 408 us, in pairs 235).  Beyond 1040, whole verifications by lane and in pairs, when nothing shared
// their launch: 2^24 entries 1.05 and 1.02 ms, 2^25 1.70 and 1.70.
//
// Where the words come ready (kLeafRowsHash), one tensor's leaves or several's, us by lane and in pairs:
//   513 to 675 groups 178 to 181 and 200 to 204; 770 to 997 by lane 182 to 188 or, in most runs, 316 to 341
//   (wavefronts meet on SIMDs while others idle), in pairs 203 to 209; 1025 to 1476 323 to 332 and 294 to 311;
//   1538 326 and 387, 1667 325 and 404 (three workgroups of pairs per compute unit are 1536 groups); 2050
//   473 and 469, 2563 478 and 551, 3074 636 and 637.
static const uint32_t kPipedLeafGroups = 512, kPipedLeafGroupsConverting = 1040;
static const uint32_t kPipedLeafGroupsHashFrom = 768, kPipedLeafGroupsHash = 1536;
template <int MODE>
static bool leaves_in_pairs(uint32_t groups) {
    if (MODE == kLeafRowsHash && groups > kPipedLeafGroupsHashFrom) return groups <= kPipedLeafGroupsHash;
    return groups <= (MODE == kLeafPlain ? kPipedLeafGroupsConverting : kPipedLeafGroups);
}

// The second wavefront's part: the schedules of all blocks of its lanes' leaves.
template <int MODE>
__device__ __forceinline__ void leaf_schedules(const VecLeavesJob& job, bool live, size_t leaf, uint32_t blocks, uint32_t steps,
                                               uint4 (*kw)[16][64]) {
    const int lane = threadIdx.x & 63;
    LeafBlocks<MODE> src;
    if (live) src.begin(job, leaf);
    for (uint32_t b = 0; b <= steps; ++b) {  // one barrier more than blocks, as the wavefront of the rounds takes
        if (b < blocks) {
            uint32_t w[16];
            const auto schedule = [&] {
#pragma unroll
                for (int g = 0; g < 16; ++g) {
                    if (g >= 4) sha256_schedule4(w, 4 * g);
                    const int i = (4 * g) & 15;
                    kw[b & 1][g][lane] = make_uint4(w[i] + kShaK[4 * g], w[i + 1] + kShaK[4 * g + 1], w[i + 2] + kShaK[4 * g + 2],
                                                    w[i + 3] + kShaK[4 * g + 3]);
                }
            };
            if (b + 1 < blocks) {
                src.data_block(w, b, schedule);
            } else {
                src.last_block(w);
                schedule();
            }
        }
        __syncthreads();
    }
}

typedef uint4 PipedSchedules[2][2][16][64];  // [pair][buffer][four rounds][lane]
template <int MODE>
__device__ __forceinline__ void piped_leaves(const VecLeavesArgs& args, uint32_t block, PipedSchedules& kw) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), pair = wave >> 1;
    const bool rounds = (wave & 1) == 0;
    // both pairs take the same number of barriers: as many as the longer leaf of the two needs
    const uint32_t group = 2 * block + pair, other = 2 * block + (pair ^ 1);
    const bool live = group < args.groups;
    const VecLeavesJob& job = leaves_job(args, live ? group : args.groups - 1);
    const VecLeavesJob& job2 = leaves_job(args, other < args.groups ? other : args.groups - 1);
    const uint32_t blocks = live ? (uint32_t)(job.n / job.L) / 2 + 1 : 0;
    const uint32_t blocks2 = other < args.groups ? (uint32_t)(job2.n / job2.L) / 2 + 1 : 0;
    const uint32_t steps = blocks > blocks2 ? blocks : blocks2;
    const size_t leaf = (size_t)(group - job.first_group) * 64 + lane;
    if (rounds) {
        uint32_t h[8];
        sha256_piped_rounds(h, kw[pair], blocks, steps);
        if (live && leaf < job.L) {
#pragma unroll
            for (int k = 0; k < 8; ++k) job.out[leaf * 8 + k] = h[k];
            if (job.to_host) mailbox_written();
        }
    } else {
        if (MODE != kLeafPlain && job.from.hash_only) leaf_schedules<kLeafRowsHash>(job, live, leaf, blocks, steps, kw[pair]);
        else if (MODE != kLeafPlain && MODE != kLeafRowsHash && job.from.rows) leaf_schedules<MODE>(job, live, leaf, blocks, steps, kw[pair]);
        else leaf_schedules<kLeafPlain>(job, live, leaf, blocks, steps, kw[pair]);
    }
}
template <int MODE>
static __global__ void __launch_bounds__(256) k_vec_leaves_piped(VecLeavesArgs args) {
    __shared__ PipedSchedules kw;
    piped_leaves<MODE>(args, blockIdx.x, kw);
    leaves_done(args);
}

// A verification's leaves in pairs, and in the same launch what does not depend on them: the leaves of m
// and the first stage of the evaluations, which reads all that the tensors hold.  A leaf's chain keeps one
// wavefront per SIMD and takes its 230 us whatever runs in the other places: half of a compute unit's
// LDS is a workgroup's here, so that one of the evaluation's has room beside one of the hash's, and
// reads in the chain's time what took 60 us after it.  A verification of 2^22 entries in 2^16 rows against
// all tensors: 502 -> 421 us.  Also where a lane per leaf is as fast for the hash by itself: 2^24 entries 1031 -> 798
// us, 2^25 1682 -> 1480, 2^26 2997 -> 2761.  The leaves come first: with the others spread among them
// where not all are resident at once 2^24 entries take 1966 us.
struct LeavesBesideArgs {
    VecLeavesArgs leaves;
    LeafDigestJob counts;  // m's; nleaves 0: none
    uint32_t count_blocks;
    MleStageArgs stage;    // publishes nothing
};
static __global__ void __launch_bounds__(kBlock) k_leaves_beside(LeavesBesideArgs args) {
    __shared__ union {
        PipedSchedules kw;
        MleParts part;
    } sh;
    static_assert(sizeof(PipedSchedules) == sizeof(MleParts) && kBlock == 256, "");
    const uint32_t leaf_blocks = (args.leaves.groups + 1) / 2;
    uint32_t block = blockIdx.x;
    if (block < leaf_blocks) {
        piped_leaves<kLeafPlain>(args.leaves, block, sh.kw);
        return;
    }
    block -= leaf_blocks;
    if (block < args.count_blocks) {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), pair = wave >> 1;
        count_leaves(args.counts, 128 * block + 64 * pair, count_leaf_blocks(args.counts), (wave & 1) == 0, sh.kw[pair]);
        return;
    }
    mle_stage_block(args.stage, block - args.count_blocks, sh.part);
}

// A by row, S (or integers) compared with T's rows: a thread per element, blockIdx.y the instance.
struct MakeAJob {
    uint32_t* A;
    size_t stride, D;
    LeafGather from;  // B: four uint4 per row
    int check;        // kLeafRows, kLeafRowsCheck, kLeafRowsInts
};
static const size_t kMadeApart = (size_t)1 << 18;
template <int NT>
struct MakeAJobs {
    MakeAJob job[NT];
    SmallSource ints;
};
template <int NT>
static __global__ void __launch_bounds__(kBlock) k_make_a(MakeAJobs<NT> jobs) {
    const MakeAJob& g = jobs.job[NT == 1 ? 0 : blockIdx.y];
    for (size_t i = blockIdx.x * (size_t)kBlock + threadIdx.x; i < g.D; i += (size_t)gridDim.x * kBlock) {
        const uint32_t row = g.from.rows[i], r = row < g.from.N ? row : 0u;
        fr_store(g.A, g.stride, i, fr_load_row<4, 0>(g.from.B, r));
        if (g.check == kLeafRows) continue;
        const Fr t = fr_load_row<2, 0>(g.from.T, r);
        Fr s;
        if (g.check == kLeafRowsInts) small_source_load(s.l, jobs.ints, i);
        else s = fr_load(g.from.S, g.from.ss, i);
        uint32_t diff = row ^ r;
#pragma unroll
        for (int k = 0; k < 8; ++k) diff |= s.l[k] ^ t.l[k];
        if (diff) atomicMin(g.from.bad, (unsigned long long)i);
    }
}

// Very few leaves: a leaf is a chain of 65 blocks, 140 us here whatever their number, and
// 3 us on a host with SHA instructions, two at a time.  A thread makes, converts and checks
// one element as above and writes its bytes to pinned host memory (`out`), one leaf's
// after another's; the host hashes them (vec_digest_finish).  `first_group` and `groups`
// count elements here.  Measured, whole proofs with hints: 2^10 entries in 2^8 rows (10
// leaves) 425 -> 300 us, 2^11 in 2^11 (32 leaves) 467 -> 367; verifying the former 260 ->
// 141.  32 leaves are what the digests' part of the pinned memory holds.
static const size_t kHostLeaves = 32;
template <int MODE>
static __global__ void __launch_bounds__(kBlock) k_leaves_to_host(VecLeavesArgs args) {
    const uint32_t g = blockIdx.x * kBlock + threadIdx.x;
    if (g < args.groups) {
        const VecLeavesJob& job = leaves_job(args, g);
        const size_t i = g - job.first_group;
        Fr x;
        if (MODE != kLeafPlain && job.from.rows) {
            const uint32_t row = job.from.rows[i], r = row < job.from.N ? row : 0u;
            fr_store(job.v, job.stride, i, fr_load_row<4, 0>(job.from.B, r));
            x = fr_load_row<4, 2>(job.from.B, r);
#pragma unroll
            for (int k = 0; k < 8; ++k) x.l[k] = __builtin_bswap32(x.l[k]);
            if constexpr (MODE >= kLeafRowsCheck) {
                const Fr t = fr_load_row<2, 0>(job.from.T, r);
                Fr s;
                if constexpr (MODE == kLeafRowsInts) small_source_load(s.l, args.ints, i);
                else s = fr_load(job.from.S, job.from.ss, i);
                uint32_t diff = row ^ r;
#pragma unroll
                for (int k = 0; k < 8; ++k) diff |= s.l[k] ^ t.l[k];
                if (diff) atomicMin(job.from.bad, (unsigned long long)i);
            }
        } else {
            x = fr_from_mont(fr_load(job.v, job.stride, i));
        }
        const size_t cnt = job.n / job.L, leaf = i % job.L, at = i / job.L;
        uint4* out = (uint4*)job.out + 2 * (leaf * cnt + at);
        out[0] = make_uint4(x.l[0], x.l[1], x.l[2], x.l[3]);
        out[1] = make_uint4(x.l[4], x.l[5], x.l[6], x.l[7]);
        mailbox_written();
    }
    leaves_done(args);
}

// One step up the trees: workgroup b of a job reduces digests [b*chunk,
// (b+1)*chunk) of `in` to one (chunk a power of four, at most kTreeChunk) and writes
// it to out[8b..8b+8).  The last rows of a tree are the host's: a level costs some 8
// us here whatever its length (three dependent blocks), 64 digests cost the host 3.
static const uint32_t kTreeChunk = 1024;
static const uint32_t kTreeHostRow = 256;  // rows of at most this many digests go to the host

struct DigestTreeJob {
    const uint32_t* in;
    uint32_t* out;
    uint32_t chunk;
    uint32_t first_block;
    int to_host;  // as in VecLeavesJob
};
struct DigestTreeArgs {
    DigestTreeJob job[kDigestMaxJobs];
    int njobs;
    uint32_t* words;
    uint32_t* ticket;
    uint32_t seq;
    BadWords bad;
};

static __global__ void __launch_bounds__(kBlock) k_digest_tree(DigestTreeArgs args) {
    __shared__ uint32_t rows[2][kTreeChunk / 4 * 8];  // the row being read and the one being written (at most chunk/4 digests)
    int q = 0;
    while (q + 1 < args.njobs && blockIdx.x >= args.job[q + 1].first_block) ++q;
    const DigestTreeJob& job = args.job[q];
    const uint32_t b = blockIdx.x - job.first_block;
    // the first row comes from memory; every later one from LDS
    const uint32_t* base = job.in + (size_t)b * job.chunk * 8;
    uint32_t cnt = job.chunk;
    int cur = 0;
    bool from_lds = false;
    while (cnt > 1) {
        const uint32_t nodes = cnt / 4;
        for (uint32_t node = threadIdx.x; node < nodes; node += kBlock) {
            uint32_t h[8];
            sha256_init(h);
#pragma unroll 1
            for (uint32_t part = 0; part < 4; part += 2) {
                uint32_t w[16];
#pragma unroll
                for (int k = 0; k < 16; ++k) {
                    const uint32_t at = (node * 4 + part) * 8 + k;
                    w[k] = from_lds ? rows[cur][at] : base[at];
                }
                sha256_compress(h, w);
            }
            sha256_compress_padding(h, kShaPad128.kw);
#pragma unroll
            for (int k = 0; k < 8; ++k) rows[cur ^ 1][node * 8 + k] = h[k];
        }
        __syncthreads();
        cur ^= 1;
        from_lds = true;
        cnt = nodes;
    }
    if (threadIdx.x < 8) {
        job.out[(size_t)b * 8 + threadIdx.x] = from_lds ? rows[cur][threadIdx.x] : base[threadIdx.x];
        if (job.to_host) mailbox_written();
    }
    if (args.seq == 0) return;
    __syncthreads();
    if (threadIdx.x == 0 && atomicAdd(args.ticket, 1u) == gridDim.x - 1) {
        *args.ticket = 0;
        bad_words_publish(args.bad);
        mailbox_publish(args.words, args.seq);
    }
}

// ---- pooled eq tables ----------------------------------------------------------------

// `count` elements of nine 29-bit limbs in three planes: limbs 0..3 of element i
// as one uint4 at base[i], limbs 4..7 at base[count + i], limb 8 as a word at
// ((uint32_t*)(base + 2 count))[i] (a wavefront reads 1 KiB, 1 KiB and 256 B, each
// contiguous).  36 * count bytes.
struct Planes29 {
    uint4* base;
    size_t count;
};

__device__ __forceinline__ F29 planes29_load(const Planes29& a, size_t i) {
    const uint4 u = a.base[i], v = a.base[a.count + i];
    const uint32_t top = reinterpret_cast<const uint32_t*>(a.base + 2 * a.count)[i];
    return F29{{u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w, top}};
}

__device__ __forceinline__ void planes29_store(const Planes29& a, size_t i, const F29& x) {
    a.base[i] = make_uint4(x.l[0], x.l[1], x.l[2], x.l[3]);
    a.base[a.count + i] = make_uint4(x.l[4], x.l[5], x.l[6], x.l[7]);
    reinterpret_cast<uint32_t*>(a.base + 2 * a.count)[i] = x.l[8];
}

// Table q covers variables [var0, var0 + nvars) of the point and occupies
// elements [offset, offset + 2^nvars) of the pool.  Tables marked `scaled` are
// the weights of the rounds on 29-bit limbs: their entries are multiplied by
// `scale` and go, as nine 29-bit limbs, into a pool of their own (three planes of
// `count29` elements, see Planes29) at offset - first29.
struct EqPoolArgs {
    Fr u[32];
    uint32_t offset[64];
    uint8_t var0[64];
    uint8_t nvars[64];
    uint8_t scaled[64];
    Fr scale;
    int ntables;
    uint32_t total;
    uint4* pool29;
    size_t count29;
    uint32_t first29;
};

// Four lanes per entry, each multiplying up a quarter of its factors: a chain of five
// products for twelve variables, and the coordinates are loaded ahead of it.  (One lane
// per entry waited for a load before each of the twelve: the tables of 25 variables 15.5 us,
// 10.4 so, those of 10 variables 18.5, 13.5 so.)
__device__ __forceinline__ Fr quad_product(const Fr& v) {
    Fr a = v, o;
#pragma unroll
    for (int k = 0; k < 8; ++k) o.l[k] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)a.l[k], 0xb1, 0xf, 0xf, true);  // 1 0 3 2
    a = fr_mul(a, o);
#pragma unroll
    for (int k = 0; k < 8; ++k) o.l[k] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)a.l[k], 0x4e, 0xf, 0xf, true);  // 2 3 0 1
    return fr_mul(a, o);
}

static __global__ void __launch_bounds__(kBlock) k_eq_pool(uint32_t* __restrict__ pool, size_t stride, EqPoolArgs args) {
    const Fr one = fr_one();
    const int part = threadIdx.x & 3;
    for (uint32_t g = (blockIdx.x * kBlock + threadIdx.x) >> 2; g < args.total; g += gridDim.x * (kBlock / 4)) {
        // the wavefront's first entry's table by scalar loads, from there each lane its own
        const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)g);
        int q = 0;
        while (q + 1 < args.ntables && args.offset[q + 1] <= first) ++q;
        while (q + 1 < args.ntables && args.offset[q + 1] <= g) ++q;
        const uint32_t x = g - args.offset[q];
        const int nv = args.nvars[q], v0 = args.var0[q];
        const bool scaled = args.scaled[q] != 0;
        Fr acc = scaled && part == 0 ? args.scale : one;
        bool started = scaled && part == 0;
        for (int t = part; t < nv; t += 4) {
            const Fr u = args.u[v0 + t];
            const Fr f = (x >> (nv - 1 - t)) & 1u ? u : fr_sub(one, u);
            acc = started ? fr_mul(acc, f) : f;
            started = true;
        }
        acc = quad_product(acc);
        if (scaled) {
            const F29 v = f29_unpack(acc.l);
            const size_t i = g - args.first29;
            if (part == 0) args.pool29[i] = make_uint4(v.l[0], v.l[1], v.l[2], v.l[3]);
            else if (part == 1) args.pool29[args.count29 + i] = make_uint4(v.l[4], v.l[5], v.l[6], v.l[7]);
            else if (part == 2) reinterpret_cast<uint32_t*>(args.pool29 + 2 * args.count29)[i] = v.l[8];
        } else if (part == 0) {
            fr_store(pool, stride, g, acc);
        }
    }
}
static inline void launch_eq_pool(uint32_t* pool, size_t stride, const EqPoolArgs& args, hipStream_t stream) {
    hipLaunchKernelGGL(k_eq_pool, dim3(grid_for((size_t)args.total * 4)), dim3(kBlock), 0, stream, pool, stride, args);
}

// ---- sumcheck rounds ---------------------------------------------------------------------

// Weights of a round: the pair with index p (the remaining variables after the
// one being bound) has weight lo[p & (2^lbits - 1)] * hi[p >> lbits]; `hi` is
// null when the low table covers every remaining variable.
struct EqSplit {
    const uint32_t* pool;
    size_t stride;
    uint32_t lo_off;
    uint32_t hi_off;
    int lbits;
    int has_hi;
};

struct PairArray {
    const uint32_t* src;
    size_t ss;
    uint32_t* dst;
    size_t ds;
};

// Loads the pair (x0, x1) of index p for this round.  Without folding the
// array has 2*half entries.  With folding it has 4*half: the previous variable
// is bound to r first (r is wave-uniform), the folded entries are written back
// (to dst) and returned.
template <bool FOLD, bool STORE = true>
__device__ __forceinline__ void load_pair(const PairArray& a, size_t p, size_t half, const Fr& r, Fr& x0, Fr& x1) {
    if constexpr (!FOLD) {
        x0 = fr_load(a.src, a.ss, p);
        x1 = fr_load(a.src, a.ss, p + half);
    } else {
        {
            Fr y0 = fr_load(a.src, a.ss, p), y2 = fr_load(a.src, a.ss, p + 2 * half);
            x0 = fr_fold(y0, y2, r);
        }
        if constexpr (STORE) fr_store(a.dst, a.ds, p, x0);
        {
            Fr y1 = fr_load(a.src, a.ss, p + half), y3 = fr_load(a.src, a.ss, p + 3 * half);
            x1 = fr_fold(y1, y3, r);
        }
        if constexpr (STORE) fr_store(a.dst, a.ds, p + half, x1);
    }
}

struct DataRoundArgs {
    PairArray A, S;
    size_t half;        // pairs in this round
    size_t block_span;  // pairs per workgroup (power of two, at most 2^eq.lbits when eq.has_hi)
    Fr r_prev, beta;
    EqSplit eq;
    uint32_t* partials;  // 5 values per workgroup
    size_t pstride;
    SmallSource ints;    // ints.x not null (first round only): S is given as small integers
};

// Data side of one round.  With w the weight of a pair and (A0, A1), (S0, S1)
// its entries, the sums are
//   q0 = w A0 (S0+beta), q1 = w A1 (S1+beta), qinf = w (A1-A0)(S1-S0), sA0 = A0, sA1 = A1,
// from which the host forms  alpha c e~(u_k, X) q(X) + sA(X).
//
// FOLD = false is the first round, straight after the inversion: there
// A_i (S_i + beta) = 1 for every i, so q0 = q1 = sum of the weights = 1 and only
// qinf and the sums of A are computed (q0 and q1 stay zero and are set by the
// host).
// The three weighted sums are sums of products: they are accumulated as
// unreduced 512-bit integers, in registers, and reduced once per thread.
struct WideInRegs {
    FrWide w[3];
    __device__ __forceinline__ void clear() {
        w[0] = fr_wide_zero();
        w[1] = fr_wide_zero();
        w[2] = fr_wide_zero();
    }
    __device__ __forceinline__ void mac(int which, const Fr& a, const Fr& b) { fr_wide_mac(w[which], a, b); }
    __device__ __forceinline__ Fr finish(int which) const { return fr_wide_reduce(w[which]); }
};

template <bool FOLD, class Wide>
__device__ __forceinline__ void data_pair(const DataRoundArgs& g, size_t p, size_t lo_mask, Wide& wide, Fr& sA0, Fr& sA1) {
    Fr a0, a1, s0, s1;
    load_pair<FOLD>(g.A, p, g.half, g.r_prev, a0, a1);
    if (!FOLD && g.ints.x) {
        small_source_load(s0.l, g.ints, p);
        small_source_load(s1.l, g.ints, p + g.half);
    } else {
        load_pair<FOLD>(g.S, p, g.half, g.r_prev, s0, s1);
    }
    Fr w = fr_load(g.eq.pool, g.eq.stride, g.eq.lo_off + (p & lo_mask));
    sA0 = fr_add(sA0, a0);
    sA1 = fr_add(sA1, a1);
    if constexpr (FOLD) {
        Fr wa0 = fr_mul(w, a0), wa1 = fr_mul(w, a1);
        wide.mac(0, wa0, fr_add(s0, g.beta));
        wide.mac(1, wa1, fr_add(s1, g.beta));
        wide.mac(2, fr_sub(wa1, wa0), fr_sub(s1, s0));
    } else {
        wide.mac(2, w, fr_mul(fr_sub(a1, a0), fr_sub(s1, s0)));
    }
}

// One workgroup's share of the data side: block_span consecutive pairs, which
// all share the high-variable factor of their weight; it is applied once to the
// workgroup's sums.
template <bool FOLD>
__device__ __forceinline__ void round_data_block(const DataRoundArgs& g, unsigned block, uint32_t* lds) {
    WideInRegs wide;
    wide.clear();
    Fr tot[5];
    tot[3] = fr_zero();
    tot[4] = fr_zero();
    const size_t start = block * g.block_span;
    const size_t lo_mask = ((size_t)1 << g.eq.lbits) - 1;
    for (size_t p = start + threadIdx.x; p < start + g.block_span; p += kBlock)
        data_pair<FOLD>(g, p, lo_mask, wide, tot[3], tot[4]);
    tot[0] = FOLD ? wide.finish(0) : fr_zero();
    tot[1] = FOLD ? wide.finish(1) : fr_zero();
    tot[2] = wide.finish(2);
    block_sum<5, 4>(tot, lds);
    if (threadIdx.x == 0) {
        if (g.eq.has_hi) {
            Fr hf = fr_load(g.eq.pool, g.eq.stride, g.eq.hi_off + (start >> g.eq.lbits));
            if constexpr (FOLD) {
                tot[0] = fr_mul(tot[0], hf);
                tot[1] = fr_mul(tot[1], hf);
            }
            tot[2] = fr_mul(tot[2], hf);
        }
#pragma unroll
        for (int q = 0; q < 5; ++q) fr_store(g.partials, g.pstride, (size_t)block * 5 + q, tot[q]);
    }
}

// The first round: 128 bytes per pair for two multiplications, bound by HBM.  (The
// large folding rounds after it are in tlookup_round29.h; round_data_block<true>
// serves the rounds that also bind a table variable.)
static __global__ void __launch_bounds__(kBlock) k_round_data0(DataRoundArgs g) {
    __shared__ uint32_t lds[4 * 6 * 8];
    round_data_block<false>(g, blockIdx.x, lds);
}

struct TableRoundArgs {
    PairArray B, T, M;
    size_t half;
    size_t block_span;
    Fr r_prev, beta;
    EqSplit eq;
    uint32_t* partials;  // 6 values per workgroup
    size_t pstride;
};

// Table side of one round (once the table's own variables are being bound):
//   t0 = w B0 (T0+beta), t1 = w B1 (T1+beta), tinf = w (B1-B0)(T1-T0),
//   m0 = B0 M0, m1 = B1 M1, minf = (B1-B0)(M1-M0).
// The two groups of sums share only B, so they can be computed by different
// threads (PART 1: the T sums, PART 2: the m sums, PART 0: both), which halves the
// dependent chain of multiplications in the rounds that are bound by latency.
// For that B is folded from one buffer into another (both parts read the
// unfolded entries; only PART 0 and PART 1 store the folded ones).
template <bool FOLD, int PART>
__device__ __forceinline__ void table_pair(const TableRoundArgs& g, size_t p, size_t lo_mask, Fr (&tot)[6]) {
    Fr b0, b1;
    load_pair<FOLD, PART != 2>(g.B, p, g.half, g.r_prev, b0, b1);
    if constexpr (PART != 1) {
        Fr m0, m1;
        load_pair<FOLD>(g.M, p, g.half, g.r_prev, m0, m1);
        tot[3] = fr_add(tot[3], fr_mul(b0, m0));
        tot[4] = fr_add(tot[4], fr_mul(b1, m1));
        tot[5] = fr_add(tot[5], fr_mul(fr_sub(b1, b0), fr_sub(m1, m0)));
    }
    if constexpr (PART != 2) {
        Fr t0, t1;
        load_pair<FOLD>(g.T, p, g.half, g.r_prev, t0, t1);
        Fr w = fr_load(g.eq.pool, g.eq.stride, g.eq.lo_off + (p & lo_mask));
        Fr wb0 = fr_mul(w, b0), wb1 = fr_mul(w, b1);
        tot[0] = fr_add(tot[0], fr_mul(wb0, fr_add(t0, g.beta)));
        tot[1] = fr_add(tot[1], fr_mul(wb1, fr_add(t1, g.beta)));
        tot[2] = fr_add(tot[2], fr_mul(fr_sub(wb1, wb0), fr_sub(t1, t0)));
    }
}

template <bool FOLD, int PART>
__device__ __forceinline__ void round_table_block(const TableRoundArgs& g, unsigned block, uint32_t* lds) {
    Fr tot[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) tot[q] = fr_zero();
    const size_t start = block * g.block_span;
    const size_t lo_mask = ((size_t)1 << g.eq.lbits) - 1;
    for (size_t p = start + threadIdx.x; p < start + g.block_span; p += kBlock)
        table_pair<FOLD, PART>(g, p, lo_mask, tot);
    block_sum<6, 4>(tot, lds);
    if (threadIdx.x == 0) {
        if (PART != 2 && g.eq.has_hi) {
            Fr hf = fr_load(g.eq.pool, g.eq.stride, g.eq.hi_off + (start >> g.eq.lbits));
            tot[0] = fr_mul(tot[0], hf);
            tot[1] = fr_mul(tot[1], hf);
            tot[2] = fr_mul(tot[2], hf);
        }
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const bool mine = PART == 0 || (PART == 1 ? q < 3 : q >= 3);
            if (mine) fr_store(g.partials, g.pstride, (size_t)block * 6 + q, tot[q]);
        }
    }
}

template <bool FOLD>
static __global__ void __launch_bounds__(kBlock) k_round_table(TableRoundArgs g) {
    __shared__ uint32_t lds[4 * 6 * 8];
    round_table_block<FOLD, 0>(g, blockIdx.x, lds);
}

// A round that binds one of the table's variables, all of it in one launch:
// workgroups with blockIdx.y = 0 do the data side, 1 the T sums and 2 the m sums
// of the table side.  The data arrays have been folded at least once by then.
template <bool FOLD_T>
static __global__ void __launch_bounds__(kBlock) k_round_both(DataRoundArgs d, TableRoundArgs t) {
    __shared__ uint32_t lds[4 * 6 * 8];
    if (blockIdx.y == 0) round_data_block<true>(d, blockIdx.x, lds);
    else if (blockIdx.y == 1) round_table_block<FOLD_T, 1>(t, blockIdx.x, lds);
    else round_table_block<FOLD_T, 2>(t, blockIdx.x, lds);
}

// The table side's sum over the whole table, sum_j m_j B_j, while the host is busy with the
// digests.  (The other one, sum_j e'_j B_j (T_j + beta), is one: B is exact and the weights sum
// to one.)  Shares by workgroup: eight words at 8 blockIdx.x of `out`, pinned host memory, or
// (stride not zero) element step blockIdx.x of limb planes.
struct TableSumJob {
    const uint32_t* B;
    const uint32_t* M;
    size_t N;
    uint32_t* out;
    size_t stride;
    uint32_t step;
};
struct TableSumJobs {
    TableSumJob job[kMaxTables];  // by blockIdx.y
};
static __global__ void __launch_bounds__(kBlock) k_table_sum(TableSumJobs jobs) {
    __shared__ uint32_t lds[4 * 8];
    const TableSumJob& g = jobs.job[blockIdx.y];
    Fr sum[1] = {fr_zero()};
    for (size_t j = blockIdx.x * (size_t)kBlock + threadIdx.x; j < g.N; j += (size_t)gridDim.x * kBlock)
        sum[0] = fr_add(sum[0], fr_mul(fr_load(g.B, g.N, j), fr_load(g.M, g.N, j)));
    block_sum<1, 4>(sum, lds);
    if (threadIdx.x != 0) return;
    if (g.stride) {
        fr_store(g.out, g.stride, (size_t)blockIdx.x * g.step, sum[0]);
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) g.out[8 * blockIdx.x + k] = sum[0].l[k];
        mailbox_written();
    }
}

// Adds up a value's `count` partial sums, one workgroup per value.
static __global__ void __launch_bounds__(kBlock) k_long_total(const uint32_t* partials, size_t pstride, unsigned count, uint32_t* out_words,
                                                              uint32_t* words, uint32_t seq, uint32_t* ticket) {
    __shared__ uint32_t lds[4 * 8];
    Fr acc[1] = {fr_zero()};
    for (unsigned b = threadIdx.x; b < count; b += kBlock) acc[0] = fr_add(acc[0], fr_load(partials, pstride, (size_t)blockIdx.x * count + b));
    block_sum<1, 4>(acc, lds);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < 8; ++k) out_words[8 * blockIdx.x + k] = acc[0].l[k];
        mailbox_written();
        if (atomicAdd(ticket, 1u) == gridDim.x - 1) {
            *ticket = 0;
            mailbox_publish(words, seq);
        }
    }
}

// Final values: each of up to five arrays is either a single entry or a pair
// still to be bound to the last challenge.  Value q goes to out_words[8q..8q+8);
// `words` is the mailbox the flag lives in.
struct FinalArgs {
    const uint32_t* p[8];
    size_t stride[8];
    int fold[8];
    int count;
    Fr r;
};

static __global__ void k_final_values(FinalArgs g, uint32_t* out_words, uint32_t* words, uint32_t seq) {
    int q = threadIdx.x;
    if (q < g.count) {
        Fr v = fr_load(g.p[q], g.stride[q], 0);
        if (g.fold[q]) v = fr_fold(v, fr_load(g.p[q], g.stride[q], 1), g.r);
#pragma unroll
        for (int k = 0; k < 8; ++k) out_words[8 * q + k] = v.l[k];
        mailbox_written();
    }
    __syncthreads();
    if (threadIdx.x == 0) mailbox_publish(words, seq);
}

}  // namespace zkmi

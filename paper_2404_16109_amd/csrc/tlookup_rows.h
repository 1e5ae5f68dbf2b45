// Data side of the long rounds of the tlookup sumcheck (Section 4, the second form of the
// identity) where every entry is a row of a table of up to 2^16 rows: S_i = T[row_i], and
// before any fold A_i = 1 / (beta + S_i) = B[row_i].  Until a challenge binds a variable
// neither needs to exist as a vector: the first pass (k_first_two_rows, two rounds) and the
// pass that binds their challenges (k_round_pair<true>) read the row numbers and the table's
// rows, 64 bytes each, which the caches hold; A is never written at its full length.  From
// there on a pass binds the two variables of the pass before it and sums what the next two
// rounds need (k_round_pair<false>).
//
// Rows come straight into LDS, 64 positions ahead, four lanes to a row: no registers wait for
// them.  (The vector memory pipe takes about a line of 64 bytes per cycle and compute unit,
// whatever lanes ask for it: 2^25 rows of 64 bytes take 155 us through registers, 132 into LDS,
// as two rows of 32 bytes each 250.)
//
// Measured at 2^25 entries in 2^16 rows: the hash of A, which neither compares S nor writes A
// any more, 1089 -> 830 us; the first two rounds, which compare, 512 -> 580; rounds 2 to 8 in
// four passes, 1115 in seven -> 620; a proof 3419 -> 2658, of 2^23 entries from integers 1651 ->
// 1274, of 2^22 without hints 1179 -> 1059, of 2^20 in 2^8 rows 680 -> 614.
#pragma once
#include "tlookup_round29.h"

namespace zkmi {

// A wavefront's sums over its lanes of wa and sa, each of at most 64 entries below 1.015 r a lane: out(wa's, sa's) in its
// last lane, reduced.
template <class Out>
__device__ __forceinline__ void rows_line_sums(const F29& wa, const F29& sa, Out&& out) {
    const F29 w = f29_shrink(wave_sum29(f29_shrink(f29_normalize(wa)))), a = f29_shrink(wave_sum29(f29_shrink(f29_normalize(sa))));
    if ((threadIdx.x & 63) == 63) {
        Fr fw, fa;
        f29_canonical(fw.l, w);
        f29_canonical(fa.l, a);
        out(fw, fa);
    }
}

// ---- the first pass ---------------------------------------------------------------------
//
// The sums of k_round_first_two, whose DataRound01Args describe the weights and the places
// of the results.  What the entries are compared with while they are at hand: nothing (the
// rows are known to be right), the caller's S, or the caller's integers (SmallSource).
enum RowsCheck { kRowsTrusted = 0, kRowsCheckWords = 1, kRowsCheckInts = 2 };

struct FirstTwoRowsArgs {
    DataRound01Args sums;           // A and S unused, but for S with kRowsCheckWords
    const uint32_t* rows;           // row numbers
    const uint4* table;             // four uint4 per row: T's balanced digits, B's words (k_rows_of)
    uint32_t N;
    unsigned long long* bad;        // smallest i with S_i != T[row_i] or row_i >= N
    SmallSource ints;
};

// A word per lane from a uniform place.
template <class W>
__device__ __forceinline__ W lane_word(const W* p, size_t first) {
    typedef const __attribute__((address_space(1))) W* global;
    global q = (global)p + first;
    asm("" : "+s"(q));
    return q[threadIdx.x & 63];
}

// A batch of 64 rows in LDS: element e's at 64 e, its pieces (0, 1 T's digits, 2, 3 B's words) in an order
// that spreads lanes over the banks, whether each reads its own element's or (row_operand) a column of many.
__device__ __forceinline__ uint32_t row_swizzle(uint32_t e) { return 2 * ((e >> 2) & 1) + ((e >> 3) & 1); }

// The operand that pieces Q, Q + 1 of the batch's rows are, as outer_get.
template <int Q>
__device__ __forceinline__ OuterOperand row_operand(const uint8_t* batch) {
    const uint32_t lane = threadIdx.x & 63, e = 16 * (lane >> 5) + ((lane & 15) >> 1), piece = Q + ((lane >> 4) & 1);
    const uint32_t at = 64 * e + 16 * (piece ^ row_swizzle(e)) + 8 * (lane & 1);  // eight elements on, the swizzle's low bit turns
    OuterOperand o;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        typedef __attribute__((address_space(3))) v2i lds_v2i;
        const v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i*)(batch + 2048 * s + at));
        const v2i hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i*)(batch + 2048 * s + 512 + (at ^ 16)));
        o.half[s] = v4i{lo.x, lo.y, hi.x, hi.y};
    }
    return o;
}

// Two wavefronts share 64 positions, wavefront half h the entries 2 h and 2 h + 1 of A; each fetches their rows
// a batch ahead into the other of two areas, and multiplies its A's by everybody's S's.  (Half of the entries' sums fit
// a wavefront's registers with another beside it; all of them did not.)
template <int CHECK>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2, 2))) k_first_two_rows(FirstTwoRowsArgs args) {
    const DataRound01Args& g = args.sums;
    __shared__ FirstTwoShared<2 * 2 * 4 * 4096> sh;  // [area][positions][entry]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = wave & 1, first = 2 * half;
    uint8_t* const batches = sh.lds + 4 * 4096 * (wave >> 1);
    v16i acc[5];  // A's two entries against: each other's S, S at the other x_0 (two), at both others, and W
#pragma unroll
    for (int q = 0; q < 5; ++q) outer_clear(acc[q]);
    F29 sa0 = f29_zero(), sa1 = sa0;
    const size_t start = blockIdx.x * g.block_span, share = g.block_span / 2, end = start + ((wave >> 1) + 1) * share;
    const size_t lo_mask = ((size_t)1 << g.lbits) - 1;
    // Four lanes fetch a row; lane l of the k-th fetch a piece of the row of element 16 k + l / 4.
    const uint32_t fetch = 16 * ((lane & 3) ^ row_swizzle(lane >> 2));
    const uint32_t own = 64 * lane + 16 * (2 ^ row_swizzle(lane));  // B's first words in a batch; its second at own ^ 16, T's digits at own ^ 32, own ^ 48
    uint32_t row[2][4];
    uint32_t s[CHECK == kRowsCheckWords ? 2 : 1][8];
    int32_t ix[2], iy[2];
    uint32_t bad_at = 0xffffffffu;  // this lane's smallest entry at fault (there are at most 2^31)
    const auto ask_rows = [&](size_t p) {
        typedef const __attribute__((address_space(1))) uint32_t* global_words;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                global_words q = (global_words)args.rows + (first + c) * g.quarter + p + 16 * k;
                asm("" : "+s"(q));
                row[c][k] = q[lane >> 2];
            }
    };
    const auto ask = [&](size_t p, uint32_t to) {
        uint32_t most = 0;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int k = 0; k < 4; ++k) most = row[c][k] > most ? row[c][k] : most;
        if (__any(most >= args.N)) {  // (never of a call that succeeds)
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t i = (uint32_t)((first + c) * g.quarter + p) + 16 * k + (lane >> 2);
                    if (row[c][k] < args.N) continue;
                    if (i < bad_at) bad_at = i;
                    row[c][k] = 0;
                }
        }
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int k = 0; k < 4; ++k) load_to_lds(args.table, 64 * row[c][k] + fetch, to + 4096 * (first + c) + 1024 * k);
    };
    const auto ask_values = [&](size_t p) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if constexpr (CHECK == kRowsCheckWords) outer_load(s[c], g.S, g.ss, (first + c) * g.quarter + p);
            if constexpr (CHECK == kRowsCheckInts) {
                ix[c] = lane_word(args.ints.x, (first + c) * g.quarter + p);
                iy[c] = args.ints.y ? lane_word(args.ints.y, (first + c) * g.quarter + p) : 0;
            }
        }
    };
    size_t p = start + (wave >> 1) * share;  // of the wavefront's first lane
    ask_rows(p);
    const uint32_t place = lds_place(batches);
    ask(p, place);
    ask_rows(p + kOuterBatch < end ? p + kOuterBatch : p);
    ask_values(p);
    uint32_t turn = 0;
#pragma unroll 1
    for (; p < end; p += kOuterBatch, ++turn) {
        const size_t next = p + kOuterBatch < end ? p + kOuterBatch : p, after = next + kOuterBatch < end ? next + kOuterBatch : next;
        uint8_t* const batch = batches + (turn & 1) * 2 * 4 * 4096;
        vector_loads_done();
        __syncthreads();  // everybody's rows are there, and nobody reads those of the positions before any more
        if (p + kOuterBatch < end) {
            ask(next, place + ((turn & 1) ^ 1) * 2 * 4 * 4096);
            ask_rows(after);
        }
        const F29 w = planes29_load(g.weights, g.lo_off + ((p + lane) & lo_mask));
        if constexpr (CHECK != kRowsTrusted) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const uint8_t* const at = batch + 4096 * (first + c);
                const uint4 t0 = *reinterpret_cast<const uint4*>(at + (own ^ 32)), t1 = *reinterpret_cast<const uint4*>(at + (own ^ 48));
                uint32_t v[8], d[8];
                if constexpr (CHECK == kRowsCheckInts) {
                    small_combine32(v, ix[c], iy[c], args.ints);
                } else {
#pragma unroll
                    for (int k = 0; k < 8; ++k) v[k] = s[c][k];
                }
                balanced_digits(d, v);  // one to one
                const uint32_t t[8] = {t0.x, t0.y, t0.z, t0.w, t1.x, t1.y, t1.z, t1.w};
                uint32_t diff = 0;
#pragma unroll
                for (int k = 0; k < 8; ++k) diff = __builtin_amdgcn_bitop3_b32(d[k], t[k], diff, 0xbe);  // (d ^ t) | diff
                if (__any(diff != 0)) {
                    const uint32_t i = (uint32_t)((first + c) * g.quarter + p) + lane;
                    if (diff && i < bad_at) bad_at = i;
                }
            }
            ask_values(next);
            __builtin_amdgcn_sched_barrier(0);
        }
        const auto words29 = [&](const uint8_t* at) {
            const uint4 b0 = *reinterpret_cast<const uint4*>(at + own), b1 = *reinterpret_cast<const uint4*>(at + (own ^ 16));
            const uint32_t words[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
            return f29_unpack(words);
        };
        const F29 a0 = words29(batch + 4096 * first), a1 = words29(batch + 4096 * (first + 1));
        sa0 = f29_add(sa0, a0);
        sa1 = f29_add(sa1, a1);
        F29 x0, x1;
        f29_mul_two(x0, x1, a0, a1, w);  // below 1.015 r
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            uint8_t* const at = batch + 4096 * (first + c);
            uint32_t xw[8], d[8];
            f29_pack(xw, c == 0 ? x0 : x1);
            balanced_digits(d, xw);
            // the weighted A takes the place of B's words
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
            *reinterpret_cast<uint4*>(at + own) = make_uint4(d[0], d[1], d[2], d[3]);
            *reinterpret_cast<uint4*>(at + (own ^ 16)) = make_uint4(d[4], d[5], d[6], d[7]);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
            const OuterOperand xo = row_operand<2>(at);
            outer_mac(acc[0], xo, row_operand<0>(batch + 4096 * (first + (c ^ 1))));
            outer_mac(acc[1 + c], xo, row_operand<0>(batch + 4096 * ((first ^ 2) + c)));
            outer_mac(acc[3], xo, row_operand<0>(batch + 4096 * ((first ^ 2) + (c ^ 1))));
            outer_mac(acc[4], xo, outer_column(first + c));
        }
        if ((turn & 3) == 3) {
            sa0 = f29_normalize(sa0);
            sa1 = f29_normalize(sa1);
        }
    }
    if (CHECK != kRowsTrusted && bad_at != 0xffffffffu) atomicMin(args.bad, (unsigned long long)bad_at);
    first_two_line(sh.values, wave >> 1, first, sa0);
    first_two_line(sh.values, wave >> 1, first + 1, sa1);
    int* const sums = (int*)sh.lds;
    __syncthreads();
    outer_sums_clear<6>(sums);
    __syncthreads();
    outer_sums_add(sums, first_two_class(first, first + 1), acc[0]);
    outer_sums_add(sums, 0, acc[1]);
    outer_sums_add(sums, 1, acc[2]);
    outer_sums_add(sums, 4, acc[3]);
    outer_sums_add(sums, 5, acc[4]);
    __syncthreads();
    outer_values<6, 32, true>(sums, [&](int q, int column, const Fr& v) { first_two_value(sh.values, q, column, v); });
    __syncthreads();
    first_two_finish<2>(g, sh.values, start);
}

// ---- passes that bind two variables and serve the next two rounds -------------------------
//
// With y_d, d = 0..3, the entries of an array of 16 P at d 4P + i, the pass writes
//   x_i = sum_d e_d y_(d 4P + i),   e_d = e~(the last two challenges, d),  i < 4 P,
// and with x_c(p) = x_(c P + p), c = 2 t_0 + t_1, sums for the classes 3 a + b (a, b = 0, 1 or 2
// for mixed in the first and the second variable, as in link_long.h)
//   sum_p w_p A_c(p) (S_d(p) + beta)  over the pairs (c, d) of the class, and sum_p A_c(p).
// A workgroup takes `span` positions, 64 at a time: wavefront c folds the entries c of A on the
// matrix cores (a few constants per output, mfma_dev.h) and weights them, wavefront 4 + c those
// of S; then each multiplies A's c-th entries by two of S's four.
struct DigitPlanes {
    uint4* base;   // balanced digits 0..15 of element i at base[i], 16..31 at base[count + i]
    size_t count;
};

struct PairArgs {
    // <true>: by row
    const uint32_t* rows;
    const uint4* table;      // four uint4 per row: the digits of B's element, of T's (k_rows_of)
    uint32_t N;
    // A and S: read from (and without WORDS written to) planes
    DigitPlanes a, s;
    // WORDS: written as limb-major words
    uint32_t* aw;
    uint32_t* sw;
    size_t aws, sws;
    size_t P, span;
    Fr e[4];
    ToepBias bias;           // a multiple of r that lifts the folds above zero
    Planes29 weights;        // as in DataRound01Args, of the second round served
    uint32_t lo_off;
    int lbits, has_hi;
    const uint32_t* hi_pool;
    size_t hi_stride;
    uint32_t hi_off;
    Fr beta;
    uint32_t* partials;      // value q of workgroup b at q gridDim.x + b: nine classes (times 2^5), four sums of A
    size_t pstride;
};
static const int kPairValues = 13, kPairThreads = 512;

template <bool ROWS, bool WORDS>
__global__ void __launch_bounds__(kPairThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) k_round_pair(PairArgs g) {
    // per wavefront the entries that bind to 64 of one array (1 KiB per entry and tile of 32), then A's and S's operands;
    // first the constants' matrices, at the end the sums by class: just what two workgroups per compute unit have
    __shared__ __attribute__((aligned(16))) uint8_t lds[8 * 8192 + 8 * kOuterStage];
    static_assert(2 * sizeof lds <= 160 * 1024 && 8 * 8192 >= 9 * 4096 + 128, "");
    static_assert(4 * kOuterMaxSpan <= kOuterMaxProducts, "a position adds four products to the class that is mixed twice");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), c = wave & 3, i = lane & 31, h = lane >> 5;
    const bool is_s = wave >= 4;
    uint8_t* const raw = lds + (ROWS ? 16384 * c : 8192 * wave);  // by row A's and S's together, half of it fetched by either wavefront
    uint8_t* const ops = lds + 8 * 8192;
    const uint32_t place = lds_place(raw);
    if (threadIdx.x < 128) {
        uint32_t digits[8];
        toeplitz_column(digits, g.e[threadIdx.x >> 5], threadIdx.x & 31);
        toeplitz_store(lds + (threadIdx.x >> 5) * kToepBytes, digits, threadIdx.x & 31);
    }
    __syncthreads();
    v4i m[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) m[d] = reinterpret_cast<const v4i*>(lds)[d * 64 + lane];
    __syncthreads();
    const size_t P = g.P, start = blockIdx.x * g.span, end = start + g.span, lo_mask = ((size_t)1 << g.lbits) - 1;
    const DigitPlanes mine = is_s ? g.s : g.a;
    // By row four lanes fetch a row (see k_first_two_rows); the places that a lane's sixteen digits come from and are read at.
    const uint32_t fetch = 16 * ((lane & 3) ^ row_swizzle(lane >> 2));
    const uint8_t* const lane_from = (const uint8_t*)(mine.base + (h ? mine.count + i : (size_t)i));
    const uint32_t lane_at = ROWS ? 64 * i + 16 * (((is_s ? 2 : 0) + h) ^ row_swizzle(i)) : 16 * lane;
    constexpr int kEntry = ROWS ? 4096 : 2048, kTile = ROWS ? 2048 : 1024;
    uint32_t row[8];  // of the positions asked for next: two entries' 64
    const auto ask_rows = [&](size_t p) {
        typedef const __attribute__((address_space(1))) uint32_t* global_words;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            global_words q = (global_words)g.rows + (4 * ((is_s ? 2 : 0) + (k >> 2)) + c) * P + p + 16 * (k & 3);
            asm("" : "+s"(q));
            row[k] = q[lane >> 2];
        }
    };
    const auto ask = [&](size_t p) {
        if constexpr (ROWS) {
#pragma unroll
            for (int k = 0; k < 8; ++k) load_to_lds(g.table, 64 * (row[k] < g.N ? row[k] : 0u) + fetch, place + (is_s ? 8192 : 0) + 1024 * k);
        } else {
#pragma unroll
            for (int d = 0; d < 4; ++d)
#pragma unroll
                for (int j = 0; j < 2; ++j) load_to_lds(lane_from + 16 * ((4 * d + c) * P + p + 32 * j), place + 1024 * (2 * d + j));
        }
    };
    v16i acc[2];  // A's entries c against S's entries 0 and 1 (2 and 3: the wavefronts that fold S)
    outer_clear(acc[0]);
    outer_clear(acc[1]);
    F29 wa = f29_zero(), sa = f29_zero();
    if constexpr (ROWS) ask_rows(start);
    ask(start);
    if constexpr (ROWS) ask_rows(start + kOuterBatch < end ? start + kOuterBatch : start);
    vector_loads_done<ROWS ? 8 : 0>();  // (nothing has been stored yet)
    uint32_t turn = 0;
#pragma unroll 1
    for (size_t p = start; p < end; p += kOuterBatch, ++turn) {
        const size_t next = p + kOuterBatch < end ? p + kOuterBatch : p, after = next + kOuterBatch < end ? next + kOuterBatch : next;
        // the entries are there; what has been asked for and stored after them need not be
        vector_loads_done<(WORDS ? 8 : 2) + (ROWS ? 8 : 0)>();
        if constexpr (ROWS) __syncthreads();
        F29 w;
        if (!is_s) w = planes29_load(g.weights, g.lo_off + ((p + lane) & lo_mask));
        v16i fold[2];
        outer_clear(fold[0]);
        outer_clear(fold[1]);
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                fold[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(m[d], *reinterpret_cast<const v4i*>(raw + kEntry * d + kTile * j + lane_at),
                                                                fold[j], 0, 0, 0);
        lds_reads_done();
        if (!ROWS && p + kOuterBatch < end) ask(next);
        __syncthreads();  // nobody reads the entries, or the operands of the positions before, any more
        if (ROWS && p + kOuterBatch < end) ask(next);
        if constexpr (ROWS) ask_rows(after);
        const Fr v = toeplitz_finish(fold[0], fold[1], g.bias);
        uint32_t d[8];
        balanced_digits(d, v.l);
        const size_t at = c * P + p + lane;
        if constexpr (WORDS) {
            fr_store(is_s ? g.sw : g.aw, is_s ? g.sws : g.aws, at, v);
        } else {
            mine.base[at] = make_uint4(d[0], d[1], d[2], d[3]);
            mine.base[mine.count + at] = make_uint4(d[4], d[5], d[6], d[7]);
        }
        if (!is_s) {
            const F29 a = f29_unpack(v.l), x = f29_mul(a, w);  // below 1.015 r
            sa = f29_add(sa, a);
            wa = f29_add(wa, x);
            if ((turn & 3) == 3) {
                sa = f29_normalize(sa);
                wa = f29_normalize(wa);
            }
            uint32_t xw[8];
            f29_pack(xw, x);
            balanced_digits(d, xw);
        }
        outer_put(d, ops + wave * kOuterStage);
        __syncthreads();
        const OuterOperand xo = outer_get(ops + c * kOuterStage);
#pragma unroll
        for (int q = 0; q < 2; ++q) outer_mac(acc[q], xo, outer_get(ops + (4 + (is_s ? 2 : 0) + q) * kOuterStage));
    }
    __syncthreads();
    uint32_t(*const beta_w)[8] = (uint32_t(*)[8])(lds + 9 * 4096);  // beta W_c, W_c = sum w A_c; behind the sums
    if (!is_s) {
        rows_line_sums(wa, sa, [&](const Fr& w_c, const Fr& a_c) {
            const Fr f = fr_mul(w_c, g.beta);
#pragma unroll
            for (int k = 0; k < 8; ++k) beta_w[c][k] = f.l[k];
            fr_store(g.partials, g.pstride, (size_t)(9 + c) * gridDim.x + blockIdx.x, a_c);
        });
    }
    int* const sums = (int*)lds;
    __syncthreads();
    outer_sums_clear<9>(sums);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int d = (is_s ? 2 : 0) + q, hi = (c >> 1) == (d >> 1) ? c >> 1 : 2, lo = (c & 1) == (d & 1) ? c & 1 : 2;
        outer_sums_add(sums, 3 * hi + lo, acc[q]);
    }
    __syncthreads();
    outer_values<9, 32, false>(sums, [&](int q, int, const Fr& x) {
        // beta enters with the W_c whose entries the class takes
        const int hi = q / 3, lo = q % 3;
        Fr v = x;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if ((hi == 2 || hi == (k >> 1)) && (lo == 2 || lo == (k & 1))) {
                Fr f;
#pragma unroll
                for (int j = 0; j < 8; ++j) f.l[j] = beta_w[k][j];
                v = fr_add(v, f);
            }
        if (g.has_hi) v = fr_mul(v, fr_load(g.hi_pool, g.hi_stride, g.hi_off + (start >> g.lbits)));
        fr_store(g.partials, g.pstride, (size_t)q * gridDim.x + blockIdx.x, v);
    });
}

}  // namespace zkmi

// Data side of the large rounds of the tlookup sumcheck (Section 4, the second form
// of the identity; Section 3.3 for the protocol), on 29-bit limbs: the first pass,
// which serves the first two rounds (k_round_first_two, on the matrix cores), and
// the large folding rounds (k_round_data29, schedule in round29_dev.h).
//
// These kernels move data at close to the rate of a plain copy only if their
// arithmetic keeps up, so they run on fr29_dev.h's multiplier (one multiply-add per
// limb product, no carry folds, lazy sums) and compute only what cannot be had
// otherwise.  A folding round forms per pair the two folds of A and of S, the two
// weighted entries of A, and the sums q0 = sum w A0 (S0+beta), qinf = sum w (A1-A0)(S1-S0)
// and sA0 = sum A0; the round's other two sums, q1 and sA1, follow on the host from
// the running claim and from the previous round's sums of A.  The first of these
// rounds after k_round_first_two binds two variables at once (FOLD2).
//
// Arrays between such rounds hold 29-bit limbs, normalized but not reduced: every
// fold adds up to 2 r to the bound on the values (they start below r), which is
// why at most kMaxLazyRounds folds happen before a round writes fully reduced
// 32-bit words again.
#pragma once
#include "outer_dev.h"
#include "round29_dev.h"
#include "small_dev.h"
#include "tlookup_kernels.h"

namespace zkmi {

// One of the two arrays a round folds.  It arrives as eight planes of 32-bit
// words (fully reduced: the first of a run of such rounds) or in `planes`, and
// leaves in `planes` (in place) or as fully reduced words (the last of a run).
struct Array29 {
    const uint32_t* words_in;
    size_t ws_in;
    Planes29 planes;
    uint32_t* words_out;
    size_t ws_out;
};

struct DataRound29Args {
    Array29 A, S;
    size_t half;
    size_t block_span;
    // Which entry of a pair the sums are taken over: pair p consists of the entries p + off0 (whose folds feed q0 and
    // sA0) and p + off1; (off0, off1) = (0, half) sums the X = 0 side of the round, (half, 0) the X = 1 side.
    size_t off0, off1;
    F29 r_prev;  // the challenge times 2^261
    F29 r_first; // FOLD2: the challenge before it (the first round's), and the product of the two, times 2^261
    F29 r_both;
    F29 beta;    // times 2^256, like the vectors
    Planes29 weights;  // the pool of low weight tables, entries times 2^266 (a weighted entry then has the vectors' form)
    uint32_t lo_off;   // this round's table in it
    int lbits;
    int has_hi;        // the workgroup's pairs share one more factor, from the pool of 32-bit tables:
    const uint32_t* hi_pool;
    size_t hi_stride;
    uint32_t hi_off;
    uint32_t* partials;  // five values per workgroup: q0, (unused), qinf, sA0, (unused)
    size_t pstride;
    // INTS: S is given as small integers (small_dev.h) and folded from them
    const int32_t* sx;
    const int32_t* sy;      // may be null
    const SmallFold4* sf;   // device memory: the constants of the fold by r_prev
};

template <bool WORDS32>
__device__ __forceinline__ F29 array29_load(const Array29& a, size_t i) {
    if constexpr (WORDS32) {
        uint32_t w[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) w[k] = a.words_in[k * a.ws_in + i];
        return f29_unpack(w);
    } else {
        return planes29_load(a.planes, i);
    }
}

// x: normalized, below 2^261.
template <bool WORDS32>
__device__ __forceinline__ void array29_store(const Array29& a, size_t i, const F29& x) {
    if constexpr (WORDS32) {
        uint32_t w[8];
        f29_canonical(w, x);
#pragma unroll
        for (int k = 0; k < 8; ++k) a.words_out[k * a.ws_out + i] = w[k];
    } else {
        planes29_store(a.planes, i, x);
    }
}

// Binds the previous variable for the two entries p0 and p1 of a pair: x = y + r (y' - y)
// with y at the entry's index and y' at that plus 2*half, written back (to the
// entry's index) and returned.  FOLD2 binds the two previous variables at once
// (the first pass has served two rounds and folded nothing): the entry at i comes
// from the four at i + c Q, c = 2 x_0 + x_1, Q = 2*half (round29_fold2).
template <bool IN32, bool OUT32, bool FOLD2>
__device__ __forceinline__ void fold_pair29(const Array29& a, size_t p0, size_t p1, size_t half, const F29& r,
                                            const Round29Fold2& r2, F29& x0, F29& x1) {
    if constexpr (FOLD2) {
        const size_t Q = 2 * half;
        x0 = round29_fold2(array29_load<IN32>(a, p0), array29_load<IN32>(a, p0 + Q), array29_load<IN32>(a, p0 + 2 * Q),
                           array29_load<IN32>(a, p0 + 3 * Q), r2);
        array29_store<OUT32>(a, p0, x0);
        x1 = round29_fold2(array29_load<IN32>(a, p1), array29_load<IN32>(a, p1 + Q), array29_load<IN32>(a, p1 + 2 * Q),
                           array29_load<IN32>(a, p1 + 3 * Q), r2);
        array29_store<OUT32>(a, p1, x1);
    } else {
        x0 = round29_fold(array29_load<IN32>(a, p0), array29_load<IN32>(a, p0 + 2 * half), r);
        array29_store<OUT32>(a, p0, x0);
        x1 = round29_fold(array29_load<IN32>(a, p1), array29_load<IN32>(a, p1 + 2 * half), r);
        array29_store<OUT32>(a, p1, x1);
    }
}

// The pair of S for the first folding round when S comes as small integers:
// folded entries straight from the four integers each, reduced, then as 29-bit limbs.
template <bool OUT32>
__device__ __forceinline__ void fold_pair29_ints(const DataRound29Args& g, size_t p0, size_t p1, F29& x0, F29& x1) {
    const size_t half = g.half;
    auto entry = [&](size_t i0, size_t i1) {
        uint32_t w[8];
        small_fold_combined(w, g.sx[i0], g.sy ? g.sy[i0] : 0, g.sx[i1], g.sy ? g.sy[i1] : 0, *g.sf);
        return f29_unpack(w);
    };
    x0 = entry(p0, p0 + 2 * half);
    array29_store<OUT32>(g.S, p0, x0);
    x1 = entry(p1, p1 + 2 * half);
    array29_store<OUT32>(g.S, p1, x1);
}

// Sums of lazy values over a wavefront: limbs are added lane to lane (data-parallel
// moves, as in reduce_dev.h) and carried every second step, before they can
// outgrow their words.  v: normalized, below 8 r; the result, in lane 63, is
// normalized and below 64 times that (below 2^264, which is about 565 r).  (Not
// spread to all lanes: what is the same in all of them goes on in the scalar ALU,
// where a multiplication is seven hundred instructions, 2 us.)
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ F29 dpp_add29(const F29& v) {
    F29 o;
#pragma unroll
    for (int k = 0; k < 9; ++k)
        o.l[k] = v.l[k] + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v.l[k], CTRL, ROW_MASK, 0xf, true);
    return o;
}

__device__ __forceinline__ F29 wave_sum29(F29 v) {
    v = dpp_add29<0x111, 0xf>(v);  // row_shr:1
    v = dpp_add29<0x112, 0xf>(v);  // row_shr:2
    v = f29_normalize(v);
    v = dpp_add29<0x114, 0xf>(v);  // row_shr:4
    v = dpp_add29<0x118, 0xf>(v);  // row_shr:8
    v = f29_normalize(v);
    v = dpp_add29<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    v = dpp_add29<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
    v = f29_normalize(v);
    return v;
}

template <bool IN32, bool OUT32, bool INTS = false, bool FOLD2 = false>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4, 4))) k_round_data29(DataRound29Args g) {
    static_assert(!INTS || IN32, "integers are what the first folding round reads");
    static_assert(!FOLD2 || (IN32 && !INTS), "two variables at once are bound from the arrays as they came");
    __shared__ uint32_t lds[4 * 3 * 9];
    Round29Sums sums;
    round29_begin(sums);
    const size_t start = blockIdx.x * g.block_span;
    const size_t lo_mask = ((size_t)1 << g.lbits) - 1;
    const Round29Fold2 r2{g.r_first, g.r_prev, g.r_both};
    for (size_t p = start + threadIdx.x; p < start + g.block_span; p += blockDim.x) {  // at most kRound29MaxPairs times
        F29 a0, a1, s0, s1;
        fold_pair29<IN32, OUT32, FOLD2>(g.A, p + g.off0, p + g.off1, g.half, g.r_prev, r2, a0, a1);
        if constexpr (INTS) fold_pair29_ints<OUT32>(g, p + g.off0, p + g.off1, s0, s1);
        else fold_pair29<IN32, OUT32, FOLD2>(g.S, p + g.off0, p + g.off1, g.half, g.r_prev, r2, s0, s1);
        const F29 w = planes29_load(g.weights, g.lo_off + (p & lo_mask));
        round29_pair(sums, a0, a1, s0, s1, w, g.beta);
    }
    F29 tot[3];
    round29_end(sums, tot);
    // over the wavefront, then over the workgroup's wavefronts (two to four) through LDS
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        tot[q] = f29_shrink(wave_sum29(tot[q]));  // below 77 r, 166 r, 403 r, then below 2.1 r, 3.4 r, 6.7 r
        if (lane == 63) {
#pragma unroll
            for (int k = 0; k < 9; ++k) lds[(wave * 3 + q) * 9 + k] = tot[q].l[k];
        }
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const int q = threadIdx.x;
        F29 v = f29_zero();
        for (int w = 0; w < nwaves; ++w) {
#pragma unroll
            for (int k = 0; k < 9; ++k) v.l[k] += lds[(w * 3 + q) * 9 + k];
        }
        Fr out;
        f29_canonical(out.l, f29_normalize(v));  // below 27 r < 2^261
        if (q < 2 && g.has_hi) out = fr_mul(out, fr_load(g.hi_pool, g.hi_stride, g.hi_off + (start >> g.lbits)));
        // q0, qinf, sA0 at the places the five sums of a round have in a workgroup's partial values
        const int slot = q == 0 ? 0 : q == 1 ? 2 : 3;
        fr_store(g.partials, g.pstride, (size_t)blockIdx.x * 5 + slot, out);
    } else if (threadIdx.x < 5) {
        fr_store(g.partials, g.pstride, (size_t)blockIdx.x * 5 + (threadIdx.x == 3 ? 1 : 4), fr_zero());
    }
}

// ---- the first pass, serving the first two rounds ------------------------------------
//
// The first round binds x_0, the second x_1.  A "quad" is the four entries of an array
// whose indices differ in those two bits only: y_c at p + c Q, c = 2 x_0 + x_1, Q a
// quarter of the array's length.  After the first challenge r the second round's pair is
//   (y'_0, y'_1) = (y_00 + r (y_10 - y_00), y_01 + r (y_11 - y_01)),
// so each of its sums is a polynomial of degree two in r whose coefficients are
// sums over the quads that do not depend on r.  With w the second round's weight
// of the quad, B(x, y) = sum w x y, and because A_i (S_i + beta) = 1 holds exactly
// for every entry before any folding (so B(A_c, S_c + beta) = sum w = 1):
//   q(0)  = 1 - r (1 - r) B(A_10 - A_00, S_10 - S_00)          [c20]
//   q(1)  = 1 - r (1 - r) B(A_11 - A_01, S_11 - S_01)          [c21]
//   q_inf = qd + r (T - qd - qe) + r^2 qe, with
//           qd = B(A_01 - A_00, S_01 - S_00),  T = B(A_11 - A_10, S_11 - S_10),
//           qe = B(A_11 - A_01 - A_10 + A_00, S_11 - S_01 - S_10 + S_00)
//   sA(x_1) = sum A_0x + r (sum A_1x - sum A_0x)
// and the first round's own leading coefficient is (1 - u_1) c20 + u_1 c21.  The
// pass therefore gives five sums of products and the four sums of A, the host
// forms both rounds' messages, and the next pass over the data binds two
// variables at once.
//
// Entries are fully reduced (below r); w is normalized and below r.
static constexpr int kRound01MaxQuads = 16;  // quads per thread (the sums of A are normalized after every seven)

// Workgroup b covers the quads p in [b * block_span, (b + 1) * block_span) of the
// first quarter of the arrays (entries at p + c * quarter, c = 0..3), at most
// kRound01MaxQuads per thread.  Weights are the SECOND round's (its pairs are
// indexed by p), low table in 29-bit planes, the high factor applied once per
// workgroup.  Out, per workgroup: c20, c21, qd, T, qe (partD, five per workgroup)
// and the four sums of A followed by two zeros (partT, six per workgroup).
struct DataRound01Args {
    const uint32_t* A;
    size_t as;
    const uint32_t* S;
    size_t ss;
    size_t quarter;
    size_t block_span;
    Planes29 weights;
    uint32_t lo_off;
    int lbits;
    int has_hi;
    const uint32_t* hi_pool;
    size_t hi_stride;
    uint32_t hi_off;
    uint32_t* partD;
    size_t pstrideD;
    uint32_t* partT;
    size_t pstrideT;
    Fr beta;
};

// The sums are taken on the matrix cores (outer_dev.h).  With X_c = w A_c and S_c the
// products X_c S_d, c != d, are added up by class,
//   M_x0 = X_00 S_10 + X_10 S_00,  M_x1 (c, d = 01, 11),  M_0x (00, 01),  M_1x (10, 11),
//   M_xx = X_00 S_11 + X_11 S_00 + X_01 S_10 + X_10 S_01,
// and with W_c = sum w A_c and sum w A_c (S_c + beta) = 1 (before any fold)
//   c20 = 2 - beta (W_00 + W_10) - M_x0,  c21, qd, T likewise with M_x1, M_0x, M_1x,
//   qe = 4 - beta sum W - M_x0 - M_x1 - M_0x - M_1x + M_xx.
// partD gets these without the constants 2 and 4 and times 2^5 (w is in the form for two
// 29-bit products).  On the vector ALU remain four multiplications per quad and A's sums,
// some 1250 instructions (on the vector ALU alone the pass took 2300 and two
// wavefronts per SIMD kept it 70 % busy); entries are asked for four ahead of their use.
// Issue and HBM bind about equally: 2^25 entries 760 -> 520 us, 4.1 TB/s; a proof of 2^17
// entries in all 524 -> 500 us.  (Tensors of 2^19 entries and more with tables of up to 2^16
// rows take k_first_two_rows.)
struct FirstTwoValues {
    uint32_t vals[9][8];  // M_x0, M_x1, M_0x, M_1x, M_xx, W_00, W_01, W_10, W_11
    uint32_t sums_a[4][4][9];
};
template <int STAGE>
struct FirstTwoShared {
    uint8_t lds[STAGE] __attribute__((aligned(16)));  // the wavefronts' operands
    FirstTwoValues values;
    static_assert(STAGE >= 6 * 4096, "outer_close's sums");
};
static_assert(4 * (size_t)kBlock * kRound01MaxQuads <= kOuterMaxProducts, "a position adds four products to M_xx");

// The class of X_c S_d, c != d.
__device__ constexpr int first_two_class(int c, int d) { return (c ^ d) == 2 ? (c & 1) : (c ^ d) == 1 ? 2 + (c >> 1) : 4; }

// A wavefront's sum of A_c, at most 32 entries per lane: `part` of the workgroup's.
__device__ __forceinline__ void first_two_line(FirstTwoValues& values, int part, int c, const F29& sa) {
    const F29 t = f29_shrink(wave_sum29(f29_shrink(f29_normalize(sa))));
    if ((threadIdx.x & 63) == 63) {
#pragma unroll
        for (int k = 0; k < 9; ++k) values.sums_a[part][c][k] = t.l[k];
    }
}

// Takes a workgroup's closed sums: the classes, and W by column.
__device__ __forceinline__ void first_two_value(FirstTwoValues& values, int q, int column, const Fr& x) {
    if (q == 5 && column >= 4) return;
    const int at = q == 5 ? 5 + column : q;
#pragma unroll
    for (int k = 0; k < 8; ++k) values.vals[at][k] = x.l[k];
}

// The results, once all of that is there; A's sums are of PARTS parts.
template <int PARTS>
__device__ __forceinline__ void first_two_finish(const DataRound01Args& g, const FirstTwoValues& values, size_t start) {
    const int q = threadIdx.x;
    if (q < 5) {
        auto value = [&](int i) {
            Fr f;
#pragma unroll
            for (int k = 0; k < 8; ++k) f.l[k] = values.vals[i][k];
            return f;
        };
        // c20: W_00 + W_10, c21: W_01 + W_11, qd: W_00 + W_01, T: W_10 + W_11, qe: all
        Fr w = q < 2 ? fr_add(value(5 + q), value(7 + q)) : fr_add(value(q == 3 ? 7 : 5), value(q == 3 ? 8 : 6));
        Fr m = value(q == 4 ? 0 : q);
        if (q == 4) {
            w = fr_add(w, fr_add(value(7), value(8)));
            m = fr_sub(fr_add(fr_add(m, value(1)), fr_add(value(2), value(3))), value(4));
        }
        Fr out = fr_sub(fr_zero(), fr_add(fr_mul(w, g.beta), m));
        if (g.has_hi) out = fr_mul(out, fr_load(g.hi_pool, g.hi_stride, g.hi_off + (start >> g.lbits)));
        fr_store(g.partD, g.pstrideD, (size_t)blockIdx.x * 5 + q, out);
    } else if (q < 11) {
        Fr out = fr_zero();
        if (q < 9) {
            F29 t = f29_zero();
            for (int s = 0; s < PARTS; ++s) {
#pragma unroll
                for (int k = 0; k < 9; ++k) t.l[k] += values.sums_a[s][q - 5][k];
            }
            f29_canonical(out.l, f29_normalize(t));
        }
        fr_store(g.partT, g.pstrideT, (size_t)blockIdx.x * 6 + (q - 5), out);
    }
}

__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2, 2))) k_round_first_two(DataRound01Args g) {
    __shared__ FirstTwoShared<4 * 5 * kOuterStage> sh;  // per wavefront S's four operands and one of A
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint8_t* const stage = sh.lds + wave * 5 * kOuterStage;
    uint8_t* const stage_x = stage + 4 * kOuterStage;
    v16i acc[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) outer_clear(acc[q]);
    F29 sa0 = f29_zero(), sa1 = sa0, sa2 = sa0, sa3 = sa0;
    const size_t start = blockIdx.x * g.block_span, share = g.block_span / 4, end = start + (wave + 1) * share;
    const size_t lo_mask = ((size_t)1 << g.lbits) - 1;
    size_t p = start + wave * share;  // of the wavefront's first lane
    uint32_t v[4][8];
#pragma unroll
    for (int c = 0; c < 4; ++c) outer_load(v[c], g.S, g.ss, c * g.quarter + p);
#pragma unroll 1
    for (size_t stop = p; p < end;) {
        // A's sums are normalized after seven turns: that many additions fit a limb
        stop = stop + 7 * kOuterBatch < end ? stop + 7 * kOuterBatch : end;
#pragma unroll 1
        for (; p < stop; p += kOuterBatch) {
            const size_t next = p + kOuterBatch < end ? p + kOuterBatch : p;
            const F29 w = planes29_load(g.weights, g.lo_off + ((p + lane) & lo_mask));
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                uint32_t d[8];
                balanced_digits(d, v[c]);
                outer_put(d, stage + c * kOuterStage);
                outer_load(v[c], g.A, g.as, c * g.quarter + p);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const F29 a = f29_unpack(v[c]);
                outer_load(v[c], g.S, g.ss, c * g.quarter + next);
                F29& sum = c == 0 ? sa0 : c == 1 ? sa1 : c == 2 ? sa2 : sa3;
                sum = f29_add(sum, a);
                uint32_t x[8];
                f29_pack(x, f29_mul(a, w));  // below 1.015 r
                __builtin_amdgcn_sched_barrier(0);
                const OuterOperand xo = outer_operand(x, stage_x);
                outer_mac(acc[5], xo, outer_column(c));
#pragma unroll
                for (int d = 0; d < 4; ++d)
                    if (d != c) outer_mac(acc[first_two_class(c, d)], xo, outer_get(stage + d * kOuterStage));
            }
        }
        sa0 = f29_normalize(sa0);
        sa1 = f29_normalize(sa1);
        sa2 = f29_normalize(sa2);
        sa3 = f29_normalize(sa3);
    }
    first_two_line(sh.values, wave, 0, sa0);
    first_two_line(sh.values, wave, 1, sa1);
    first_two_line(sh.values, wave, 2, sa2);
    first_two_line(sh.values, wave, 3, sa3);
    outer_close<6, 32, true>(acc, (int*)sh.lds, [&](int q, int column, const Fr& x) { first_two_value(sh.values, q, column, x); });
    __syncthreads();
    first_two_finish<4>(g, sh.values, start);
}

}  // namespace zkmi

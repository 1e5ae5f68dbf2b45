// The long rounds of the linking sumcheck (zkattn_link.hip), several from one pass over
// the arrays, for one and two segments.
//
// A pass serves the next V variables (two; three where it reads the integer tensors):
// with the arrays as functions of t in {0,1}^V and the position p of what is left it
// sums, for every t,
//   sum_p w_p Y(t,p)   and   sum_p rw_p Y(t,p)          (w: all variables, rw: row variables)
// and, with two segments, the products  sum_p w_p Y^(1)(t,p) Y^(2)(t',p)  by class: per
// variable 0 (t = t' = 0), 1 (t = t' = 1) or mixed (t != t'), added over the two orders.
// That is what V rounds need whatever their challenges (grid_dev.h; the leading
// coefficient in a variable is 0 + 1 - mixed).  All sums run on the matrix cores
// (outer_dev.h).  Between passes the arrays are bound to V challenges at once, also there
// (k_long_fold: a few constants per output, mfma_dev.h), so both kinds of kernel are
// bound by HBM.  A fold of V variables reads the arrays once where V rounds read them V
// times.  Measured, two segments: 2^24 scores from vectors 3.17 -> 1.93 ms, 2^28 from
// integers 20.9 -> 6.15 ms.  Two variables over field elements because their nine classes
// of sums fit a wavefront's registers (27 do not) with another wavefront beside it.
#pragma once
#include "outer_dev.h"
#include "tlookup_kernels.h"

namespace zkmi {

static const int kLongVars = 2;     // variables of a pass over field elements
static const int kLongIntVars = 3;  // of the first pass where the tensors are integers
static const int kLongLo = 12;      // low weight tables: the last variables, kOuterMaxSpan positions
static const int kLongMixed = 19;   // classes of three variables that are mixed in one at least

// ---- sums ------------------------------------------------------------------------------

struct LongWeights {
    const uint32_t* pool;  // w_p = lo[p & 4095] hi[p >> 12], rw_p = rlo[(p & 4095) >> rlo_shift] rhi[p >> (12 + rhi_shift)]
    size_t stride;
    Planes29 lo29;         // lo times 2^261
    const uint4* lo_ops;   // lo and rlo of all 4096 places as operands
    const uint4* rlo_ops;
    uint32_t hi, rhi;
    int rhi_shift;

    __device__ __forceinline__ Fr high(size_t p) const { return fr_load(pool, stride, hi + (p >> kLongLo)); }
    __device__ __forceinline__ Fr row_high(size_t p) const { return fr_load(pool, stride, rhi + ((p >> kLongLo) >> rhi_shift)); }
    __device__ __forceinline__ F29 low29(size_t p) const { return planes29_load(lo29, p & (((size_t)1 << kLongLo) - 1)); }
    // of the 64 positions from p on
    __device__ __forceinline__ OuterOperand low(size_t p) const { return outer_saved(lo_ops, (p >> 6) & ((1 << kLongLo) / 64 - 1)); }
    __device__ __forceinline__ OuterOperand row_low(size_t p) const { return outer_saved(rlo_ops, (p >> 6) & ((1 << kLongLo) / 64 - 1)); }
};

// The low tables as operands: workgroup b makes four of them, of lo or (blockIdx.y) rlo.
static __global__ void __launch_bounds__(kBlock) k_long_operands(const uint32_t* pool, size_t stride, uint32_t lo, uint32_t rlo,
                                                                 int rlo_shift, uint4* lo_ops, uint4* rlo_ops) {
    __shared__ __attribute__((aligned(16))) uint8_t stage[4 * kOuterStage];
    const uint32_t p = blockIdx.x * kBlock + threadIdx.x, wave = threadIdx.x >> 6;
    const Fr v = fr_load(pool, stride, blockIdx.y ? rlo + (p >> rlo_shift) : lo + p);
    outer_save(blockIdx.y ? rlo_ops : lo_ops, blockIdx.x * 4 + wave, outer_operand(v.l, stage + wave * kOuterStage));
}

// The products of two arrays of 4 P elements by class (class 3 a + b: a, b = 0, 1 or 2
// for mixed in the first and the second variable).  A workgroup takes `span` positions,
// its wavefronts a quarter each.  Per position four multiplications by the weight remain
// on the vector ALU; sixteen products go to the matrix cores.
struct LongGridArgs {
    const uint32_t* x;
    const uint32_t* y;
    size_t xs, ys;
    size_t P, span;
    LongWeights w;
    uint32_t* partials;  // value q of workgroup b at q gridDim.x + b (as in all kernels here)
    size_t pstride;
};

// Entries are asked for four ahead of their use: Y's of the next positions as X's are
// taken, X's as Y's are staged.  At 2^24 entries 274 us, 3.9 TB/s (328 with entries asked
// for where they are used); issue and HBM about equal.
static __global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2, 2))) k_long_grid(LongGridArgs g) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[4 * 5 * kOuterStage];  // per wavefront Y's four operands and one of X
    static_assert(sizeof lds >= 9 * 4096, "outer_close's sums");
    static_assert(4 * kOuterMaxSpan <= kOuterMaxProducts, "a position adds four products to the class that is mixed twice");
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint8_t* const stage = lds + wave * 5 * kOuterStage;
    uint8_t* const stage_x = stage + 4 * kOuterStage;
    v16i acc[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) outer_clear(acc[q]);
    const size_t start = blockIdx.x * g.span, share = g.span / 4, end = start + (wave + 1) * share;
    size_t p = start + wave * share;  // of the wavefront's first lane
    uint32_t v[4][8];
#pragma unroll
    for (int c = 0; c < 4; ++c) outer_load(v[c], g.y, g.ys, c * g.P + p);
#pragma unroll 1
    for (; p < end; p += kOuterBatch) {
        const size_t next = p + kOuterBatch < end ? p + kOuterBatch : p;
        const F29 w = g.w.low29(p + (threadIdx.x & 63));
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            uint32_t d[8];
            balanced_digits(d, v[c]);
            outer_put(d, stage + c * kOuterStage);
            outer_load(v[c], g.x, g.xs, c * g.P + p);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            uint32_t x[8];
            f29_pack(x, f29_mul(f29_unpack(v[c]), w));  // below 1.015 r
            outer_load(v[c], g.y, g.ys, c * g.P + next);
            __builtin_amdgcn_sched_barrier(0);
            const OuterOperand a = outer_operand(x, stage_x);
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const int hi = (c >> 1) == (d >> 1) ? c >> 1 : 2, lo = (c & 1) == (d & 1) ? c & 1 : 2;
                outer_mac(acc[3 * hi + lo], a, outer_get(stage + d * kOuterStage));
            }
        }
    }
    outer_close<9, 32>(acc, (int*)lds, [&](int q, int, const Fr& x) {
        fr_store(g.partials, g.pstride, (size_t)q * gridDim.x + blockIdx.x, fr_mul(x, g.w.high(start)));
    });
}

// The weighted sums of NA arrays of 4 P elements at the four t, and the first array's
// with the row weights.  Workgroup (b, t).  Four arrays of 2^24 entries 372 us, 5.8 TB/s (637
// with entries asked for where they are used, by flat loads, and weights staged each time).
template <int NA>
struct LongLinesArgs {
    const uint32_t* a[NA];
    size_t as[NA];
    size_t P, span;
    LongWeights w;
    uint32_t* partials;  // values (NA + 1) t + ..
    size_t pstride;
};

template <int NA>
static __global__ void __launch_bounds__(kBlock) k_long_lines(LongLinesArgs<NA> g) {
    __shared__ __attribute__((aligned(16))) int sums[(NA + 1) * 1024];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint8_t* stage = (uint8_t*)sums + wave * kOuterStage;
    v16i acc[NA + 1];
#pragma unroll
    for (int q = 0; q <= NA; ++q) outer_clear(acc[q]);
    const size_t start = blockIdx.x * g.span, share = g.span / 4, t = blockIdx.y, end = start + (wave + 1) * share;
    size_t p = start + wave * share;  // of the wavefront's first lane
    uint32_t v[NA][8];
#pragma unroll
    for (int q = 0; q < NA; ++q) outer_load(v[q], g.a[q], g.as[q], t * g.P + p);
#pragma unroll 1
    for (; p < end; p += kOuterBatch) {
        const size_t next = p + kOuterBatch < end ? p + kOuterBatch : p;
        const OuterOperand w = g.w.low(p), rw = g.w.row_low(p);
#pragma unroll
        for (int q = 0; q < NA; ++q) {
            uint32_t d[8];
            balanced_digits(d, v[q]);
            outer_load(v[q], g.a[q], g.as[q], t * g.P + next);  // asked for a turn ahead
            __builtin_amdgcn_sched_barrier(0);
            const OuterOperand b = outer_stage(d, stage);
            outer_mac(acc[q], w, b);
            if (q == 0) outer_mac(acc[NA], rw, b);
        }
    }
    outer_close<NA + 1, 32>(acc, sums, [&](int q, int, const Fr& x) {
        const Fr f = q == NA ? g.w.row_high(start) : g.w.high(start);
        fr_store(g.partials, g.pstride, (t * (NA + 1) + q) * gridDim.x + blockIdx.x, fr_mul(x, f));
    });
}

// ---- the first pass over the integer tensors ----------------------------------------------
//
// 8 P entries.  Every entry is checked against the relations exactly (Z' + sum_k B^(k)
// X^(k) = 0, Y = prod_k Y^(k)), so the unmixed products are Y itself; the mixed ones are
// sums of up to eight products below 2^60, exact in 64 bits.  Four 64-bit integers make
// one operand of 32 digits: the whole pass is nine accumulators.  Their digits go in as
// d - 128 (top bit flipped): the sums come out for v - 0x8080808080808080, which the host
// puts right, the weights' sums being known.  Bound by HBM: 2^28 entries 1.56 ms, 5.5 TB/s
// (3.55 with entries asked for where they are used; 3.39 for one round by the vector ALU).
struct LongIntsArgs {
    const int64_t* Z;
    const uint64_t* Y;
    const uint32_t* X[2];
    const uint32_t* Yk[2];
    uint64_t base[2];
    uint32_t yk_bound;
    size_t P, span;
    LongWeights w;
    uint32_t* partials;  // 8 + 19 (two segments) + 8 values: with w at t = 0..7, the mixed classes, with rw at t = 0..7
    size_t pstride;
    uint32_t* bad;       // device word: 1 = a relation fails somewhere, 2 = an entry is out of range
};

// The mixed classes in order: 9 a + 3 b + c with a digit that is 2.
struct LongMixedClasses {
    int id[kLongMixed];
    constexpr LongMixedClasses() : id() {
        int n = 0;
        for (int v = 0; v < 27; ++v)
            if (v / 9 == 2 || v / 3 % 3 == 2 || v % 3 == 2) id[n++] = v;
    }
};

// sum over the pairs (t, t') of a class of f_t h_t'
template <int CLASS>
__device__ __forceinline__ uint64_t long_class(const uint32_t (&f)[8], const uint32_t (&h)[8]) {
    constexpr int d0 = CLASS / 9, d1 = CLASS / 3 % 3, d2 = CLASS % 3;
    uint64_t s = 0;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const int t0 = t >> 2, t1 = (t >> 1) & 1, t2 = t & 1;
        if ((d0 != 2 && t0 != d0) || (d1 != 2 && t1 != d1) || (d2 != 2 && t2 != d2)) continue;
        const int o = ((d0 == 2 ? 1 - t0 : t0) << 2) | ((d1 == 2 ? 1 - t1 : t1) << 1) | (d2 == 2 ? 1 - t2 : t2);
        s += (uint64_t)f[t] * h[o];
    }
    return s;
}

__device__ __forceinline__ void long_flip64(uint32_t* d, uint64_t v) {
    d[0] = (uint32_t)v ^ kFlip;
    d[1] = (uint32_t)(v >> 32) ^ kFlip;
}

template <int FIRST>
__device__ __forceinline__ void long_mixed_digits(uint32_t (&d)[8], const uint32_t (&f)[8], const uint32_t (&h)[8]) {
    constexpr LongMixedClasses mixed;
    long_flip64(d, long_class<mixed.id[FIRST]>(f, h));
    long_flip64(d + 2, long_class<mixed.id[FIRST + 1]>(f, h));
    long_flip64(d + 4, long_class<mixed.id[FIRST + 2]>(f, h));
    if constexpr (FIRST + 3 < kLongMixed) long_flip64(d + 6, long_class<mixed.id[FIRST + 3]>(f, h));
    else long_flip64(d + 6, 0);
}

// One entry of every tensor.
template <int K>
struct LongIntsEntry {
    uint64_t z, y;
    uint32_t x[K], yk[K];

    // of this lane, the first lane's being entry `first`
    template <class T>
    static __device__ __forceinline__ T at(const T* p, size_t first) {
        typedef const __attribute__((address_space(1))) T* global;
        global q = (global)p + first;
        asm("" : "+s"(q));
        return q[threadIdx.x & 63];
    }
    __device__ __forceinline__ void load(const LongIntsArgs& g, size_t first) {
        z = (uint64_t)at(g.Z, first);
        y = at(g.Y, first);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            x[k] = at(g.X[k], first);
            yk[k] = at(g.Yk[k], first);
        }
    }
    __device__ __forceinline__ uint32_t check(const LongIntsArgs& g) const {
        const int64_t zlim = (int64_t)1 << 62, zs = (int64_t)z;
        uint32_t bad = zs <= -zlim || zs >= zlim || y >= (uint64_t)zlim ? 2u : 0u;
        __int128 lin = zs;
        uint64_t prod = 1;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            lin += (__int128)g.base[k] * x[k];
            if (yk[k] >= g.yk_bound) bad |= 2;
            prod *= yk[k];  // below 2^60 when every factor is in range (else the entry is reported anyway)
        }
        if (lin != 0 || prod != y) bad |= 1;
        return bad;
    }
};

// Entries are asked for four ahead of their use.
template <int K>
static __global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2, 2))) k_long_ints(LongIntsArgs g) {
    constexpr int NW = K == 2 ? 7 : 2, N = NW + 2, NV = K == 2 ? 16 + kLongMixed : 16;
    __shared__ __attribute__((aligned(16))) int sums[N * 1024];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint8_t* stage = (uint8_t*)sums + wave * kOuterStage;
    v16i acc[N];
#pragma unroll
    for (int q = 0; q < N; ++q) outer_clear(acc[q]);
    uint32_t bad = 0;
    const size_t start = blockIdx.x * g.span, share = g.span / 4, end = start + (wave + 1) * share;
    size_t p = start + wave * share;  // of the wavefront's first lane
    LongIntsEntry<K> e[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) e[t].load(g, t * g.P + p);
#pragma unroll 1
    for (; p < end; p += kOuterBatch) {
        const size_t next = p + kOuterBatch < end ? p + kOuterBatch : p;
        const OuterOperand w = g.w.low(p), rw = g.w.row_low(p);
        uint32_t yk[K][8];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t d[8];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                bad |= e[t].check(g);
#pragma unroll
                for (int k = 0; k < K; ++k) yk[k][4 * h + t] = e[t].yk[k];
                long_flip64(d + 2 * t, e[t].y);
                e[t].load(g, h == 0 ? (4 + t) * g.P + p : t * g.P + next);
                __builtin_amdgcn_sched_barrier(0);
            }
            const OuterOperand b = outer_stage(d, stage);
            outer_mac(acc[h], w, b);
            outer_mac(acc[NW + h], rw, b);
        }
        if constexpr (K == 2) {
            uint32_t d[8];
            long_mixed_digits<0>(d, yk[0], yk[1]);
            outer_mac(acc[2], w, outer_stage(d, stage));
            long_mixed_digits<4>(d, yk[0], yk[1]);
            outer_mac(acc[3], w, outer_stage(d, stage));
            long_mixed_digits<8>(d, yk[0], yk[1]);
            outer_mac(acc[4], w, outer_stage(d, stage));
            long_mixed_digits<12>(d, yk[0], yk[1]);
            outer_mac(acc[5], w, outer_stage(d, stage));
            long_mixed_digits<16>(d, yk[0], yk[1]);
            outer_mac(acc[6], w, outer_stage(d, stage));
        }
    }
    if (bad) atomicOr(g.bad, bad);
    outer_close<N, 8>(acc, sums, [&](int q, int slot, const Fr& v) {
        const bool row = q >= NW;
        const int value = row ? NV - 8 + 4 * (q - NW) + slot : 4 * q + slot;
        if (!row && value >= NV - 8) return;  // the place the mixed classes leave free
        fr_store(g.partials, g.pstride, (size_t)value * gridDim.x + blockIdx.x, fr_mul(v, row ? g.w.row_high(start) : g.w.high(start)));
    });
}

// ---- the X^(k) at the final point ------------------------------------------------------------
//
// X^(k)~(v) = sum_(i,j) hi_i lo_j X^(k)[4096 i + j], a sum over j for every i.  Bound by HBM: two
// tensors of 2^24 vectors' entries 223 us, 4.8 TB/s (267 on the vector ALU), of 2^28 integers
// 410 us, 5.2 TB/s (1475).
struct LongEvalArgs {
    const uint32_t* src[3];  // by blockIdx.y
    size_t stride[3];        // (of vectors)
    const uint4* lo_ops;
    const uint32_t* pool;
    size_t pool_stride;
    uint32_t hi;
    uint32_t* partials;      // of tensor k, workgroup b: k gridDim.x + b
    size_t pstride;

    __device__ __forceinline__ Fr high(size_t i) const { return fr_load(pool, pool_stride, hi + i); }
    __device__ __forceinline__ void store(const Fr& x) const { fr_store(partials, pstride, (size_t)blockIdx.y * gridDim.x + blockIdx.x, x); }
};

// Of vectors: a workgroup takes one i.
static __global__ void __launch_bounds__(kBlock) k_long_eval(LongEvalArgs g) {
    __shared__ __attribute__((aligned(16))) int sums[2 * 1024];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint8_t* stage = (uint8_t*)sums + wave * kOuterStage;
    v16i acc[1];
    outer_clear(acc[0]);
    constexpr uint32_t share = (1u << kLongLo) / 4;
    const uint32_t start = wave * share, end = start + share;
    const uint32_t* const src = g.src[blockIdx.y] + ((size_t)blockIdx.x << kLongLo);
    const size_t stride = g.stride[blockIdx.y];
    uint32_t v[2][8];  // asked for two batches ahead
    outer_load(v[0], src, stride, start);
    outer_load(v[1], src, stride, start + kOuterBatch);
#pragma unroll 1
    for (uint32_t p = start; p < end; p += 2 * kOuterBatch) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const uint32_t at = p + q * kOuterBatch, next = at + 2 * kOuterBatch < end ? at + 2 * kOuterBatch : at;
            const OuterOperand w = outer_saved(g.lo_ops, at >> 6);
            uint32_t d[8];
            balanced_digits(d, v[q]);
            outer_load(v[q], src, stride, next);
            __builtin_amdgcn_sched_barrier(0);
            outer_mac(acc[0], w, outer_stage(d, stage));
        }
    }
    outer_close<1, 32>(acc, sums, [&](int, int, const Fr& x) { g.store(fr_mul(x, g.high(blockIdx.x))); });
}

// Of integers: the entries of eight values of i at one j are an operand (four digits
// each, taken as d - 128); a workgroup takes 8 NA values of i.
template <int NA>
static __global__ void __launch_bounds__(kBlock) k_long_eval_ints(LongEvalArgs g) {
    typedef const __attribute__((address_space(1))) uint32_t* global_words;
    __shared__ __attribute__((aligned(16))) int sums[(NA < 2 ? 2 : NA) * 1024];
    __shared__ uint32_t rows[8 * NA][8];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint8_t* stage = (uint8_t*)sums + wave * kOuterStage;
    v16i acc[NA];
#pragma unroll
    for (int q = 0; q < NA; ++q) outer_clear(acc[q]);
    const size_t first = (size_t)blockIdx.x * 8 * NA;
    const global_words from = (global_words)g.src[blockIdx.y] + (first << kLongLo);
    constexpr uint32_t share = (1u << kLongLo) / 4;
    const uint32_t start = wave * share, end = start + share;
    uint32_t v[NA][8];  // asked for a turn ahead
    auto load = [&](int q, uint32_t p) {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            global_words at = from + (((size_t)8 * q + s) << kLongLo) + p;
            asm("" : "+s"(at));
            v[q][s] = at[lane];
        }
    };
#pragma unroll
    for (int q = 0; q < NA; ++q) load(q, start);
#pragma unroll 1
    for (uint32_t p = start; p < end; p += kOuterBatch) {
        const uint32_t next = p + kOuterBatch < end ? p + kOuterBatch : p;
        const OuterOperand w = outer_saved(g.lo_ops, p >> 6);
#pragma unroll
        for (int q = 0; q < NA; ++q) {
            uint32_t d[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) d[s] = v[q][s] ^ kFlip;
            load(q, next);
            __builtin_amdgcn_sched_barrier(0);
            outer_mac(acc[q], w, outer_stage(d, stage));
        }
    }
    outer_close<NA, 4>(acc, sums, [&](int q, int slot, const Fr& x) {
        const Fr f = fr_mul(x, g.high(first + 8 * q + slot));
#pragma unroll
        for (int k = 0; k < 8; ++k) rows[8 * q + slot][k] = f.l[k];
    });
    __syncthreads();
    if (wave == 0) {
        Fr f = fr_zero();
        if (lane < 8 * NA) {
#pragma unroll
            for (int k = 0; k < 8; ++k) f.l[k] = rows[lane][k];
        }
        f = wave_sum(f);
        if (lane == 0) g.store(f);
    }
}

// ---- folds -----------------------------------------------------------------------------------
//
// dst_p = sum_c e_c src_(c P + p), p < P (a multiple of 128).  A wavefront makes 128
// outputs at a time, the constants' matrices staying in its registers; blockIdx.y is the
// array.  dst may be src.  Three arrays of 2^24 entries 386 us, 5.2 TB/s; from 2^28 integers
// (three variables) 1.42 ms, 5.3 TB/s.
struct LongFoldJob {
    const uint32_t* src;
    size_t ss;
    uint32_t* dst;
    size_t ds;
    int vec;    // 16-byte loads allowed
    int scale;  // which constants
};
struct LongFoldArgs {
    LongFoldJob job[3];
    size_t P;
    Fr e[2][1 << kLongVars];
    ToepBias bias[2];
};

// The outputs of four tiles: x[0] and x[1] of a lane are, with 16-byte places, elements
// 4 i + 2 h and the next (i = lane % 32, h = lane / 32), else elements lane and 64 + lane.
__device__ __forceinline__ void long_store(uint32_t* dst, size_t ds, size_t base, bool vec, const Fr& x0, const Fr& x1) {
    const int lane = threadIdx.x & 63;
    if (vec) {
        uint32_t* at = dst + base + 4 * (lane & 31) + 2 * (lane >> 5);
#pragma unroll
        for (int k = 0; k < 8; ++k) *reinterpret_cast<uint2*>(at + k * ds) = make_uint2(x0.l[k], x1.l[k]);
    } else {
        fr_store(dst, ds, base + lane, x0);
        fr_store(dst, ds, base + 64 + lane, x1);
    }
}

template <bool VEC>
__device__ __forceinline__ void long_finish(uint32_t* dst, size_t ds, size_t base, const v16i (&acc)[4], const ToepBias& bias) {
    const Fr x0 = toeplitz_finish(acc[0], VEC ? acc[2] : acc[1], bias), x1 = toeplitz_finish(VEC ? acc[1] : acc[2], acc[3], bias);
    long_store(dst, ds, base, VEC, x0, x1);
}

template <bool VEC>
__device__ __forceinline__ void long_fold_words(const LongFoldJob& job, size_t P, const v4i (&m)[1 << kLongVars], const ToepBias& bias) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 31, h = lane >> 5;
#pragma unroll 1
    for (size_t base = ((size_t)blockIdx.x * 4 + wave) * 128; base < P; base += (size_t)gridDim.x * 512) {
        v16i acc[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) outer_clear(acc[j]);
        const uint32_t* at = job.src + 4 * h * job.ss + base + (VEC ? 4 * i : i);
#pragma unroll
        for (int c = 0; c < 1 << kLongVars; ++c) {
            uint32_t x[4][4];  // [limb][tile]
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t* from = at + c * P + q * job.ss;
                if constexpr (VEC) {
                    const uint4 v = *reinterpret_cast<const uint4*>(from);
                    x[q][0] = v.x; x[q][1] = v.y; x[q][2] = v.z; x[q][3] = v.w;
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[q][j] = from[32 * j];
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const v4i b = {(int)(x[0][j] ^ kFlip), (int)(x[1][j] ^ kFlip), (int)(x[2][j] ^ kFlip), (int)(x[3][j] ^ kFlip)};
                acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(m[c], b, acc[j], 0, 0, 0);
            }
        }
        long_finish<VEC>(job.dst, job.ds, base, acc, bias);
    }
}

static __global__ void __launch_bounds__(kBlock) k_long_fold(LongFoldArgs g) {
    constexpr int C = 1 << kLongVars;
    __shared__ __attribute__((aligned(16))) uint8_t table[C * kToepBytes];
    const LongFoldJob& job = g.job[blockIdx.y];
    if (threadIdx.x < 32 * C) {
        uint32_t digits[8];
        toeplitz_column(digits, g.e[job.scale][threadIdx.x >> 5], threadIdx.x & 31);
        toeplitz_store(table + (threadIdx.x >> 5) * kToepBytes, digits, threadIdx.x & 31);
    }
    __syncthreads();
    v4i m[C];
#pragma unroll
    for (int c = 0; c < C; ++c) m[c] = reinterpret_cast<const v4i*>(table)[c * 64 + (threadIdx.x & 63)];
    if (job.vec) long_fold_words<true>(job, g.P, m, g.bias[job.scale]);
    else long_fold_words<false>(job, g.P, m, g.bias[job.scale]);
}

// The same from integers, eight to an output: an integer of B bytes is B columns of the
// constants' matrices, 32 bytes to an instruction.
struct LongFoldIntsArgs {
    const uint64_t* Y;
    const uint32_t* Yk[2];
    int vec[3];         // 16-byte loads allowed: of Y, of the Y^(k)
    uint32_t* dst[3];   // of Y, of the Y^(k)
    size_t ds;
    size_t P;
    Fr e[2][1 << kLongIntVars];  // [1]: Y's.  e_c 2^256 in Montgomery form, so that results come out in it
    ToepBias bias[2];
};

template <bool VEC, int BYTES>
__device__ __forceinline__ void long_fold_ints(const uint32_t* src, uint32_t* dst, size_t ds, size_t P, const uint8_t* table, const ToepBias& bias) {
    constexpr int WORDS = BYTES / 4, STEPS = BYTES / 4;  // words of an entry; instructions for eight entries
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 31, h = lane >> 5;
    v4i m[STEPS];
#pragma unroll
    for (int s = 0; s < STEPS; ++s) m[s] = reinterpret_cast<const v4i*>(table)[s * 64 + lane];
#pragma unroll 1
    for (size_t base = ((size_t)blockIdx.x * 4 + wave) * 128; base < P; base += (size_t)gridDim.x * 512) {
        v16i acc[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) outer_clear(acc[j]);
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            int x[4][4];  // [word of the lane's sixteen bytes][tile]
#pragma unroll
            for (int e = 0; e < 4 / WORDS; ++e) {
                const size_t c = (size_t)(8 / STEPS) * s + (4 / WORDS) * h + e;
                const uint32_t* from = src + WORDS * (c * P + base + (VEC ? 4 * i : i));
                uint32_t v[4 * WORDS];  // four entries
                if constexpr (VEC) {
#pragma unroll
                    for (int q = 0; q < WORDS; ++q) {
                        const uint4 u = reinterpret_cast<const uint4*>(from)[q];
                        v[4 * q] = u.x; v[4 * q + 1] = u.y; v[4 * q + 2] = u.z; v[4 * q + 3] = u.w;
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int q = 0; q < WORDS; ++q) v[WORDS * j + q] = from[WORDS * 32 * j + q];
                }
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int q = 0; q < WORDS; ++q) x[WORDS * e + q][j] = (int)(v[WORDS * j + q] ^ kFlip);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(m[s], v4i{x[0][j], x[1][j], x[2][j], x[3][j]}, acc[j], 0, 0, 0);
        }
        long_finish<VEC>(dst, ds, base, acc, bias);
    }
}

static __global__ void __launch_bounds__(kBlock) k_long_fold_ints(LongFoldIntsArgs g) {
    __shared__ __attribute__((aligned(16))) uint8_t table[2 * kToepBytes];
    const int q = blockIdx.y, bytes = q == 0 ? 8 : 4;
    if ((int)threadIdx.x < 8 * bytes) {
        uint32_t digits[8];
        toeplitz_column(digits, g.e[q == 0][threadIdx.x / bytes], threadIdx.x % bytes);
        toeplitz_store(table + (threadIdx.x >> 5) * kToepBytes, digits, threadIdx.x & 31);
    }
    __syncthreads();
    const uint32_t* src = q == 0 ? (const uint32_t*)g.Y : g.Yk[q - 1];
    const ToepBias& bias = g.bias[q == 0];
    if (q == 0 && g.vec[0]) long_fold_ints<true, 8>(src, g.dst[0], g.ds, g.P, table, bias);
    else if (q == 0) long_fold_ints<false, 8>(src, g.dst[0], g.ds, g.P, table, bias);
    else if (g.vec[q]) long_fold_ints<true, 4>(src, g.dst[q], g.ds, g.P, table, bias);
    else long_fold_ints<false, 4>(src, g.dst[q], g.ds, g.P, table, bias);
}

}  // namespace zkmi

// The sumcheck that closes zkAttn-Prove (Protocol 2 of the paper, last step):
// one proof that, for a rows x cols score matrix and K digit segments,
//     Z'_x + sum_k B^(k) X^(k)_x = 0,   Y_x = prod_k Y^(k)_x,   yhat_i = sum_j Y_(i,j)
// (the relations of Section 5.1 plus the row sums of Protocol 2's compute step).
// The paper names the relations and leaves the batching open; with u in F^n,
// n = log2(rows cols), and alpha from the transcript the identity proved is
//
//   alpha^2 yhat~(u_rows) = sum_x [ e~(u,x) ( Z'(x) + sum_k B^(k) X^(k)(x) + alpha Y(x) )
//                                  - alpha e~(u,x) prod_k Y^(k)(x)
//                                  + alpha^2 e~(u_rows, x_rows) Y(x) ]
//
// by the generic sumcheck of Section 3.3, degree K+1 per variable, row variables
// (the top index bits) first.
//
// How a round is computed.  With x = (X, rest) after binding t variables,
// e~(u,x) = c_t e~(u_t,X) e_rest(rest), c_t = prod_{s<t} e~(u_s,r_s), and e_rest
// is never folded: while a row variable is being bound it is the product of a
// table over the remaining row variables (one factor per workgroup, a workgroup
// never straddles rows) and the table over all column variables; afterwards it
// is one table over the remaining column variables.  The factor over the row
// variables is at the same time the weight e~(u_rows, .) of the row-sum term.
// Per round the device returns
//     L(0), L(1)        of  L(X) = sum_rest e_rest (Z' + sum_k B^(k) X^(k) + alpha Y)(X,rest)  (linear),
//     Q(0..K)           of  Q(X) = sum_rest e_rest prod_k Y^(k)(X,rest)                        (degree K),
//     sY(0), sY(1)      of  sY(X) = sum_rest [row weight] alpha Y(X,rest)                      (linear),
// and the host forms g(X) = c_t e~(u_t,X) (L(X) - alpha Q(X)) + alpha w(X) sY(X),
// w(X) = c_t e~(u_t,X) in the row rounds and the constant c_(log2 rows) after them.
//
// The linear relation leaves the rounds after the first.  Z' + sum_k B^(k) X^(k)
// is multilinear and zero on the whole cube, hence the zero polynomial: once the
// first round has found its weighted sum to be zero, every folded entry of it is
// zero too, L(X) is alpha times the weighted sum of Y alone, and Z' and the X^(k)
// are neither folded nor read again.  Their values at the final point, which the
// proof ends with, are multilinear evaluations of the tensors as they came
// (k_link_mle: one pass, against two small tables of e~(v, .)), and
// Z'~(v) = - sum_k B^(k) X^(k)~(v).
//
// Y is multiplied by alpha on the way: in the first round on the fly, in the
// second when the folded array is first written; from then on the array holds
// the scaled values (the final claim is scaled back on the host).
//
// Of one and two segments and more than kLinkPassVars variables these sums do not come
// round by round: a pass yields those of the next two rounds (of the next three from
// integers), and one fold binds their variables (link_long.h; the host scales the first
// pass's sums of Y, the first fold the array).
// The kernels below serve three segments and shorter proofs.
#include "internal.h"
#include "small_dev.h"
#include "tlookup_kernels.h"
#include "grid_dev.h"
#include "link_long.h"
#include "long_host.h"
#include "transcript.h"

#include <algorithm>

namespace zkmi {

static const int kLinkMaxK = 3;

// The last rounds (from the third on, once at most kLinkPassVars variables are left, up
// to two segments) come several from one pass (grid_dev.h): L and sY are linear in
// every variable, Q is of degree two.  The last kLinkHostVars variables are the host's.
// With three segments Q is of degree three, which the passes do not cover.  Measured,
// 2^24 scores and two segments: 3.79 -> 3.33 ms.
static const int kLinkPassVars = 16, kLinkHostVars = 6;
static const uint32_t kLinkGridValues = 27 + 2 * 8;

template <int K>
struct LinkRoundArgs {
    PairArray Z, Y;
    PairArray X[K], Yk[K];
    Fr base[K];  // B^(k)
    int scale_x[K];  // 0: B^(k) = 1 (or already applied)
    Fr alpha;
    size_t half;
    size_t block_span;
    Fr r_prev;
    EqSplit eq;
    int row_round;  // the workgroup's high factor also weighs the sums of Y
    uint32_t* partials;  // K + 5 values per workgroup: L0 L1 Q0..QK sY0 sY1
    size_t pstride;
    // The tensors as the integers they are (zkattn_link_prove_small), read by the
    // first two rounds instead of the PairArray sources.
    const int64_t* Zs;
    const uint64_t* Ys;
    const uint32_t* Xs[K];
    const uint32_t* Yks[K];
    // second round: what the integers are folded with by the first challenge, in device
    // memory (as launch arguments they would crowd the scalar registers):
    // [0] scaled by 1 (the Y^(k)), [1] by alpha (Y)
    const SmallFoldConsts* fold;
    int side;            // folding rounds: the X (0 or 1) at which L, Q and sY are summed
    uint64_t base_small[K];
    uint32_t yk_bound;   // segment outputs stay below it, so that products of K extrapolated factors fit 63 bits
    Fr raw_scale;        // 2^96: what turns a short-reduced raw sum into its Montgomery form
    uint32_t* bad;       // device word: 1 = a relation fails somewhere, 2 = an entry is out of range
};

// x0 = fold of (in[p], in[p + 2 half]), x1 = fold of (in[p + half], in[p + 3 half]), as field
// elements (scaled, see SmallFoldConsts), written to dst and returned.
__device__ __forceinline__ void small_pair64(const int64_t* __restrict__ in, size_t p, size_t half, const SmallFoldConsts& k,
                                             const PairArray& dst, Fr& x0, Fr& x1) {
    small_fold64(x0.l, in[p], in[p + 2 * half], k);
    small_fold64(x1.l, in[p + half], in[p + 3 * half], k);
    fr_store(dst.dst, dst.ds, p, x0);
    fr_store(dst.dst, dst.ds, p + half, x1);
}
__device__ __forceinline__ void small_pair32(const uint32_t* __restrict__ in, size_t p, size_t half, const SmallFoldConsts& k,
                                             const PairArray& dst, Fr& x0, Fr& x1) {
    small_fold32(x0.l, in[p], in[p + 2 * half], k);
    small_fold32(x1.l, in[p + half], in[p + 3 * half], k);
    fr_store(dst.dst, dst.ds, p, x0);
    fr_store(dst.dst, dst.ds, p + half, x1);
}

// The first round on field elements: nothing to fold, Z' and the X^(k) take part (the only round in which they do).
template <int K>
static __global__ void __launch_bounds__(kBlock) k_link_round0(LinkRoundArgs<K> g) {
    constexpr int NV = K + 5;
    __shared__ uint32_t lds[4 * NV * 8];
    Fr tot[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) tot[q] = fr_zero();
    const size_t start = blockIdx.x * g.block_span;
    const size_t lo_mask = ((size_t)1 << g.eq.lbits) - 1;
    for (size_t p = start + threadIdx.x; p < start + g.block_span; p += kBlock) {
        const Fr w = fr_load(g.eq.pool, g.eq.stride, g.eq.lo_off + (p & lo_mask));
        Fr lin0, lin1;
        load_pair<false>(g.Z, p, g.half, g.r_prev, lin0, lin1);
        {
            Fr y0, y1;
            load_pair<false>(g.Y, p, g.half, g.r_prev, y0, y1);
            y0 = fr_mul(y0, g.alpha);
            y1 = fr_mul(y1, g.alpha);
            tot[K + 3] = fr_add(tot[K + 3], y0);
            tot[K + 4] = fr_add(tot[K + 4], y1);
            lin0 = fr_add(lin0, y0);
            lin1 = fr_add(lin1, y1);
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            Fr x0, x1;
            load_pair<false>(g.X[k], p, g.half, g.r_prev, x0, x1);
            if (g.scale_x[k]) {
                x0 = fr_mul(x0, g.base[k]);
                x1 = fr_mul(x1, g.base[k]);
            }
            lin0 = fr_add(lin0, x0);
            lin1 = fr_add(lin1, x1);
        }
        tot[0] = fr_add(tot[0], fr_mul(w, lin0));
        tot[1] = fr_add(tot[1], fr_mul(w, lin1));
        // the product of the segment outputs at X = 0..K, the weight folded into the first factor
        Fr f[K], d[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            Fr a0, a1;
            load_pair<false>(g.Yk[k], p, g.half, g.r_prev, a0, a1);
            if (k == 0) {
                a0 = fr_mul(a0, w);
                a1 = fr_mul(a1, w);
            }
            f[k] = a0;
            d[k] = fr_sub(a1, a0);
        }
#pragma unroll
        for (int X = 0; X <= K; ++X) {
            Fr prod = f[0];
#pragma unroll
            for (int k = 1; k < K; ++k) prod = fr_mul(prod, f[k]);
            tot[2 + X] = fr_add(tot[2 + X], prod);
            if (X < K) {
#pragma unroll
                for (int k = 0; k < K; ++k) f[k] = fr_add(f[k], d[k]);
            }
        }
    }
    block_sum<NV, 4>(tot, lds);
    if (threadIdx.x == 0) {
        if (g.eq.has_hi) {
            const Fr hf = fr_load(g.eq.pool, g.eq.stride, g.eq.hi_off + (start >> g.eq.lbits));
#pragma unroll
            for (int q = 0; q < K + 3; ++q) tot[q] = fr_mul(tot[q], hf);
            if (g.row_round) {
                tot[K + 3] = fr_mul(tot[K + 3], hf);
                tot[K + 4] = fr_mul(tot[K + 4], hf);
            }
        }
#pragma unroll
        for (int q = 0; q < NV; ++q) fr_store(g.partials, g.pstride, (size_t)blockIdx.x * NV + q, tot[q]);
    }
}

// A folding round: binds the previous variable, writes the folded entries back and
// sums one side X = a of the round only,
//     L(a), sY(a), Q(a), the leading coefficient of Q (K > 1), Q(2) (K = 3).
// The other side follows on the host from the round before: with r its challenge,
//     L_prev(r) = e~(u_t,0) L(0) + e~(u_t,1) L(1),   the same for Q, and for sY while a row variable is bound
// (afterwards sY_prev(r) = sY(0) + sY(1)).  The weighted sums are added up as 512-bit
// integers and reduced once per thread.  Bound by instruction issue: for two segments
// eight multiplications and three unreduced products per pair, where both sides and
// Q at 0, 1, 2 took thirteen.  Measured, 2^28 scores in two segments, the third round
// (2^25 pairs): 5.27 -> 4.34 ms, 4.5 TB/s.
// SCALE: the sources hold unscaled Y (the second round); SMALL: they are the integer
// tensors (with SCALE).
template <int K>
struct LinkFoldValues {
    static constexpr int count = K == 1 ? 3 : K + 2;  // L, sY, Q(a), lead, Q(2)
};
template <int K, bool SCALE, bool SMALL = false>
static __global__ void __launch_bounds__(kBlock, K == 3 ? 2 : 3) k_link_round(LinkRoundArgs<K> g) {
    static_assert(!SMALL || SCALE, "integer sources are read by the first two rounds only");
    constexpr int NV = LinkFoldValues<K>::count;
    __shared__ uint32_t lds[4 * NV * 8];
    FrWide wide[NV - 1];  // L, Q(a), lead, Q(2)
#pragma unroll
    for (int q = 0; q < NV - 1; ++q) wide[q] = fr_wide_zero();
    Fr sy = fr_zero();
    const size_t start = blockIdx.x * g.block_span;
    const size_t lo_mask = ((size_t)1 << g.eq.lbits) - 1;
    for (size_t p = start + threadIdx.x; p < start + g.block_span; p += kBlock) {
        const Fr w = fr_load(g.eq.pool, g.eq.stride, g.eq.lo_off + (p & lo_mask));
        {
            Fr y0, y1;
            if constexpr (SMALL) small_pair64((const int64_t*)g.Ys, p, g.half, g.fold[1], g.Y, y0, y1);
            else load_pair<true, !SCALE>(g.Y, p, g.half, g.r_prev, y0, y1);
            if constexpr (SCALE && !SMALL) {
                y0 = fr_mul(y0, g.alpha);
                y1 = fr_mul(y1, g.alpha);
                fr_store(g.Y.dst, g.Y.ds, p, y0);
                fr_store(g.Y.dst, g.Y.ds, p + g.half, y1);
            }
            const Fr y = g.side ? y1 : y0;
            sy = fr_add(sy, y);
            fr_wide_mac(wide[0], w, y);
        }
        Fr at, lead, two;  // products of all factors but the last, at X = a, of the differences, at X = 2
#pragma unroll
        for (int k = 0; k < K; ++k) {
            Fr a0, a1;
            if constexpr (SMALL) small_pair32(g.Yks[k], p, g.half, g.fold[0], g.Yk[k], a0, a1);
            else load_pair<true>(g.Yk[k], p, g.half, g.r_prev, a0, a1);
            const Fr d = fr_sub(a1, a0), x = g.side ? a1 : a0;
            if (k + 1 < K) {
                at = fr_mul(k == 0 ? w : at, x);
                lead = fr_mul(k == 0 ? w : lead, d);
                if constexpr (K == 3) two = fr_mul(k == 0 ? w : two, fr_add(a1, d));
            } else {
                fr_wide_mac(wide[1], k == 0 ? w : at, x);
                if constexpr (K > 1) fr_wide_mac(wide[2], lead, d);
                if constexpr (K == 3) fr_wide_mac(wide[3], two, fr_add(a1, d));
            }
        }
    }
    Fr tot[NV];
    tot[0] = fr_wide_reduce(wide[0]);
    tot[1] = sy;
#pragma unroll
    for (int q = 1; q < NV - 1; ++q) tot[q + 1] = fr_wide_reduce(wide[q]);
    block_sum<NV, 4>(tot, lds);
    if (threadIdx.x == 0) {
        if (g.eq.has_hi) {
            const Fr hf = fr_load(g.eq.pool, g.eq.stride, g.eq.hi_off + (start >> g.eq.lbits));
#pragma unroll
            for (int q = 0; q < NV; ++q)
                if (q != 1 || g.row_round) tot[q] = fr_mul(tot[q], hf);
        }
#pragma unroll
        for (int q = 0; q < NV; ++q) fr_store(g.partials, g.pstride, (size_t)blockIdx.x * NV + q, tot[q]);
    }
}

struct LinkFoldConsts {
    SmallFoldConsts c[2];
};
static __global__ void k_store_fold_consts(LinkFoldConsts v, SmallFoldConsts* dst, int count) {
    const int which = threadIdx.x >> 5, word = threadIdx.x & 31;
    if (which < count) ((uint32_t*)&dst[which])[word] = ((const uint32_t*)&v.c[which])[word];
}

// t += w m.  Values are mostly below 2^32: lanes whose high word is zero skip its
// eight products (the branch is taken by no lane of most wavefronts).
template <int NL>
__device__ __forceinline__ void link_mac(uint32_t (&t)[NL], const Fr& w, uint64_t m) {
    small_mac32<NL, 0>(t, w.l, (uint32_t)m);
    if (m >> 32) small_mac32<NL, 1>(t, w.l, (uint32_t)(m >> 32));
}

// The first round on the integer tensors.  Every entry is checked against the
// relations exactly (Z' + sum_k B^(k) X^(k) = 0 and Y = prod_k Y^(k) as integers),
// so what is left of the round's sums is
//   L(X) = alpha sum w Y(X),  Q(X) = sum w Y(X)  at X = 0, 1,
//   Q(X) = sum w prod_k (Y^(k)_0 + X (Y^(k)_1 - Y^(k)_0))  at X = 2..K,   sY(X) = alpha sum Y(X),
// all of them sums of a weight times a small integer: sixteen multiply-adds per
// term, accumulated unreduced and reduced once per thread.
template <int K>
static __global__ void __launch_bounds__(kBlock) k_link_round0_small(LinkRoundArgs<K> g) {
    constexpr int NV = K + 5, NS = K + 3;  // sums taken here: S0 S1 P2..PK sy0 sy1
    __shared__ uint32_t lds[4 * NS * 8];
    uint32_t s0[12], s1[12], pos[K > 1 ? K - 1 : 1][12], neg[K > 1 ? K - 1 : 1][12];
#pragma unroll
    for (int j = 0; j < 12; ++j) {
        s0[j] = s1[j] = 0;
#pragma unroll
        for (int q = 0; q < K - 1; ++q) pos[q][j] = neg[q][j] = 0;
    }
    unsigned __int128 sy0 = 0, sy1 = 0;
    uint32_t bad = 0;
    const size_t start = blockIdx.x * g.block_span;
    const size_t lo_mask = ((size_t)1 << g.eq.lbits) - 1;
    const int64_t zlim = (int64_t)1 << 62;
    for (size_t p = start + threadIdx.x; p < start + g.block_span; p += kBlock) {
        const Fr w = fr_load(g.eq.pool, g.eq.stride, g.eq.lo_off + (p & lo_mask));
        uint64_t y[2];
        int64_t yk[K][2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const size_t i = p + e * g.half;
            const int64_t z = g.Zs[i];
            y[e] = g.Ys[i];
            if (z <= -zlim || z >= zlim || y[e] >= (uint64_t)zlim) bad |= 2;
            __int128 lin = z;
            uint64_t prod = 1;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                lin += (__int128)g.base_small[k] * g.Xs[k][i];
                const uint32_t v = g.Yks[k][i];
                if (v >= g.yk_bound) bad |= 2;
                yk[k][e] = v;
                prod *= v;  // below 2^63 when every factor is in range (else the entry is reported anyway)
            }
            if (lin != 0 || prod != y[e]) bad |= 1;
        }
        link_mac(s0, w, y[0]);
        link_mac(s1, w, y[1]);
        sy0 += y[0];
        sy1 += y[1];
#pragma unroll
        for (int X = 2; X <= K; ++X) {
            int64_t pr = 1;
#pragma unroll
            for (int k = 0; k < K; ++k) pr *= yk[k][0] + X * (yk[k][1] - yk[k][0]);
            if (pr < 0) link_mac(neg[X - 2], w, 0ull - (uint64_t)pr);
            else link_mac(pos[X - 2], w, (uint64_t)pr);
        }
    }
    if (bad) atomicOr(g.bad, bad);
    // raw sums (below 16 * 2^63 * 2^256 < r 2^96) to field elements
    Fr tot[NS];
    auto to_field = [&](uint32_t (&t)[12]) {
        Fr x;
        small_reduce<3>(x.l, t);
        return fr_mul(x, g.raw_scale);
    };
    tot[0] = to_field(s0);
    tot[1] = to_field(s1);
#pragma unroll
    for (int q = 0; q < K - 1; ++q) tot[2 + q] = fr_sub(to_field(pos[q]), to_field(neg[q]));
    {
        Fr c0 = fr_zero(), c1 = fr_zero();
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            c0.l[j] = (uint32_t)(sy0 >> (32 * j));
            c1.l[j] = (uint32_t)(sy1 >> (32 * j));
        }
        tot[K + 1] = fr_to_mont(c0);
        tot[K + 2] = fr_to_mont(c1);
    }
    block_sum<NS, 4>(tot, lds);
    if (threadIdx.x == 0) {
        Fr out[NV];
        Fr S0 = tot[0], S1 = tot[1], y0 = fr_mul(tot[K + 1], g.alpha), y1 = fr_mul(tot[K + 2], g.alpha);
        if (g.eq.has_hi) {
            const Fr hf = fr_load(g.eq.pool, g.eq.stride, g.eq.hi_off + (start >> g.eq.lbits));
            S0 = fr_mul(S0, hf);
            S1 = fr_mul(S1, hf);
#pragma unroll
            for (int q = 0; q < K - 1; ++q) tot[2 + q] = fr_mul(tot[2 + q], hf);
            if (g.row_round) {
                y0 = fr_mul(y0, hf);
                y1 = fr_mul(y1, hf);
            }
        }
        out[0] = fr_mul(S0, g.alpha);
        out[1] = fr_mul(S1, g.alpha);
        out[2] = S0;
        out[3] = S1;
#pragma unroll
        for (int q = 0; q < K - 1; ++q) out[4 + q] = tot[2 + q];
        out[K + 3] = y0;
        out[K + 4] = y1;
#pragma unroll
        for (int q = 0; q < NV; ++q) fr_store(g.partials, g.pstride, (size_t)blockIdx.x * NV + q, out[q]);
    }
}

// X^(k)~(v) for the K digit tensors at once: sum_i e~(v, i) X^(k)_i with
// e~(v, i) = hi[i >> lbits] lo[i & (2^lbits - 1)].  A workgroup takes 2^lbits
// consecutive entries (one value of the high index), workgroup (b, k) writes its
// part of tensor k to partials[b K + k].  SMALL: the tensors are 32-bit integers.
template <bool SMALL>
struct LinkMleArgs {
    const uint32_t* src[kLinkMaxK];  // SMALL: the integers themselves; else eight word planes
    size_t stride[kLinkMaxK];
    int K;
    EqSplit eq;        // lo and hi tables of the point
    Fr raw_scale;      // 2^64 (see SmallFoldConsts): short-reduced raw sums to Montgomery form
    uint32_t* partials;
    size_t pstride;
};

template <bool SMALL>
static __global__ void __launch_bounds__(kBlock) k_link_mle(LinkMleArgs<SMALL> g) {
    __shared__ uint32_t lds[4 * 8];
    const int k = blockIdx.y;
    const size_t span = (size_t)1 << g.eq.lbits;
    const size_t start = blockIdx.x * span;
    Fr tot[1];
    if constexpr (SMALL) {
        uint32_t t[11];
#pragma unroll
        for (int j = 0; j < 11; ++j) t[j] = 0;
        // at most 2^12 / 256 = 16 terms below 2^288 each
        for (size_t c = threadIdx.x; c < span; c += kBlock) {
            const Fr w = fr_load(g.eq.pool, g.eq.stride, g.eq.lo_off + c);
            small_mac32(t, w.l, g.src[k][start + c]);
        }
        Fr x;
        small_reduce<2>(x.l, t);
        tot[0] = fr_mul(x, g.raw_scale);
    } else {
        WideInRegs wide;
        wide.clear();
        for (size_t c = threadIdx.x; c < span; c += kBlock)
            wide.mac(0, fr_load(g.eq.pool, g.eq.stride, g.eq.lo_off + c), fr_load(g.src[k], g.stride[k], start + c));
        tot[0] = wide.finish(0);
    }
    block_sum<1, 4>(tot, lds);
    if (threadIdx.x == 0) {
        if (g.eq.has_hi) tot[0] = fr_mul(tot[0], fr_load(g.eq.pool, g.eq.stride, g.eq.hi_off + blockIdx.x));
        fr_store(g.partials, g.pstride, (size_t)blockIdx.x * g.K + k, tot[0]);
    }
}

// ---- weight tables -------------------------------------------------------------------------
//
// Round t < nr (row variables):  hi over variables t+1 .. nr-1, lo over nr .. n-1.
// Round t >= nr (column variables): lo over variables t+1 .. n-1.
struct LinkTables {
    uint32_t* pool = nullptr;
    size_t stride = 0;
    uint32_t row_off[32];  // hi table of row round t
    uint32_t cols_off = 0; // the table over all column variables
    uint32_t col_off[32];  // lo table of column round t (index t - nr)
    int nr = 0, nc = 0;

    static size_t entries(int nr, int nc) {
        size_t total = 0;
        for (int t = 0; t < nr; ++t) total += (size_t)1 << (nr - t - 1);
        total += (size_t)1 << nc;
        for (int t = 0; t < nc; ++t) total += (size_t)1 << (nc - t - 1);
        return total;
    }

    EqSplit round(int t) const {
        EqSplit e;
        e.pool = pool;
        e.stride = stride;
        if (t < nr) {
            e.lbits = nc;
            e.lo_off = cols_off;
            e.has_hi = 1;
            e.hi_off = row_off[t];
        } else {
            e.lbits = nr + nc - t - 1;
            e.lo_off = col_off[t - nr];
            e.has_hi = 0;
            e.hi_off = 0;
        }
        return e;
    }
};

static int link_tables_build(LinkTables& lt, const host::F* u, int nr, int nc, Carver& cv, hipStream_t stream) {
    lt.nr = nr;
    lt.nc = nc;
    lt.stride = LinkTables::entries(nr, nc);
    lt.pool = cv.limbs(lt.stride);
    if (!lt.pool) return ZK_E_BUFSZ;
    EqPoolArgs args;
    memset(&args, 0, sizeof args);
    const int n = nr + nc;
    for (int t = 0; t < n; ++t) args.u[t] = to_dev(u[t]);
    int q = 0;
    uint32_t off = 0;
    auto table = [&](int var0, int nvars) {
        args.offset[q] = off;
        args.var0[q] = (uint8_t)var0;
        args.nvars[q] = (uint8_t)nvars;
        uint32_t at = off;
        off += 1u << nvars;
        ++q;
        return at;
    };
    for (int t = 0; t < nr; ++t) lt.row_off[t] = table(t + 1, nr - t - 1);
    lt.cols_off = table(nr, nc);
    for (int t = nr; t < n; ++t) lt.col_off[t - nr] = table(t + 1, n - t - 1);
    args.ntables = q;
    args.total = off;
    if (q > 64) return ZK_E_BADARG;
    args.scale = to_dev(host::one());
    launch_eq_pool(lt.pool, lt.stride, args, stream);
    ZK_HIP_TRY(hipGetLastError());
    return ZK_OK;
}

// ---- the long rounds' weights and passes (link_long.h) ----------------------------------------
//
// Tensors of more than kLinkPassVars variables, one or two segments: passes over two
// variables (three of the integers first) until at most kLinkPassVars are left.  Each has
// its high tables; the low ones are the same for all.
static bool link_long(int n, int K) { return n > kLinkPassVars && K <= 2; }
static int link_long_vars(int t, bool ints) { return ints && t == 0 ? kLongIntVars : kLongVars; }

struct LongTables {
    uint32_t* pool = nullptr;
    size_t stride = 0;
    uint4* pool29 = nullptr;
    uint4* lo_ops = nullptr;
    uint4* rlo_ops = nullptr;
    uint32_t hi[32], rhi[32];  // by the pass's first variable
    int n = 0, nr = 0;

    static int row_low_vars(int n, int nr) { return nr > n - kLongLo ? nr - (n - kLongLo) : 0; }
    static int high_vars(int n, int t, int vars) { return n - kLongLo - t - vars; }
    static int row_high_vars(int n, int nr, int t, int vars) {
        const int v = std::min(nr, n - kLongLo) - t - vars;
        return v > 0 ? v : 0;
    }
    static size_t entries(int n, int nr, bool ints) {
        size_t total = ((size_t)2 << kLongLo) + ((size_t)1 << row_low_vars(n, nr));
        for (int t = 0; n - t > kLinkPassVars; t += link_long_vars(t, ints)) {
            const int v = link_long_vars(t, ints);
            total += ((size_t)1 << high_vars(n, t, v)) + ((size_t)1 << row_high_vars(n, nr, t, v));
        }
        return total;
    }
    static size_t bytes(int n, int nr, bool ints) {
        Carver cv(nullptr, 0);
        cv.limbs(entries(n, nr, ints));
        cv.take((size_t)36 << kLongLo);
        for (int q = 0; q < 2; ++q) cv.take((size_t)32 << kLongLo);
        return cv.used();
    }
    int build(const host::F* u, int n_, int nr_, bool ints, Carver& cv, hipStream_t stream) {
        n = n_;
        nr = nr_;
        stride = entries(n, nr, ints);
        pool = cv.limbs(stride);
        pool29 = (uint4*)cv.take((size_t)36 << kLongLo);
        lo_ops = (uint4*)cv.take((size_t)32 << kLongLo);
        rlo_ops = (uint4*)cv.take((size_t)32 << kLongLo);
        if (!pool || !pool29 || !lo_ops || !rlo_ops) return ZK_E_BUFSZ;
        EqPoolArgs args;
        memset(&args, 0, sizeof args);
        for (int t = 0; t < n; ++t) args.u[t] = to_dev(u[t]);
        uint32_t off = 0;
        auto table = [&](int var0, int nvars) {
            const int q = args.ntables++;
            args.offset[q] = off;
            args.var0[q] = (uint8_t)var0;
            args.nvars[q] = (uint8_t)nvars;
            off += 1u << nvars;
            return args.offset[q];
        };
        const uint32_t lo = table(n - kLongLo, kLongLo), rlo = table(n - kLongLo, row_low_vars(n, nr));
        for (int t = 0; n - t > kLinkPassVars; t += link_long_vars(t, ints)) {
            const int v = link_long_vars(t, ints);
            hi[t] = table(t + v, high_vars(n, t, v));
            rhi[t] = table(t + v, row_high_vars(n, nr, t, v));
        }
        args.scale = to_dev(host::from_u64(32));
        args.pool29 = pool29;
        args.count29 = (size_t)1 << kLongLo;
        args.first29 = off;
        args.scaled[args.ntables] = 1;
        table(n - kLongLo, kLongLo);
        args.total = off;
        launch_eq_pool(pool, stride, args, stream);
        hipLaunchKernelGGL(k_long_operands, dim3((1 << kLongLo) / kBlock, 2), dim3(kBlock), 0, stream, pool, stride, lo, rlo,
                           kLongLo - row_low_vars(n, nr), lo_ops, rlo_ops);
        ZK_HIP_TRY(hipGetLastError());
        return ZK_OK;
    }
    // of the pass that serves `vars` variables from t on
    LongWeights weights(int t, int vars) const {
        LongWeights w;
        w.pool = pool;
        w.stride = stride;
        w.lo29 = Planes29{pool29, (size_t)1 << kLongLo};
        w.lo_ops = lo_ops;
        w.rlo_ops = rlo_ops;
        w.hi = hi[t];
        w.rhi = rhi[t];
        w.rhi_shift = high_vars(n, t, vars) - row_high_vars(n, nr, t, vars);
        return w;
    }
};

// Positions per workgroup: as many as the weights' high factor and the sums allow, but at
// least 1024 workgroups while a wavefront has a batch for itself.
static size_t long_span(size_t P) {
    size_t span = P / 1024;
    if (span < (size_t)4 * kOuterBatch) span = (size_t)4 * kOuterBatch;
    return span < kOuterMaxSpan ? span : kOuterMaxSpan;
}
// Most partial values of a pass: the integers' first, or nine classes and four t of five sums.
static const size_t kLongValues = 16 + kLongMixed;
static size_t long_partials(int n) {
    return link_long(n, 1) ? ((size_t)1 << (n - kLongVars)) / long_span((size_t)1 << (n - kLongVars)) * kLongValues : 0;
}

static unsigned long_fold_blocks(size_t P) {
    const size_t b = P / 512;
    return (unsigned)(b < 1 ? 1 : b > 1024 ? 1024 : b);
}
static bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// ---- prover -----------------------------------------------------------------------------------

static size_t link_proof_len(int n, int K) { return 64 + (size_t)n * (K + 2) * 32 + (size_t)(2 * K + 2) * 32; }

static const int kLongEvalVars = kLongLo + 3;  // from here on on the matrix cores: eight values of the high index are an operand
static const int kLinkMleLoBits = kLongLo;  // low table of the final point's weights: up to this many variables

struct LinkWs {
    uint32_t* Y;
    uint32_t* Yk[kLinkMaxK];
    uint32_t* mle_tables;    // 2^lb + 2^(n - lb) entries, lb = min(n, kLinkMleLoBits)
    uint32_t* mle_partials;  // K 2^(n - lb) entries
    size_t mle_entries;
    uint4* mle_ops;          // the low table as operands (tensors of kLongEvalVars variables or more)
    uint32_t* partials;
    uint32_t* ticket;
    SmallFoldConsts* fold;  // 2 + K sets of constants of the integer path
    size_t part_blocks;
};

// Pairs per workgroup in round t: a workgroup's pairs share the high factor of
// their weights, i.e. lie in one row while row variables are being bound.
static size_t link_span(int t, int nr, int nc) {
    const int n = nr + nc;
    const size_t half = (size_t)1 << (n - t - 1);
    const int lbits = t < nr ? nc : n - t - 1;
    size_t span = half / 1024;
    if (span < (size_t)kBlock) span = (size_t)kBlock;
    if (span > ((size_t)1 << lbits)) span = (size_t)1 << lbits;
    if (span > half) span = half;
    return span;
}

static size_t link_blocks_max(int nr, int nc) {
    size_t most = 1;
    for (int t = 0; t < nr + nc; ++t) {
        size_t b = ((size_t)1 << (nr + nc - t - 1)) / link_span(t, nr, nc);
        if (b > most) most = b;
    }
    return most;
}

static void carve_link(LinkWs& w, Carver& cv, size_t D, size_t cols, int K) {
    const size_t h = D / 2 ? D / 2 : 1;
    w.Y = cv.limbs(h);
    for (int k = 0; k < K; ++k) w.Yk[k] = cv.limbs(h);
    {
        const int n = log2_floor(D), lb = n < kLinkMleLoBits ? n : kLinkMleLoBits;
        w.mle_entries = ((size_t)1 << lb) + ((size_t)1 << (n - lb));
        w.mle_tables = cv.limbs(w.mle_entries);
        w.mle_partials = cv.limbs((size_t)K << (n - lb));
        w.mle_ops = n >= kLongEvalVars ? (uint4*)cv.take((size_t)32 << kLongLo) : nullptr;
    }
    w.part_blocks = link_blocks_max(log2_floor(D / cols), log2_floor(cols));
    w.partials = cv.limbs(std::max({w.part_blocks * (K + 5), (size_t)kLinkGridValues * kGridChunks, long_partials(log2_floor(D))}));
    w.ticket = (uint32_t*)cv.take(256);
    w.fold = (SmallFoldConsts*)cv.take(sizeof(SmallFoldConsts) * 2);
}

static size_t link_ws_bytes(size_t rows, size_t cols, int K) {
    Carver cv(nullptr, 0);
    LinkWs w;
    carve_link(w, cv, rows * cols, cols, K);
    const int nr = log2_floor(rows), n = nr + log2_floor(cols);
    cv.limbs(LinkTables::entries(nr, n - nr));
    if (link_long(n, K)) cv.take(std::max(LongTables::bytes(n, nr, false), LongTables::bytes(n, nr, true)));
    cv.take(mle_scratch_bytes(log2_floor(rows)));
    return cv.used();
}

// Value at X = npts of the polynomial of degree < npts through y[0..npts) at 0..npts-1.
static host::F extrapolate_next(const host::F* y, int npts) {
    using namespace host;
    F d[8];
    for (int j = 0; j < npts; ++j) d[j] = y[j];
    // the npts-th forward difference vanishes: y[npts] = sum of the last entries of the difference table
    F next = zero();
    for (int level = 0; level < npts; ++level) {
        next = add(next, d[npts - 1 - level]);
        for (int j = 0; j + 1 < npts - level; ++j) d[j] = sub(d[j + 1], d[j]);
    }
    return next;
}

// Value at x of the polynomial of degree < npts through y[j] at X = j (Newton's
// forward differences: p(x) = sum_j (Delta^j y)(0) binom(x, j)).
static host::F newton_at(const host::F* y, int npts, const host::F& x) {
    using namespace host;
    static const F inv_small[8] = {zero(), one(), inv(from_u64(2)), inv(from_u64(3)), inv(from_u64(4)),
                                   inv(from_u64(5)), inv(from_u64(6)), inv(from_u64(7))};
    F d[8];
    for (int j = 0; j < npts; ++j) d[j] = y[j];
    for (int level = 1; level < npts; ++level)
        for (int j = npts - 1; j >= level; --j) d[j] = sub(d[j], d[j - 1]);
    F acc = d[0], binom = one();
    for (int j = 1; j < npts; ++j) {
        binom = mul(mul(binom, sub(x, from_u64((uint64_t)(j - 1)))), inv_small[j]);
        acc = add(acc, mul(d[j], binom));
    }
    return acc;
}

// The tensors as device arrays of integers (zkattn_link_prove_small).
struct LinkSmallIn {
    const int64_t* Zp;
    const uint32_t* const* X;
    const uint64_t* Y;
    const uint32_t* const* Yk;
    const uint64_t* bases;
};

static SmallFoldConsts small_fold_consts(const host::F& scale, const host::F& rho) {
    using namespace host;
    const F two32 = from_u64((uint64_t)1 << 32);
    const F a = mul(scale, mul(two32, two32)), d = mul(a, rho);
    SmallFoldConsts k;
    to_device_limbs(k.plus_a, a);
    to_device_limbs(k.minus_a, neg(a));
    to_device_limbs(k.plus_d, d);
    to_device_limbs(k.minus_d, neg(d));
    return k;
}

// The rounds left to the host: the arrays, and the weights of the round to come, of all its later variables (w)
// and of the row variables among them (rw).
template <int K>
struct LinkHost {
    static const size_t kMax = (size_t)1 << kLinkHostVars;
    host::F Y[kMax], Yk[K][kMax], w[kMax / 2], rw[kMax / 2];

    // round t of n variables, the first nr of them row variables
    void weights(const host::F* u, int t, int n, int nr) {
        using namespace host;
        w[0] = rw[0] = one();
        for (int v = t + 1; v < n; ++v)
            for (size_t e = (size_t)1 << (v - t - 1); e-- > 0;) {
                const F hi = mul(w[e], u[v]), rhi = v < nr ? mul(rw[e], u[v]) : rw[e];
                w[2 * e + 1] = hi;
                w[2 * e] = sub(w[e], hi);
                rw[2 * e + 1] = rhi;
                rw[2 * e] = v < nr ? sub(rw[e], rhi) : rw[e];
            }
    }
    void sums(size_t half, host::F L[2], host::F Q[K + 1], host::F s[2]) const {
        using namespace host;
        L[0] = L[1] = s[0] = s[1] = zero();
        for (int X = 0; X <= K; ++X) Q[X] = zero();
        for (size_t p = 0; p < half; ++p) {
            for (int e = 0; e < 2; ++e) {
                const F& y = Y[p + e * half];
                L[e] = add(L[e], mul(w[p], y));
                s[e] = add(s[e], mul(rw[p], y));
            }
            F f[K], d[K];
            for (int k = 0; k < K; ++k) {
                f[k] = Yk[k][p];
                d[k] = sub(Yk[k][p + half], f[k]);
            }
            f[0] = mul(f[0], w[p]);
            d[0] = mul(d[0], w[p]);
            for (int X = 0; X <= K; ++X) {
                F prod = f[0];
                for (int k = 1; k < K; ++k) prod = mul(prod, f[k]);
                Q[X] = add(Q[X], prod);
                for (int k = 0; k < K; ++k) f[k] = add(f[k], d[k]);
            }
        }
    }
    void bind(size_t half, const host::F& r, bool next_is_row) {
        using namespace host;
        auto fold = [&](F* x) {
            for (size_t p = 0; p < half; ++p) x[p] = add(x[p], mul(r, sub(x[p + half], x[p])));
        };
        fold(Y);
        for (int k = 0; k < K; ++k) fold(Yk[k]);
        for (size_t p = 0; p < half / 2; ++p) {  // the next variable summed out
            w[p] = add(w[p], w[p + half / 2]);
            if (next_is_row) rw[p] = add(rw[p], rw[p + half / 2]);
        }
    }
};

// small != null: the tensors come as integers (Zp, X, Y, Yk and bases are then unused).
template <int K>
static int link_prove_k(const uint8_t seed[32], fr_vec Zp, const fr_vec* X, fr_vec Y, const fr_vec* Yk, fr_vec yhat,
                        const fr_t* bases, size_t rows, size_t cols, uint8_t* proof, void* ws, size_t ws_bytes,
                        hipStream_t stream, const LinkSmallIn* small = nullptr) {
    using namespace host;
    const int nr = log2_floor(rows), nc = log2_floor(cols), n = nr + nc;
    const size_t D = rows * cols;
    constexpr int NV = K + 5, NPTS = K + 2;
    Mailbox* mb;
    ZK_TRY(mailbox_get(&mb));
    Carver cv(ws, ws_bytes);
    LinkWs w;
    carve_link(w, cv, D, cols, K);
    if (cv.overflow()) return ZK_E_BUFSZ;
    launch_fill_u32(w.ticket, 1, 0u, stream);

    F base[K];
    uint64_t dims[3] = {rows, cols, (uint64_t)K};
    uint8_t extra[32 * K];
    for (int k = 0; k < K; ++k) {
        if (small) {
            base[k] = from_u64(small->bases[k]);
        } else {
            if (!canonical_in_range(bases[k])) return ZK_E_BADARG;
            base[k] = from_canonical(bases[k]);
        }
        if (is_zero(base[k])) return ZK_E_BADARG;
        to_bytes(extra + 32 * k, base[k]);
    }
    uint32_t* bad_word = w.ticket + 16;  // within the ticket's 256 bytes
    if (small) launch_fill_u32(bad_word, 1, 0u, stream);
    Transcript tr("zkmi/zkattn-link/v1", seed, dims, 3, extra, sizeof extra);
    F u[32];
    for (int t = 0; t < n; ++t) u[t] = tr.challenge("u");

    // yhat~(u_rows)
    F cy;
    {
        Carver mcv = cv;
        const uint32_t seq = mb->next_seq();
        ZK_TRY(mle_eval_run(yhat.limbs, yhat.stride, nr, u, mcv, mb, seq, stream));
        ZK_TRY(mailbox_wait(mb, seq, stream));
        cy = from_dev(mb->words);
    }
    uint8_t* out = proof;
    memcpy(out, "ZKAL", 4);
    out[4] = 1; out[5] = out[6] = out[7] = 0;
    put_le64(out + 8, rows);
    put_le64(out + 16, cols);
    put_le64(out + 24, (uint64_t)K);
    to_bytes(out + 32, cy);
    tr.absorb("yhat", out + 32, 32);
    out += 64;
    const F alpha = tr.challenge("alpha");
    if (is_zero(alpha)) {  // the scaled Y could not be scaled back (probability 1/|F|)
        ZK_HIP_TRY(hipStreamSynchronize(stream));
        return ZK_E_ZERO_DENOM;
    }
    F claim = mul(sqr(alpha), cy);

    LinkTables lt;
    ZK_TRY(link_tables_build(lt, u, nr, nc, cv, stream));
    const bool long_rounds = link_long(n, K);
    LongTables lw;
    if (long_rounds) ZK_TRY(lw.build(u, n, nr, small != nullptr, cv, stream));

    F c = one();      // prod_{s<t} e~(u_s, r_s)
    F c_rows = one(); // its value once the row variables are bound
    F r_prev = zero();
    F point[32];      // the challenges: where the final claims are
    F r_last[3] = {zero(), zero(), zero()};  // the last three of them, the last one in [2]
    F prev_L[2], prev_s[2], prev_Q[K + 1];   // the last round's sums
    int pending = 0;  // of them, those that the arrays in the workspace have yet to be bound to
    int pass_left = 0;
    bool passes = false;  // a pass of grid_dev.h has run
    HostGrid gq;
    HostLine gl, gs, gq1;
    LinkHost<K> tail;
    bool on_host = false;
    // the arrays with the pending challenges bound, into the mailbox and to the host
    auto ship = [&](int t) -> int {
        const size_t count = (size_t)1 << (n - t);
        GridPass pass;
        pass.challenges(r_last);
        for (int q = 0; q <= K; ++q)
            pass.add_fold(q ? w.Yk[q - 1] : w.Y, D / 2, mb->words + kMailboxShip + 8 * count * q, 0, count, pending, true);
        const uint32_t seq = mb->next_seq();
        ZK_TRY(pass.launch_folds(mb, seq, w.ticket, stream));
        ZK_TRY(mailbox_wait(mb, seq, stream));
        const uint32_t* at = mb->words + kMailboxShip;
        for (int q = 0; q <= K; ++q)
            for (size_t j = 0; j < count; ++j, at += 8) (q ? tail.Yk[q - 1] : tail.Y)[j] = from_dev(at);
        if (t < n) tail.weights(u, t, n, nr);
        on_host = true;
        return ZK_OK;
    };
    // The long rounds' passes (link_long.h).  The arrays, 2^left elements each, with the pending challenges bound:
    bool moved = false;  // they are in the workspace, Y scaled by alpha
    const F two256 = F{{kRR[0], kRR[1], kRR[2], kRR[3]}};
    auto long_fold = [&](int left) -> int {
        if constexpr (K <= 2) {
            const size_t P = (size_t)1 << left;
            const dim3 grid(long_fold_blocks(P), K + 1);
            if (small && !moved) {
                LongFoldIntsArgs f;
                memset(&f, 0, sizeof f);
                f.Y = small->Y;
                f.vec[0] = aligned16(small->Y);
                f.dst[0] = w.Y;
                for (int k = 0; k < K; ++k) {
                    f.Yk[k] = small->Yk[k];
                    f.vec[1 + k] = aligned16(small->Yk[k]);
                    f.dst[1 + k] = w.Yk[k];
                }
                f.ds = D / 2;
                f.P = P;
                for (int s = 0; s < 2; ++s) {
                    const F scale = s ? mul(alpha, two256) : two256;
                    F e[1 << kLongIntVars];
                    long_constants(e, r_last, kLongIntVars, scale);
                    for (int c = 0; c < 1 << kLongIntVars; ++c) f.e[s][c] = to_dev(e[c]);
                    f.bias[s] = long_bias(scale, s ? 8 : 4, 2);
                }
                hipLaunchKernelGGL(k_long_fold_ints, grid, dim3(kBlock), 0, stream, f);
            } else {
                LongFoldArgs f;
                memset(&f, 0, sizeof f);
                for (int q = 0; q <= K; ++q) {
                    uint32_t* const dst = q ? w.Yk[q - 1] : w.Y;
                    const fr_vec in = moved ? fr_vec{dst, D / 2, D / 2} : q ? Yk[q - 1] : Y;
                    f.job[q] = LongFoldJob{in.limbs, in.stride, dst, D / 2, aligned16(in.limbs) && in.stride % 4 == 0, q == 0 && !moved};
                }
                f.P = P;
                for (int s = 0; s < 2; ++s) {
                    const F scale = s ? alpha : one();
                    F e[1 << kLongVars];
                    long_constants(e, r_last, kLongVars, scale);
                    for (int c = 0; c < 1 << kLongVars; ++c) f.e[s][c] = to_dev(e[c]);
                    f.bias[s] = long_bias(scale, 32, 1 << kLongVars);
                }
                hipLaunchKernelGGL(k_long_fold, grid, dim3(kBlock), 0, stream, f);
            }
            ZK_HIP_TRY(hipGetLastError());
            moved = true;
            pending = 0;
        }
        return ZK_OK;
    };
    // the sums of the pass that starts at round t
    auto long_pass = [&](int t) -> int {
        if constexpr (K <= 2) {
            const bool ints = small && t == 0, first = t == 0;
            const int left = n - t, vars = link_long_vars(t, small != nullptr);
            if (pending) ZK_TRY(long_fold(left));
            const size_t P = (size_t)1 << (left - vars), span = long_span(P);
            const unsigned blocks = (unsigned)(P / span);
            const LongWeights weights = lw.weights(t, vars);
            const uint32_t seq = mb->next_seq();
            int lines = 0;  // arrays summed by themselves
            if (ints) {
                LongIntsArgs a;
                memset(&a, 0, sizeof a);
                a.Z = small->Zp;
                a.Y = small->Y;
                for (int k = 0; k < K; ++k) {
                    a.X[k] = small->X[k];
                    a.Yk[k] = small->Yk[k];
                    a.base[k] = small->bases[k];
                }
                a.yk_bound = K == 1 ? 0xffffffffu : 1u << 30;
                a.P = P;
                a.span = span;
                a.w = weights;
                a.partials = w.partials;
                const int nv = K == 2 ? 16 + kLongMixed : 16;
                a.pstride = (size_t)blocks * nv;
                a.bad = bad_word;
                hipLaunchKernelGGL((k_long_ints<K == 1 ? 1 : 2>), dim3(blocks), dim3(kBlock), 0, stream, a);
                hipLaunchKernelGGL(k_long_total, dim3(nv), dim3(kBlock), 0, stream, w.partials, a.pstride, blocks, mb->words, mb->words, seq, w.ticket);
            } else {
                auto vec_of = [&](int q) { return q ? (moved ? fr_vec{w.Yk[q - 1], D / 2, D / 2} : Yk[q - 1]) : moved ? fr_vec{w.Y, D / 2, D / 2} : Y; };
                fr_vec arrays[4] = {vec_of(0)};
                lines = 1;
                if (first) {
                    arrays[lines++] = Zp;
                    for (int k = 0; k < K; ++k) arrays[lines++] = X[k];
                }
                if (K == 1) arrays[lines++] = vec_of(1);
                // the classes' sums first, then those of the lines
                const int nq = K == 2 ? 9 : 0, nl = 4 * (lines + 1);
                const size_t pstride = (size_t)blocks * (nq + nl);
                if (K == 2) {
                    LongGridArgs a;
                    memset(&a, 0, sizeof a);
                    const fr_vec x = vec_of(1), y = vec_of(2);
                    a.x = x.limbs;
                    a.xs = x.stride;
                    a.y = y.limbs;
                    a.ys = y.stride;
                    a.P = P;
                    a.span = span;
                    a.w = weights;
                    a.partials = w.partials;
                    a.pstride = pstride;
                    hipLaunchKernelGGL(k_long_grid, dim3(blocks), dim3(kBlock), 0, stream, a);
                }
                auto launch_lines = [&](auto args) {
                    for (int q = 0; q < lines; ++q) {
                        args.a[q] = arrays[q].limbs;
                        args.as[q] = arrays[q].stride;
                    }
                    args.P = P;
                    args.span = span;
                    args.w = weights;
                    args.partials = w.partials + (size_t)blocks * nq;
                    args.pstride = pstride;
                    return args;
                };
                const dim3 grid(blocks, 4);
                if (lines == 1) hipLaunchKernelGGL(k_long_lines<1>, grid, dim3(kBlock), 0, stream, launch_lines(LongLinesArgs<1>()));
                else if (lines == 2) hipLaunchKernelGGL(k_long_lines<2>, grid, dim3(kBlock), 0, stream, launch_lines(LongLinesArgs<2>()));
                else hipLaunchKernelGGL(k_long_lines<4>, grid, dim3(kBlock), 0, stream, launch_lines(LongLinesArgs<4>()));
                hipLaunchKernelGGL(k_long_total, dim3(nq + nl), dim3(kBlock), 0, stream, w.partials, pstride, blocks, mb->words, mb->words, seq, w.ticket);
            }
            ZK_HIP_TRY(hipGetLastError());
            ZK_TRY(mailbox_wait(mb, seq, stream));
            gl.vars = gs.vars = gq.vars = gq1.vars = vars;
            if (ints) {
                // what the pass found entry by entry
                uint32_t bad = 0;
                ZK_HIP_TRY(hipMemcpyAsync(&bad, bad_word, 4, hipMemcpyDeviceToHost, stream));
                ZK_HIP_TRY(hipStreamSynchronize(stream));
                if (bad & 2) return ZK_E_BADARG;  // an entry outside the ranges the integer path is written for
                if (bad & 1) return ZK_E_REJECT;  // the tensors do not satisfy the relations
                // sums for v - 0x80..80, integers times weights in Montgomery form, divided by 2^256: the weights w add up to one,
                // the row weights to the number of column positions
                const F flip = from_u64(0x8080808080808080ull);
                F columns = one();
                for (int v = std::max(nr, vars); v < n; ++v) columns = add(columns, columns);
                auto value = [&](int q) { return mul(from_dev(mb->words + 8 * q), two256); };
                const int nw = K == 2 ? 8 + kLongMixed : 8;
                for (int c = 0; c < 8; ++c) {
                    const F y = add(value(c), flip);
                    gl.g[c] = mul(alpha, y);
                    gs.g[c] = mul(alpha, add(value(nw + c), mul(columns, flip)));
                    gq1.g[c] = y;
                    gq.g[9 * (c >> 2) + 3 * ((c >> 1) & 1) + (c & 1)] = y;
                }
                if (K == 2) {
                    constexpr LongMixedClasses mixed;
                    for (int m = 0; m < kLongMixed; ++m) gq.g[mixed.id[m]] = add(value(8 + m), flip);
                    long_classes_to_grid(gq);
                }
            } else {
                if (K == 2) {
                    for (int i = 0; i < 9; ++i) gq.g[i] = from_dev(mb->words + 8 * i);
                    long_classes_to_grid(gq);
                }
                const uint32_t* at = mb->words + (K == 2 ? 72 : 0);
                for (int c = 0; c < 4; ++c, at += 8 * (lines + 1)) {
                    F y = from_dev(at), s = from_dev(at + 8 * lines);
                    if (K == 1) gq1.g[c] = from_dev(at + 8 * (lines - 1));
                    if (first) {
                        y = add(mul(alpha, y), from_dev(at + 8));
                        s = mul(alpha, s);
                        for (int k = 0; k < K; ++k) y = add(y, mul(base[k], from_dev(at + 8 * (2 + k))));
                    }
                    gl.g[c] = y;
                    gs.g[c] = s;
                }
            }
            pass_left = pending = vars;
        }
        return ZK_OK;
    };
    for (int t = 0; t < n; ++t) {
        const size_t half = (size_t)1 << (n - t - 1);
        const int left = n - t;
        F L0, L1, s0, s1, Q[NPTS];
        if (long_rounds && pass_left == 0 && left > kLinkPassVars) ZK_TRY(long_pass(t));
        if (K <= 2 && t >= 2 && left <= kLinkHostVars && pass_left == 0) {
            if (!on_host) ZK_TRY(ship(t));
            F L2[2], s2[2];
            tail.sums(half, L2, Q, s2);
            L0 = L2[0];
            L1 = L2[1];
            s0 = s2[0];
            s1 = s2[1];
        } else if (K <= 2 && (pass_left > 0 || (t >= 2 && left <= kLinkPassVars))) {
            if (pass_left == 0) {
                if (long_rounds && pending && !passes) ZK_TRY(long_fold(left));
                passes = true;
                const int vars = pass_left = (left - kLinkHostVars - 1) % kGridVars + 1;
                GridPass pass;
                pass.challenges(r_last);
                if (pending)
                    for (int q = 0; q <= K; ++q)
                        pass.add_fold(q ? w.Yk[q - 1] : w.Y, D / 2, q ? w.Yk[q - 1] : w.Y, D / 2, (size_t)1 << left, pending);
                const EqSplit eq = lt.round(t + vars - 1);
                const size_t P = (size_t)1 << (left - vars);
                const uint32_t at_l = pass.add(w.Y, D / 2, nullptr, 0, vars, kGridLine, P, eq);
                const uint32_t at_s = pass.add(w.Y, D / 2, nullptr, 0, vars, kGridRowLine, P, eq);
                const uint32_t at_q = K == 1 ? pass.add(w.Yk[0], D / 2, nullptr, 0, vars, kGridLine, P, eq)
                                             : pass.add(w.Yk[0], D / 2, w.Yk[K - 1], D / 2, vars, kGridTable, P, eq);
                const uint32_t seq = mb->next_seq();
                ZK_TRY(pass.launch(mb, zero(), w.partials, mb->words + kMailboxGrid, seq, w.ticket, stream));
                ZK_TRY(mailbox_wait(mb, seq, stream));
                gl.read(mb->words + kMailboxGrid + 8 * at_l, vars);
                gs.read(mb->words + kMailboxGrid + 8 * at_s, vars);
                if (K == 1) gq1.read(mb->words + kMailboxGrid + 8 * at_q, vars);
                else gq.read(mb->words + kMailboxGrid + 8 * at_q, vars);
                pending = vars;
            }
            const int later = pass_left - 1;
            F o[3];
            gl.sums(o, u + t + 1, later);
            L0 = o[0];
            L1 = o[1];
            gs.sums(o, u + t + 1, std::max(0, std::min(later, nr - t - 1)));
            s0 = o[0];
            s1 = o[1];
            if (K == 1) {
                gq1.sums(Q, u + t + 1, later);
            } else {
                gq.sums(o, u + t + 1);
                Q[0] = o[0];
                Q[1] = o[1];
                Q[K] = add(sub(add(o[1], o[1]), o[0]), add(o[2], o[2]));  // at 2, from the leading coefficient
            }
        } else {
            const EqSplit eq = lt.round(t);
            const size_t span = link_span(t, nr, nc);
            const unsigned blocks = (unsigned)(half / span);
            if (blocks > w.part_blocks) return ZK_E_BUFSZ;
            LinkRoundArgs<K> g;
            memset(&g, 0, sizeof g);
            // sources: the caller's tensors in the first two rounds, the workspace afterwards;
            // Z' and the X^(k) are only read by the first round
            const bool from_input = t <= 1 && !small;  // (the integer tensors have sources of their own)
            if (t == 0 && !small) g.Z = PairArray{Zp.limbs, Zp.stride, nullptr, 0};
            g.Y = PairArray{from_input ? Y.limbs : w.Y, from_input ? Y.stride : D / 2, w.Y, D / 2};
            for (int k = 0; k < K; ++k) {
                if (t == 0 && !small) g.X[k] = PairArray{X[k].limbs, X[k].stride, nullptr, 0};
                g.Yk[k] = PairArray{from_input ? Yk[k].limbs : w.Yk[k], from_input ? Yk[k].stride : D / 2, w.Yk[k], D / 2};
                g.base[k] = to_dev(base[k]);
                g.scale_x[k] = equal(base[k], one()) ? 0 : 1;
            }
            g.alpha = to_dev(alpha);
            g.half = half;
            g.block_span = span;
            g.r_prev = to_dev(r_prev);
            g.eq = eq;
            g.row_round = t < nr ? 1 : 0;
            g.partials = w.partials;
            g.pstride = w.part_blocks * NV;
            g.side = is_zero(u[t]) ? 1 : 0;  // the side that was not summed must carry weight
            if (small && t <= 1) {
                g.Zs = small->Zp;
                g.Ys = small->Y;
                for (int k = 0; k < K; ++k) {
                    g.Xs[k] = small->X[k];
                    g.Yks[k] = small->Yk[k];
                    g.base_small[k] = small->bases[k];
                }
                g.fold = w.fold;
                if (t == 1) {
                    LinkFoldConsts fc;
                    fc.c[0] = small_fold_consts(one(), r_prev);
                    fc.c[1] = small_fold_consts(alpha, r_prev);
                    hipLaunchKernelGGL(k_store_fold_consts, dim3(1), dim3(64), 0, stream, fc, w.fold, 2);
                }
                g.yk_bound = K == 1 ? 0xffffffffu : K == 2 ? 1u << 30 : 1u << 18;
                const F two32 = from_u64((uint64_t)1 << 32);
                g.raw_scale = to_dev(mul(two32, mul(two32, two32)));
                g.bad = bad_word;
            }
            if (small && t == 0) hipLaunchKernelGGL(k_link_round0_small<K>, dim3(blocks), dim3(kBlock), 0, stream, g);
            else if (small && t == 1) hipLaunchKernelGGL((k_link_round<K, true, true>), dim3(blocks), dim3(kBlock), 0, stream, g);
            else if (t == 0) hipLaunchKernelGGL(k_link_round0<K>, dim3(blocks), dim3(kBlock), 0, stream, g);
            else if (t == 1) hipLaunchKernelGGL((k_link_round<K, true>), dim3(blocks), dim3(kBlock), 0, stream, g);
            else hipLaunchKernelGGL((k_link_round<K, false>), dim3(blocks), dim3(kBlock), 0, stream, g);
            const uint32_t seq = mb->next_seq();
            launch_final_sum(w.partials, g.pstride, blocks, t == 0 ? NV : LinkFoldValues<K>::count, mb->words, mb->words, seq,
                             w.ticket, stream);
            ZK_HIP_TRY(hipGetLastError());
            // while the device works: what the other side is divided by
            const F e_other = g.side ? sub(one(), u[t]) : u[t];
            const F inv_other = t == 0 ? one() : inv(e_other);
            ZK_TRY(mailbox_wait(mb, seq, stream));
            if (small && t == 0) {
                // what the first round found entry by entry
                uint32_t bad = 0;
                ZK_HIP_TRY(hipMemcpyAsync(&bad, bad_word, 4, hipMemcpyDeviceToHost, stream));
                ZK_HIP_TRY(hipStreamSynchronize(stream));
                if (bad & 2) return ZK_E_BADARG;  // an entry outside the ranges the integer path is written for
                if (bad & 1) return ZK_E_REJECT;  // the tensors do not satisfy the relations
            }

            if (t == 0) {
                L0 = from_dev(mb->words);
                L1 = from_dev(mb->words + 8);
                for (int pt = 0; pt <= K; ++pt) Q[pt] = from_dev(mb->words + 8 * (2 + pt));
                s0 = from_dev(mb->words + 8 * (K + 3));
                s1 = from_dev(mb->words + 8 * (K + 4));
            } else {
                // the round before at its challenge: its lines, and Q through its values at 0..K
                F v[5];
                for (int q = 0; q < LinkFoldValues<K>::count; ++q) v[q] = from_dev(mb->words + 8 * q);
                const F e_side = sub(one(), e_other);
                const F Lp = add(prev_L[0], mul(r_prev, sub(prev_L[1], prev_L[0])));
                const F sp = add(prev_s[0], mul(r_prev, sub(prev_s[1], prev_s[0])));
                const F Qp = newton_at(prev_Q, K + 1, r_prev);
                const F L_other = mul(sub(Lp, mul(e_side, v[0])), inv_other);
                const F s_other = t < nr ? mul(sub(sp, mul(e_side, v[1])), inv_other) : sub(sp, v[1]);
                const F Q_other = mul(sub(Qp, mul(e_side, v[2])), inv_other);
                L0 = g.side ? L_other : v[0];
                L1 = g.side ? v[0] : L_other;
                s0 = g.side ? s_other : v[1];
                s1 = g.side ? v[1] : s_other;
                Q[0] = g.side ? Q_other : v[2];
                Q[1] = g.side ? v[2] : Q_other;
                if (K == 2) Q[2] = add(sub(add(Q[1], Q[1]), Q[0]), add(v[3], v[3]));
                if (K == 3) {
                    Q[2] = v[4];
                    // third difference: 6 times the leading coefficient
                    const F c3 = add(add(v[3], v[3]), v[3]), d21 = sub(Q[2], Q[1]);
                    Q[K] = add(add(add(add(d21, d21), d21), Q[0]), add(c3, c3));
                }
            }
            pending = t >= 1 ? 1 : 0;
        }
        Q[K + 1] = extrapolate_next(Q, K + 1);
        prev_L[0] = L0;
        prev_L[1] = L1;
        prev_s[0] = s0;
        prev_s[1] = s1;
        for (int pt = 0; pt <= K; ++pt) prev_Q[pt] = Q[pt];
        F gX[NPTS];
        F e = sub(one(), u[t]), de = sub(u[t], e);  // e~(u_t, X) = (1-u_t) + X (2 u_t - 1)
        F L = L0, dL = sub(L1, L0), s = s0, ds = sub(s1, s0);
        for (int pt = 0; pt < NPTS; ++pt) {
            F ce = mul(c, e);
            F wy = t < nr ? ce : c_rows;
            gX[pt] = add(mul(ce, sub(L, mul(alpha, Q[pt]))), mul(alpha, mul(wy, s)));
            e = add(e, de);
            L = add(L, dL);
            s = add(s, ds);
        }
        if (t == 0 && !equal(add(gX[0], gX[1]), claim)) {
            ZK_HIP_TRY(hipStreamSynchronize(stream));
            return ZK_E_REJECT;  // the tensors do not satisfy the relations
        }
        for (int pt = 0; pt < NPTS; ++pt) to_bytes(out + 32 * pt, gX[pt]);
        tr.absorb("g", out, 32 * NPTS);
        out += 32 * NPTS;
        const F r = tr.challenge("r");
        c = mul(c, add(mul(sub(one(), u[t]), sub(one(), r)), mul(u[t], r)));
        if (t == nr - 1) c_rows = c;
        r_prev = r;
        point[t] = r;
        r_last[0] = r_last[1];
        r_last[1] = r_last[2];
        r_last[2] = r;
        if (pass_left > 0) {
            --pass_left;
            gl.bind(r);
            gs.bind(r);
            if (K == 1) gq1.bind(r);
            else gq.bind(r);
        } else if (on_host) {
            tail.bind(half, r, t + 1 < nr);
        }
    }

    // -- final claims: Z' X^(0..K-1) Y Y^(0..K-1) at the point of the challenges -----------------
    {
        F fin[2 * kLinkMaxK + 2];
        const bool folded = n >= 2;  // the workspace holds Y and the Y^(k) (Y scaled) once a second round has run
        if (!folded) {
            // at most one round: everything from the tensors as they came
            FinalArgs f;
            memset(&f, 0, sizeof f);
            f.count = 2 * K + 2;
            f.r = to_dev(r_prev);
            auto src = [&](int slot, fr_vec in) {
                f.p[slot] = in.limbs;
                f.stride[slot] = in.stride;
                f.fold[slot] = n >= 1;
            };
            src(0, Zp);
            for (int k = 0; k < K; ++k) src(1 + k, X[k]);
            src(1 + K, Y);
            for (int k = 0; k < K; ++k) src(2 + K + k, Yk[k]);
            const uint32_t seq = mb->next_seq();
            hipLaunchKernelGGL(k_final_values, dim3(1), dim3(64), 0, stream, f, mb->words, mb->words, seq);
            ZK_HIP_TRY(hipGetLastError());
            ZK_TRY(mailbox_wait(mb, seq, stream));
            ZK_HIP_TRY(hipStreamSynchronize(stream));
            for (int q = 0; q < 2 * K + 2; ++q) fin[q] = from_dev(mb->words + 8 * q);
        } else {
            // Y and the Y^(k) from the folded arrays; the X^(k) by evaluating the tensors at the point;
            // Z' from them (the linear relation holds as an identity of multilinear polynomials)
            uint32_t seq;
            if (!on_host) ZK_TRY(ship(n));
            fin[1 + K] = mul(tail.Y[0], inv(alpha));  // scaled back
            for (int k = 0; k < K; ++k) fin[2 + K + k] = tail.Yk[k][0];

            const int lb = n < kLinkMleLoBits ? n : kLinkMleLoBits;
            EqPoolArgs ea;
            memset(&ea, 0, sizeof ea);
            for (int t = 0; t < n; ++t) ea.u[t] = to_dev(point[t]);
            ea.offset[0] = 0; ea.var0[0] = (uint8_t)(n - lb); ea.nvars[0] = (uint8_t)lb;        // low variables
            ea.offset[1] = 1u << lb; ea.var0[1] = 0; ea.nvars[1] = (uint8_t)(n - lb);           // high variables
            ea.ntables = 2;
            ea.total = (uint32_t)w.mle_entries;
            ea.scale = to_dev(one());
            launch_eq_pool(w.mle_tables, w.mle_entries, ea, stream);
            const EqSplit eq{w.mle_tables, w.mle_entries, 0, 1u << lb, lb, 1};
            const unsigned blocks = 1u << (n - lb);
            seq = mb->next_seq();
            if (n >= kLongEvalVars) {
                hipLaunchKernelGGL(k_long_operands, dim3((1 << kLongLo) / kBlock, 1), dim3(kBlock), 0, stream, w.mle_tables, w.mle_entries,
                                   0u, 0u, 0, w.mle_ops, w.mle_ops);
                LongEvalArgs a;
                memset(&a, 0, sizeof a);
                for (int k = 0; k < K; ++k) {
                    a.src[k] = small ? small->X[k] : X[k].limbs;
                    a.stride[k] = small ? 0 : X[k].stride;
                }
                a.lo_ops = w.mle_ops;
                a.pool = w.mle_tables;
                a.pool_stride = w.mle_entries;
                a.hi = 1u << lb;
                a.partials = w.mle_partials;
                // integers: 32 (8) values of the high index per workgroup
                const unsigned per = !small ? 1 : n >= kLongLo + 11 ? 32 : 8, groups = blocks / per;
                a.pstride = (size_t)K * groups;
                if (!small) hipLaunchKernelGGL(k_long_eval, dim3(groups, K), dim3(kBlock), 0, stream, a);
                else if (per == 32) hipLaunchKernelGGL(k_long_eval_ints<4>, dim3(groups, K), dim3(kBlock), 0, stream, a);
                else hipLaunchKernelGGL(k_long_eval_ints<1>, dim3(groups, K), dim3(kBlock), 0, stream, a);
                hipLaunchKernelGGL(k_long_total, dim3(K), dim3(kBlock), 0, stream, w.mle_partials, a.pstride, groups, mb->words, mb->words, seq, w.ticket);
            } else if (small) {
                LinkMleArgs<true> a;
                memset(&a, 0, sizeof a);
                for (int k = 0; k < K; ++k) a.src[k] = small->X[k];
                a.K = K;
                a.eq = eq;
                const F two32 = from_u64((uint64_t)1 << 32);
                a.raw_scale = to_dev(mul(two32, two32));
                a.partials = w.mle_partials;
                a.pstride = (size_t)K * blocks;
                hipLaunchKernelGGL(k_link_mle<true>, dim3(blocks, K), dim3(kBlock), 0, stream, a);
                launch_final_sum(w.mle_partials, (size_t)K * blocks, blocks, K, mb->words, mb->words, seq, w.ticket, stream);
            } else {
                LinkMleArgs<false> a;
                memset(&a, 0, sizeof a);
                for (int k = 0; k < K; ++k) { a.src[k] = X[k].limbs; a.stride[k] = X[k].stride; }
                a.K = K;
                a.eq = eq;
                a.partials = w.mle_partials;
                a.pstride = (size_t)K * blocks;
                hipLaunchKernelGGL(k_link_mle<false>, dim3(blocks, K), dim3(kBlock), 0, stream, a);
                launch_final_sum(w.mle_partials, (size_t)K * blocks, blocks, K, mb->words, mb->words, seq, w.ticket, stream);
            }
            ZK_HIP_TRY(hipGetLastError());
            ZK_TRY(mailbox_wait(mb, seq, stream));
            ZK_HIP_TRY(hipStreamSynchronize(stream));  // everything of this call has left the device
            fin[0] = zero();
            for (int k = 0; k < K; ++k) {
                fin[1 + k] = from_dev(mb->words + 8 * k);
                if (small && n >= kLongEvalVars)  // integers times weights in Montgomery form, divided by 2^256, of X - 0x80808080
                    fin[1 + k] = add(mul(fin[1 + k], two256), from_u64(0x80808080u));
                fin[0] = sub(fin[0], mul(base[k], fin[1 + k]));
            }
        }
        if (n == 0) {
            // a single entry: no round has compared the sum with the claim
            F lin = fin[0], prod = one();
            for (int k = 0; k < K; ++k) {
                lin = add(lin, mul(base[k], fin[1 + k]));
                prod = mul(prod, fin[2 + K + k]);
            }
            F val = add(add(lin, mul(alpha, sub(fin[1 + K], prod))), mul(sqr(alpha), fin[1 + K]));
            if (!equal(val, claim)) return ZK_E_REJECT;
        }
        for (int q = 0; q < 2 * K + 2; ++q) to_bytes(out + 32 * q, fin[q]);
        tr.absorb("final", out, 32 * (2 * K + 2));
    }
    return ZK_OK;
}

static int link_verify(const uint8_t seed[32], const uint8_t* proof, size_t len, size_t rows, size_t cols, int K,
                       const fr_t* bases, const zkattn_link_witness* wit, zkattn_link_claims* claims, void* ws,
                       size_t ws_bytes, hipStream_t stream) {
    using namespace host;
    const int nr = log2_floor(rows), nc = log2_floor(cols), n = nr + nc, npts = K + 2;
    const size_t D = rows * cols;
    if (len != link_proof_len(n, K) || memcmp(proof, "ZKAL\x01\0\0\0", 8) != 0) return ZK_E_REJECT;
    if (get_le64(proof + 8) != rows || get_le64(proof + 16) != cols || get_le64(proof + 24) != (uint64_t)K)
        return ZK_E_REJECT;
    F base[kLinkMaxK];
    uint8_t extra[32 * kLinkMaxK];
    for (int k = 0; k < K; ++k) {
        if (!canonical_in_range(bases[k])) return ZK_E_BADARG;
        base[k] = from_canonical(bases[k]);
        to_bytes(extra + 32 * k, base[k]);
    }
    uint64_t dims[3] = {rows, cols, (uint64_t)K};
    Transcript tr("zkmi/zkattn-link/v1", seed, dims, 3, extra, 32 * (size_t)K);
    F u[32], v[32];
    for (int t = 0; t < n; ++t) u[t] = tr.challenge("u");
    F cy;
    if (!from_bytes(&cy, proof + 32)) return ZK_E_REJECT;
    tr.absorb("yhat", proof + 32, 32);
    const F alpha = tr.challenge("alpha");
    F claim = mul(sqr(alpha), cy);
    const uint8_t* body = proof + 64;
    for (int t = 0; t < n; ++t) {
        F g[8];
        for (int X = 0; X < npts; ++X)
            if (!from_bytes(&g[X], body + 32 * X)) return ZK_E_REJECT;
        if (!equal(add(g[0], g[1]), claim)) return ZK_E_REJECT;
        tr.absorb("g", body, 32 * (size_t)npts);
        body += 32 * npts;
        v[t] = tr.challenge("r");
        claim = newton_at(g, npts, v[t]);
    }
    F fin[2 * kLinkMaxK + 2];
    for (int q = 0; q < 2 * K + 2; ++q)
        if (!from_bytes(&fin[q], body + 32 * q)) return ZK_E_REJECT;
    // the summand at the final point
    F e = one(), erow = one();
    for (int t = 0; t < n; ++t) {
        e = mul(e, add(mul(u[t], v[t]), mul(sub(one(), u[t]), sub(one(), v[t]))));
        if (t == nr - 1) erow = e;
    }
    if (nr == 0) erow = one();
    F lin = fin[0], prod = one();
    for (int k = 0; k < K; ++k) {
        lin = add(lin, mul(base[k], fin[1 + k]));
        prod = mul(prod, fin[2 + K + k]);
    }
    const F& fy = fin[1 + K];
    F val = add(mul(e, add(lin, mul(alpha, sub(fy, prod)))), mul(sqr(alpha), mul(erow, fy)));
    if (!equal(val, claim)) return ZK_E_REJECT;

    if (claims) {
        memset(claims, 0, sizeof *claims);
        claims->nvars = n;
        claims->K = K;
        claims->yhat_u = to_canonical(cy);
        claims->Zp_v = to_canonical(fin[0]);
        claims->Y_v = to_canonical(fy);
        for (int k = 0; k < K; ++k) {
            claims->X_v[k] = to_canonical(fin[1 + k]);
            claims->Yk_v[k] = to_canonical(fin[2 + K + k]);
        }
        for (int t = 0; t < n; ++t) {
            claims->u[t] = to_canonical(u[t]);
            claims->v[t] = to_canonical(v[t]);
        }
    }
    if (!wit) return ZK_OK;

    // tensors standing in for the openings: recompute the stated values from them
    Mailbox* mb;
    ZK_TRY(mailbox_get(&mb));
    if (!ws || ws_bytes < mle_scratch_bytes(n)) return ZK_E_BUFSZ;
    Carver cv(ws, ws_bytes);
    auto check = [&](fr_vec a, size_t count, int nv, const F* pt, const F& want) -> int {
        if (!a.limbs) return ZK_OK;
        if (!vec_ok(a, count)) return ZK_E_BADARG;
        Carver scratch = cv;
        uint32_t seq = mb->next_seq();
        ZK_TRY(mle_eval_run(a.limbs, a.stride, nv, pt, scratch, mb, seq, stream));
        ZK_TRY(mailbox_wait(mb, seq, stream));
        ZK_HIP_TRY(hipStreamSynchronize(stream));
        return equal(from_dev(mb->words), want) ? ZK_OK : ZK_E_REJECT;
    };
    ZK_TRY(check(wit->yhat, rows, nr, u, cy));
    ZK_TRY(check(wit->Zp, D, n, v, fin[0]));
    ZK_TRY(check(wit->Y, D, n, v, fy));
    for (int k = 0; k < K; ++k) {
        ZK_TRY(check(wit->X[k], D, n, v, fin[1 + k]));
        ZK_TRY(check(wit->Yk[k], D, n, v, fin[2 + K + k]));
    }
    return ZK_OK;
}

}  // namespace zkmi

using namespace zkmi;

extern "C" {

size_t zkattn_link_proof_bytes(size_t rows, size_t cols, size_t K) {
    if (!is_pow2(rows) || !is_pow2(cols) || K < 1 || K > (size_t)kLinkMaxK) return 0;
    return link_proof_len(log2_floor(rows) + log2_floor(cols), (int)K);
}

size_t zkattn_link_workspace_bytes(size_t rows, size_t cols, size_t K) {
    if (!is_pow2(rows) || !is_pow2(cols) || K < 1 || K > (size_t)kLinkMaxK) return 0;
    return link_ws_bytes(rows, cols, (int)K);
}

int zkattn_link_prove(const uint8_t seed[32], fr_vec Zp, const fr_vec* X, fr_vec Y, const fr_vec* Yk, fr_vec yhat,
                      const fr_t* bases, size_t rows, size_t cols, size_t K, uint8_t* proof, size_t cap, size_t* len,
                      void* ws, size_t ws_bytes, void* stream) {
    if (!seed || !X || !Yk || !bases || !is_pow2(rows) || !is_pow2(cols) || K < 1 || K > (size_t)kLinkMaxK)
        return ZK_E_BADARG;
    if (rows > ((size_t)1 << 31) / cols) return ZK_E_BADARG;
    const size_t D = rows * cols;
    if (!vec_ok(Zp, D) || !vec_ok(Y, D) || !vec_ok(yhat, rows)) return ZK_E_BADARG;
    for (size_t k = 0; k < K; ++k)
        if (!vec_ok(X[k], D) || !vec_ok(Yk[k], D)) return ZK_E_BADARG;
    const size_t need = link_proof_len(log2_floor(rows) + log2_floor(cols), (int)K);
    if (len) *len = need;
    if (!proof || cap < need) return ZK_E_BUFSZ;
    if (!ws || ws_bytes < link_ws_bytes(rows, cols, (int)K)) return ZK_E_BUFSZ;
    hipStream_t s = as_stream(stream);
    switch (K) {
        case 1: return link_prove_k<1>(seed, Zp, X, Y, Yk, yhat, bases, rows, cols, proof, ws, ws_bytes, s);
        case 2: return link_prove_k<2>(seed, Zp, X, Y, Yk, yhat, bases, rows, cols, proof, ws, ws_bytes, s);
        default: return link_prove_k<3>(seed, Zp, X, Y, Yk, yhat, bases, rows, cols, proof, ws, ws_bytes, s);
    }
}

int zkattn_link_prove_small(const uint8_t seed[32], const int64_t* Zp, const uint32_t* const* X, const uint64_t* Y,
                            const uint32_t* const* Yk, fr_vec yhat, const uint64_t* bases, size_t rows, size_t cols, size_t K,
                            uint8_t* proof, size_t cap, size_t* len, void* ws, size_t ws_bytes, void* stream) {
    if (!seed || !Zp || !X || !Y || !Yk || !bases || !is_pow2(rows) || !is_pow2(cols) || K < 1 || K > (size_t)kLinkMaxK)
        return ZK_E_BADARG;
    if (rows > ((size_t)1 << 31) / cols || rows * cols < 4) return ZK_E_BADARG;  // two rounds read the integers
    if (!vec_ok(yhat, rows)) return ZK_E_BADARG;
    for (size_t k = 0; k < K; ++k)
        if (!X[k] || !Yk[k] || bases[k] == 0 || bases[k] >= ((uint64_t)1 << 32)) return ZK_E_BADARG;
    const size_t need = link_proof_len(log2_floor(rows) + log2_floor(cols), (int)K);
    if (len) *len = need;
    if (!proof || cap < need) return ZK_E_BUFSZ;
    if (!ws || ws_bytes < link_ws_bytes(rows, cols, (int)K)) return ZK_E_BUFSZ;
    hipStream_t s = as_stream(stream);
    const LinkSmallIn in{Zp, X, Y, Yk, bases};
    const fr_vec none = {nullptr, 0, 0};
    switch (K) {
        case 1: return link_prove_k<1>(seed, none, nullptr, none, nullptr, yhat, nullptr, rows, cols, proof, ws, ws_bytes, s, &in);
        case 2: return link_prove_k<2>(seed, none, nullptr, none, nullptr, yhat, nullptr, rows, cols, proof, ws, ws_bytes, s, &in);
        default: return link_prove_k<3>(seed, none, nullptr, none, nullptr, yhat, nullptr, rows, cols, proof, ws, ws_bytes, s, &in);
    }
}

size_t zkattn_link_verify_workspace_bytes(size_t rows, size_t cols) {
    if (!is_pow2(rows) || !is_pow2(cols)) return 0;
    return mle_scratch_bytes(log2_floor(rows) + log2_floor(cols)) + 256;
}

int zkattn_link_verify(const uint8_t seed[32], const uint8_t* proof, size_t len, size_t rows, size_t cols, size_t K,
                       const fr_t* bases, const zkattn_link_witness* witness, zkattn_link_claims* claims, void* ws,
                       size_t ws_bytes, void* stream) {
    if (!seed || !proof || !bases || !is_pow2(rows) || !is_pow2(cols) || K < 1 || K > (size_t)kLinkMaxK)
        return ZK_E_BADARG;
    if (rows > ((size_t)1 << 31) / cols) return ZK_E_BADARG;
    return link_verify(seed, proof, len, rows, cols, (int)K, bases, witness, claims, ws, ws_bytes, as_stream(stream));
}

}  // extern "C"

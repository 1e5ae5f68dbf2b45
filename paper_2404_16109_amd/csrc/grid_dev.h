// Several sumcheck rounds from one pass over the arrays.
//
// A round that binds one variable of short arrays costs a launch and a trip to the
// host and back, some 45 us, whatever it computes.  But what the next V rounds need
// is a handful of sums that do not depend on their challenges.  With the arrays as
// functions of V variables t and the position p of what is left,
//   G(t) = sum_p w_p X(t, p) Y(t, p)
// is of degree two in every t_i, so its values on the grid {0, 1, inf}^V (inf: the
// leading coefficient, for which the entries at 0 and 1 enter by their difference)
// determine it: a round's sums are the grid's values with the later variables summed
// over {0, 1} (weighted where the identity weights them), and a challenge r takes one
// coordinate out, G(0) + r (G(1) - G(0) + (r - 1) G(inf)).  Both are the host's, some
// fifty multiplications per pass.  A pass over V = 3 variables is three launches: the
// arrays with the last pass's variables bound (k_grid_fold), the 27 grid sums of every
// product (k_grid), the wavefronts' shares added up (k_grid_sum).
//
// Bound by latency: a wavefront does one grid point of 64 positions, which keeps the
// chain at two multiplications (three where the positions do not share their weights'
// high factor) and a reduction.  A sum is at most 128 shares (fewer where several instances
// share the room for them), so that one launch adds them up: of more than 2^13 positions a
// wavefront takes more, one after the other (four times 64 of the 2^15 in a pass over one of
// sixteen variables; with 32 shares, sixteen times, that pass took 38 us instead of 16).
// Measured, a proof of 2^20 entries with a table of 256 rows: 914 -> 766 us; three lookups
// of 2^11 to 2^18 entries under one sumcheck, whose rounds used to follow each other
// instance by instance: 2.07 -> 1.24 ms.
#pragma once
#include "common.h"
#include "reduce_dev.h"

namespace zkmi {

static const int kGridVars = 3;
static const uint32_t kGridChunks = 128;  // most shares a sum is made of (GridPass may be told fewer)

static inline uint32_t grid_points(int vars) { return vars == 0 ? 1 : vars == 1 ? 3 : vars == 2 ? 9 : 27; }

enum GridKind {
    kGridWeighted = 0,  // w_p X (Y + beta), with the sums of X over p too (one for every t in {0,1}^V)
    kGridTable = 1,     // w_p X (Y + beta)
    kGridPlain = 2,     // X Y
    kGridLine = 3,      // w_p X at every t in {0,1}^V (it is linear in each t_i)
    kGridRowLine = 4    // the same with the high factor of the weights alone (none: unweighted)
};

// X and Y: 2^vars * P elements each, position p of point c at c * P + p.
struct GridJob {
    const uint32_t* x;
    const uint32_t* y;
    size_t xs, ys;
    EqSplit eq;           // weights of the P positions
    uint32_t P;
    uint32_t span;        // positions a wavefront takes: 64 or more
    uint32_t chunks;      // wavefronts per sum
    uint32_t first_wave;  // in the launch
    uint32_t first_value;
    int vars, kind;
    int hi_by_lane;       // 64 positions do not share the high factor of their weights: every lane applies its own
    static uint32_t values(int vars, int kind) {
        return kind >= kGridLine ? 1u << vars : grid_points(vars) + (kind == kGridWeighted ? 1u << vars : 0u);
    }
};
static const int kGridMaxJobs = 24;  // three products of eight instances
struct GridArgs {
    GridJob job[kGridMaxJobs];
    int njobs;
    uint32_t waves;
    uint32_t* partials;  // value v, share c: eight words at 8 (shares v + c)
    uint32_t shares;     // of the job that has most
    Fr beta;
};

// X at a grid point: NI of its coordinates are inf.  `at`: the entry with those at 0;
// step: how far the other entries are (2^vars entries of P positions).
template <int NI>
__device__ __forceinline__ Fr grid_entry(const uint32_t* x, size_t xs, size_t at, const size_t (&step)[3]) {
    Fr v[1 << NI];
#pragma unroll
    for (int j = 0; j < 1 << NI; ++j) {
        size_t i = at;
#pragma unroll
        for (int b = 0; b < NI; ++b)
            if ((j >> b) & 1) i += step[b];
        v[j] = fr_load(x, xs, i);
    }
#pragma unroll
    for (int b = NI - 1; b >= 0; --b)
#pragma unroll
        for (int j = 0; j < 1 << b; ++j) v[j] = fr_sub(v[j + (1 << b)], v[j]);
    return v[0];
}

template <int NI>
__device__ __forceinline__ Fr grid_share(const GridJob& g, const Fr& beta, uint32_t from, uint32_t to, uint32_t base,
                                         const size_t (&step)[3]) {
    FrWide acc = fr_wide_zero();
    const uint32_t lo_mask = (1u << g.eq.lbits) - 1;
    for (uint32_t p = from + (threadIdx.x & 63); p < to; p += 64) {
        const size_t at = (size_t)base * g.P + p;
        Fr a = grid_entry<NI>(g.x, g.xs, at, step), b = grid_entry<NI>(g.y, g.ys, at, step);
        if (g.kind != kGridPlain) {
            a = fr_mul(a, fr_load(g.eq.pool, g.eq.stride, g.eq.lo_off + (p & lo_mask)));
            if (g.hi_by_lane) a = fr_mul(a, fr_load(g.eq.pool, g.eq.stride, g.eq.hi_off + (p >> g.eq.lbits)));
            if (NI == 0) b = fr_add(b, beta);
        }
        fr_wide_mac(acc, a, b);
    }
    return fr_wide_reduce(acc);
}

// One entry of X over the positions, weighted as its kind says.
__device__ __forceinline__ Fr grid_line_share(const GridJob& g, uint32_t from, uint32_t to, uint32_t entry, bool weighted) {
    Fr tot = fr_zero();
    const uint32_t lo_mask = (1u << g.eq.lbits) - 1;
    for (uint32_t p = from + (threadIdx.x & 63); p < to; p += 64) {
        Fr a = fr_load(g.x, g.xs, (size_t)entry * g.P + p);
        if (weighted && g.kind == kGridLine) a = fr_mul(a, fr_load(g.eq.pool, g.eq.stride, g.eq.lo_off + (p & lo_mask)));
        if (weighted && g.hi_by_lane) a = fr_mul(a, fr_load(g.eq.pool, g.eq.stride, g.eq.hi_off + (p >> g.eq.lbits)));
        tot = fr_add(tot, a);
    }
    return tot;
}

static __global__ void __launch_bounds__(kBlock) k_grid(GridArgs args) {
    const uint32_t wave = __builtin_amdgcn_readfirstlane(blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6));
    if (wave >= args.waves) return;
    int q = 0;
    while (q + 1 < args.njobs && wave >= args.job[q + 1].first_wave) ++q;
    const GridJob& g = args.job[q];
    const uint32_t value = (wave - g.first_wave) / g.chunks, chunk = (wave - g.first_wave) % g.chunks;
    const uint32_t from = chunk * g.span, to = from + g.span < g.P ? from + g.span : g.P;
    uint32_t points = 1;
    for (int v = 0; v < g.vars; ++v) points *= 3;
    const bool line = g.kind >= kGridLine;
    bool weighted = g.kind != kGridPlain;
    Fr tot;
    if (line) {
        tot = grid_line_share(g, from, to, value, true);
    } else if (value >= points) {  // a sum of X alone
        weighted = false;
        tot = grid_line_share(g, from, to, value - points, false);
    } else {
        // the point's coordinates, the first variable's in the highest digit and on the top bit of the entry's index
        uint32_t base = 0, rest = value;
        size_t step[3] = {0, 0, 0};
        int inf = 0;
        for (int v = 0; v < g.vars; ++v) {
            const uint32_t digit = rest % 3;
            rest /= 3;
            if (digit == 1) base |= 1u << v;
            if (digit == 2) {
                const size_t s = (size_t)g.P << v;
                if (inf == 0) step[0] = s;
                else if (inf == 1) step[1] = s;
                else step[2] = s;
                ++inf;
            }
        }
        if (inf == 0) tot = grid_share<0>(g, args.beta, from, to, base, step);
        else if (inf == 1) tot = grid_share<1>(g, args.beta, from, to, base, step);
        else if (inf == 2) tot = grid_share<2>(g, args.beta, from, to, base, step);
        else tot = grid_share<3>(g, args.beta, from, to, base, step);
    }
    tot = wave_sum(tot);
    if ((threadIdx.x & 63) == 0) {
        if (weighted && g.eq.has_hi && !g.hi_by_lane)
            tot = fr_mul(tot, fr_load(g.eq.pool, g.eq.stride, g.eq.hi_off + (from >> g.eq.lbits)));
        uint4* out = (uint4*)args.partials + 2 * ((size_t)(g.first_value + value) * args.shares + chunk);
        out[0] = make_uint4(tot.l[0], tot.l[1], tot.l[2], tot.l[3]);
        out[1] = make_uint4(tot.l[4], tot.l[5], tot.l[6], tot.l[7]);
    }
}

// Value v's shares added up, to words 8 v .. 8 v + 7 of `out` (pinned host memory): LANES
// lanes per value, 32 where that is as many as there are shares (fewer workgroups, each of
// which fences its results for the host).
struct GridSumArgs {
    uint32_t first_value[kGridMaxJobs];  // of each job,
    uint32_t chunks[kGridMaxJobs];       // and its shares
    int njobs;
    uint32_t values;
    const uint32_t* partials;
    uint32_t shares;
    uint32_t* out;
    uint32_t* words;   // the mailbox
    uint32_t* ticket;
    uint32_t seq;
};

template <int LANES>
static __global__ void __launch_bounds__(kBlock) k_grid_sum(GridSumArgs args) {
    const uint32_t value = blockIdx.x * (kBlock / LANES) + threadIdx.x / LANES, lane = threadIdx.x % LANES;
    const bool live = value < args.values;
    int q = 0;
    while (q + 1 < args.njobs && value >= args.first_value[q + 1]) ++q;
    Fr v = fr_zero();
    const uint4* at = (const uint4*)args.partials + 2 * ((size_t)value * args.shares + lane);
    if (live && lane < args.chunks[q]) {
        const uint4 lo = at[0], hi = at[1];
        v = Fr{{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w}};
    }
    if constexpr (LANES == 64) {
        static_assert(kGridChunks <= 128, "two shares to a lane");
        if (live && lane + 64 < args.chunks[q]) {
            const uint4 lo = at[128], hi = at[129];
            v = fr_add(v, Fr{{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w}});
        }
    }
    v = dpp_add_step<0x111, 0xf>(v);
    v = dpp_add_step<0x112, 0xf>(v);
    v = dpp_add_step<0x114, 0xf>(v);
    v = dpp_add_step<0x118, 0xf>(v);
    v = dpp_add_step<0x142, 0xa>(v);  // the sum of 32 lanes is in their last
    if constexpr (LANES == 64) v = dpp_add_step<0x143, 0xc>(v);
    if (live && lane == LANES - 1) {
#pragma unroll
        for (int k = 0; k < 8; ++k) args.out[8 * value + k] = v.l[k];
        mailbox_written();
    }
    if (args.seq) {
        __syncthreads();
        if (threadIdx.x == 0 && atomicAdd(args.ticket, 1u) == gridDim.x - 1) {
            *args.ticket = 0;
            mailbox_publish(args.words, args.seq);
        }
    }
}

// dst_x = sum_d e_d src_(d n + x), x < n: up to three variables bound at once, e_d =
// e~(their challenges, d).  One thread per output.  dst may be src (a thread writes the
// first of the entries it alone reads) or, `rows` set, consecutive eight-word rows in
// pinned host memory.
struct GridFoldJob {
    const uint32_t* src;
    uint32_t* dst;
    size_t ss, ds;
    uint32_t n;
    uint32_t first_block;
    int vars;  // the last `vars` challenges
    int rows;
};
static const int kGridMaxFolds = 40;  // five arrays of eight instances
struct GridFoldArgs {
    GridFoldJob job[kGridMaxFolds];
    int njobs;
    Fr e[14];          // of the last challenge (two), the last two (four), the last three (eight)
    uint32_t* words;   // the mailbox, if this launch publishes
    uint32_t* ticket;
    uint32_t seq;
};

template <int VARS>
__device__ __forceinline__ Fr grid_bound(const GridFoldJob& g, uint32_t x, const Fr* e) {
    Fr v[1 << VARS];
#pragma unroll
    for (int d = 0; d < 1 << VARS; ++d) v[d] = fr_load(g.src, g.ss, (size_t)d * g.n + x);
    FrWide acc = fr_wide_zero();
#pragma unroll
    for (int d = 0; d < 1 << VARS; ++d) fr_wide_mac(acc, v[d], e[d]);
    return fr_wide_reduce(acc);
}

static __global__ void __launch_bounds__(64) k_grid_fold(GridFoldArgs args) {
    int q = 0;
    while (q + 1 < args.njobs && blockIdx.x >= args.job[q + 1].first_block) ++q;
    const GridFoldJob& g = args.job[q];
    const uint32_t x = (blockIdx.x - g.first_block) * 64 + threadIdx.x;
    if (x < g.n) {
        Fr v;
        if (g.vars == 0) v = fr_load(g.src, g.ss, x);
        else if (g.vars == 1) v = grid_bound<1>(g, x, args.e);
        else if (g.vars == 2) v = grid_bound<2>(g, x, args.e + 2);
        else v = grid_bound<3>(g, x, args.e + 6);
        if (g.rows) {
#pragma unroll
            for (int k = 0; k < 8; ++k) g.dst[8 * (size_t)x + k] = v.l[k];
            mailbox_written();
        } else {
            fr_store(g.dst, g.ds, x, v);
        }
    }
    if (args.seq) {
        __syncthreads();
        if (threadIdx.x == 0 && atomicAdd(args.ticket, 1u) == gridDim.x - 1) {
            *args.ticket = 0;
            mailbox_publish(args.words, args.seq);
        }
    }
}

// ---- host side ----------------------------------------------------------------------

// The launches of one pass.  Jobs and folds are added instance by instance; values come
// out in the order the jobs were added.
struct GridPass {
    GridArgs grid;
    GridSumArgs sum;
    GridFoldArgs fold;
    uint32_t values = 0, fold_blocks = 0;
    const uint32_t most_chunks;  // shares per sum the partial sums have room for

    explicit GridPass(uint32_t most = kGridChunks) : most_chunks(most) {
        memset(&grid, 0, sizeof grid);
        memset(&sum, 0, sizeof sum);
        memset(&fold, 0, sizeof fold);
    }
    // Binds the `vars` (0..3) last challenges: n elements from src into dst.
    void add_fold(const uint32_t* src, size_t ss, uint32_t* dst, size_t ds, size_t n, int vars, bool rows = false) {
        fold.job[fold.njobs++] = GridFoldJob{src, dst, ss, ds, (uint32_t)n, fold_blocks, vars, rows};
        fold_blocks += (uint32_t)div_up(n, 64);
    }
    // Returns the job's first value.
    uint32_t add(const uint32_t* x, size_t xs, const uint32_t* y, size_t ys, int vars, int kind, size_t P, const EqSplit& eq) {
        GridJob& g = grid.job[grid.njobs];
        g = GridJob{x, y, xs, ys, eq, (uint32_t)P, 64, 1, grid.waves, values, vars, kind, 0};
        while ((size_t)g.span * most_chunks < P) g.span *= 2;
        g.hi_by_lane = eq.has_hi && g.span > (1u << eq.lbits);
        g.chunks = (uint32_t)div_up(P, g.span);
        sum.first_value[grid.njobs] = values;
        sum.chunks[grid.njobs++] = g.chunks;
        if (g.chunks > grid.shares) grid.shares = g.chunks;
        const uint32_t count = GridJob::values(vars, kind);
        grid.waves += count * g.chunks;
        values += count;
        return g.first_value;
    }
    // r: the last three challenges, the last one in r[2] (those not bound yet are not used)
    void challenges(const host::F r[3]) {
        using namespace host;
        F e[8] = {one()};
        for (int vars = 1; vars <= kGridVars; ++vars) {
            // one more variable in front: its zero half, then its one half
            const F& f = r[3 - vars];
            const int half = 1 << (vars - 1);
            for (int d = 0; d < half; ++d) {
                e[half + d] = mul(e[d], f);
                e[d] = sub(e[d], e[half + d]);
            }
            for (int d = 0; d < 2 * half; ++d) fold.e[(1 << vars) - 2 + d] = to_dev(e[d]);
        }
    }
    int launch_folds(Mailbox* mb, uint32_t seq, uint32_t* ticket, hipStream_t stream) {
        if (fold.njobs == 0) return ZK_OK;
        fold.words = mb->words;
        fold.ticket = ticket;
        fold.seq = seq;
        hipLaunchKernelGGL(k_grid_fold, dim3(fold_blocks), dim3(64), 0, stream, fold);
        ZK_HIP_TRY(hipGetLastError());
        return ZK_OK;
    }
    int launch(Mailbox* mb, const host::F& beta, uint32_t* partials, uint32_t* out, uint32_t seq, uint32_t* ticket,
               hipStream_t stream) {
        ZK_TRY(launch_folds(mb, 0, ticket, stream));
        grid.partials = partials;
        grid.beta = to_dev(beta);
        sum.njobs = grid.njobs;
        sum.values = values;
        sum.partials = partials;
        sum.shares = grid.shares;
        sum.out = out;
        sum.words = mb->words;
        sum.ticket = ticket;
        sum.seq = seq;
        hipLaunchKernelGGL(k_grid, dim3((grid.waves + 3) / 4), dim3(kBlock), 0, stream, grid);
        if (grid.shares <= 32) hipLaunchKernelGGL(k_grid_sum<32>, dim3((values + 7) / 8), dim3(kBlock), 0, stream, sum);
        else hipLaunchKernelGGL(k_grid_sum<64>, dim3((values + 3) / 4), dim3(kBlock), 0, stream, sum);
        ZK_HIP_TRY(hipGetLastError());
        return ZK_OK;
    }
};

// The weights of `later` variables in {0,1}: e~(u, .) of the first `weighted` of them.
static inline void grid_later_weights(host::F w[4], const host::F* u, int later, int weighted) {
    using namespace host;
    w[0] = one();
    for (int t = 0; t < later; ++t)
        for (int e = (1 << t) - 1; e >= 0; --e) {
            const F hi = t < weighted ? mul(w[e], u[t]) : w[e];
            w[2 * e] = t < weighted ? sub(w[e], hi) : w[e];
            w[2 * e + 1] = hi;
        }
}

// One product's grid on the host, coordinate by coordinate.
struct HostGrid {
    host::F g[27];
    int vars = 0;

    void read(const uint32_t* words, int v) {
        vars = v;
        for (uint32_t i = 0; i < grid_points(v); ++i) g[i] = from_dev(words + 8 * i);
    }
    // The sums of the next round at 0, 1 and inf: over the later variables in {0,1}, weighted by e~(u, .) of
    // those (u: their coordinates) or, with u null, not.
    void sums(host::F out[3], const host::F* u) const {
        using namespace host;
        const int later = vars - 1;
        F w[4];
        if (u) grid_later_weights(w, u, later, later);
        for (int X = 0; X < 3; ++X) {
            out[X] = zero();
            for (int x = 0; x < 1 << later; ++x) {
                uint32_t at = (uint32_t)X;
                for (int t = later - 1; t >= 0; --t) at = 3 * at + ((x >> t) & 1);
                out[X] = add(out[X], u ? mul(w[x], g[at]) : g[at]);
            }
        }
    }
    void bind(const host::F& r) {
        using namespace host;
        const uint32_t rest = grid_points(vars - 1);
        const F rm = sub(r, one());
        for (uint32_t i = 0; i < rest; ++i)
            g[i] = add(g[i], mul(r, add(sub(g[rest + i], g[i]), mul(rm, g[2 * rest + i]))));
        --vars;
    }
};

// The same for a kGridLine.
struct HostLine {
    host::F g[1 << kGridVars];
    int vars = 0;

    void read(const uint32_t* words, int v) {
        vars = v;
        for (int i = 0; i < 1 << v; ++i) g[i] = from_dev(words + 8 * i);
    }
    // at 0 and 1, the later variables summed over {0,1}, the first `weighted` of them by e~(u, .)
    void sums(host::F out[2], const host::F* u, int weighted) const {
        using namespace host;
        const int later = vars - 1;
        F w[4];
        grid_later_weights(w, u, later, weighted);
        for (int X = 0; X < 2; ++X) {
            out[X] = zero();
            for (int x = 0; x < 1 << later; ++x)
                out[X] = add(out[X], weighted > 0 ? mul(w[x], g[(X << later) + x]) : g[(X << later) + x]);
        }
    }
    void bind(const host::F& r) {
        using namespace host;
        const int half = 1 << --vars;
        for (int i = 0; i < half; ++i) g[i] = add(g[i], mul(r, sub(g[half + i], g[i])));
    }
};

}  // namespace zkmi

// Product sumcheck (Section 3.3 of the paper) and the matrix-multiplication
// proof built on it (Section 6.1.1):
//   Y~(u,v) = sum_k X~(u,k) W~(k,v),  a_k = X~(u,k) = sum_i e~(u,i) X[i,k],
//                                      b_k = W~(k,v) = sum_j W[k,j] e~(v,j).
#include "internal.h"
#include "tlookup_kernels.h"
#include "grid_dev.h"
#include "outer_dev.h"
#include "transcript.h"

namespace zkmi {

struct ProductRoundArgs {
    PairArray a, b;
    size_t half;
    size_t block_span;
    Fr r_prev;
    uint32_t* partials;  // 3 values per workgroup
    size_t pstride;
};

// g(0) = sum a0 b0, g(1) = sum a1 b1 and the leading coefficient sum (a1-a0)(b1-b0).
template <bool FOLD>
__global__ void __launch_bounds__(kBlock) k_round_product(ProductRoundArgs g) {
    __shared__ uint32_t lds[4 * 3 * 8];
    Fr tot[3] = {fr_zero(), fr_zero(), fr_zero()};
    const size_t start = blockIdx.x * g.block_span;
    for (size_t p = start + threadIdx.x; p < start + g.block_span; p += kBlock) {
        Fr a0, a1, b0, b1;
        load_pair<FOLD>(g.a, p, g.half, g.r_prev, a0, a1);
        load_pair<FOLD>(g.b, p, g.half, g.r_prev, b0, b1);
        tot[0] = fr_add(tot[0], fr_mul(a0, b0));
        tot[1] = fr_add(tot[1], fr_mul(a1, b1));
        tot[2] = fr_add(tot[2], fr_mul(fr_sub(a1, a0), fr_sub(b1, b0)));
    }
    block_sum<3, 4>(tot, lds);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < 3; ++q) fr_store(g.partials, g.pstride, (size_t)blockIdx.x * 3 + q, tot[q]);
    }
}

// ---- the last rounds ------------------------------------------------------------------------
//
// Arrays of at most 2^kPassVars elements run their rounds several from one pass
// (grid_dev.h), and the very last are the host's: a round of 64 pairs is a few hundred
// multiplications, which the host does in a fraction of the forty microseconds a trip
// to it and back costs.  The arrays then go into the mailbox behind its result words,
// the last challenges bound, and the host computes the remaining rounds' sums, folds
// and the two final values -- the same sums over the same values, exact arithmetic, so
// the same bytes.  Measured, the thirteen rounds of a proof with their trips: 220 -> 95 us.
//
// Products of exactly 2^8 elements have one round more than the host takes.  A resident
// workgroup does it and the handing over in one launch: it writes the round's three sums
// to the mailbox, waits (bounded) for the challenge on the command channel, binds it and
// writes both arrays.  Every thread takes every barrier, and a wait that fails ends the
// kernel for all of them.  A pass over the one variable and a launch for the arrays are
// the other way: 58 us instead of 57 for the product alone, 122 instead of 97 for a
// matrix product of 100 x 200 x 100, where the pass's kernels queue behind the sums.
static const int kPassVars = 16;
static const int kHostVars = 7;
static const int kTailThreads = 1024;
static const size_t kHostPairs = (size_t)1 << (kHostVars - 1);
static_assert(2 * 2 * kHostPairs * 8 <= kMailboxGrid - kMailboxShip, "both arrays fit behind the result words");

struct ProductTailArgs {
    const uint32_t* a;
    size_t as;
    const uint32_t* b;
    size_t bs;
    uint32_t half;         // pairs: 2 half elements in each array, at most kTailThreads pairs
    uint32_t* words;       // mailbox: the sums at words[0..24); half elements of a, then of b, with the round's variable
                           // bound, eight words each, from words[kMailboxShip] on
    const uint32_t* cmd;
    uint32_t out_seq[2];   // the sums are there; the arrays are
    uint32_t cmd_seq;      // the challenge
    uint32_t spin_limit;
};

static __global__ void __launch_bounds__(kTailThreads) k_product_tail(ProductTailArgs g) {
    __shared__ uint32_t lds[16 * 3 * 8];
    __shared__ uint32_t sh_r[8];
    __shared__ int sh_ok;
    Fr tot[3] = {fr_zero(), fr_zero(), fr_zero()};
    if (threadIdx.x < g.half) {
        const Fr a0 = fr_load(g.a, g.as, threadIdx.x), a1 = fr_load(g.a, g.as, threadIdx.x + g.half);
        const Fr b0 = fr_load(g.b, g.bs, threadIdx.x), b1 = fr_load(g.b, g.bs, threadIdx.x + g.half);
        tot[0] = fr_mul(a0, b0);
        tot[1] = fr_mul(a1, b1);
        tot[2] = fr_mul(fr_sub(a1, a0), fr_sub(b1, b0));
    }
    block_sum<3, 16>(tot, lds);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int k = 0; k < 8; ++k) g.words[8 * q + k] = tot[q].l[k];
        mailbox_written();
        mailbox_publish(g.words, g.out_seq[0]);
        uint32_t limbs[8];
        const bool got = mailbox_receive_challenge(g.cmd, g.cmd_seq, g.spin_limit, limbs);
        if (got) {
#pragma unroll
            for (int k = 0; k < 8; ++k) sh_r[k] = limbs[k];
        }
        sh_ok = got ? 1 : 0;
    }
    __syncthreads();
    if (!sh_ok) return;  // the same for every thread
    Fr r;
#pragma unroll
    for (int k = 0; k < 8; ++k) r.l[k] = __builtin_amdgcn_readfirstlane(sh_r[k]);
    for (uint32_t t = threadIdx.x; t < 2 * g.half; t += kTailThreads) {
        const bool first = t < g.half;
        const uint32_t* arr = first ? g.a : g.b;
        const size_t stride = first ? g.as : g.bs;
        const uint32_t j = first ? t : t - g.half;
        const Fr v = fr_fold(fr_load(arr, stride, j), fr_load(arr, stride, j + g.half), r);
#pragma unroll
        for (int k = 0; k < 8; ++k) g.words[kMailboxShip + 8 * (size_t)t + k] = v.l[k];
        mailbox_written();
    }
    __syncthreads();
    if (threadIdx.x == 0) mailbox_publish(g.words, g.out_seq[1]);
}

// Launches it with fresh sequence numbers.
static int product_tail_launch(ProductTailArgs& g, Mailbox* mb, uint32_t spin_limit, hipStream_t stream) {
    g.words = mb->words;
    g.cmd = mb->cmd;
    g.out_seq[0] = mb->next_seq();
    g.out_seq[1] = mb->next_seq();
    g.cmd_seq = mb->next_cmd_seq();
    g.spin_limit = spin_limit;
    mailbox_channel_reset(mb);
    hipLaunchKernelGGL(k_product_tail, dim3(1), dim3(kTailThreads), 0, stream, g);
    ZK_HIP_TRY(hipGetLastError());
    return ZK_OK;
}

static size_t product_scratch_bytes() {
    Carver cv(nullptr, 0);
    cv.limbs((size_t)kMaxPartialBlocks * 3);
    cv.take(256);  // ticket of the final sums
    return cv.used();
}

// d rounds over a and b (2^d elements, stride given, folded in place).  The
// claim is absorbed here: either the caller's, or (claim == nullptr) the one
// the first round's sums imply, g(0) + g(1); it is written to claim_bytes.
// `out` receives d x 3 round values and the two final values.
static int product_rounds_run(host::Transcript& tr, uint32_t* a, size_t as, uint32_t* b, size_t bs, int d,
                              const host::F* claim, uint8_t* claim_bytes, uint8_t* out, Carver& cv, Mailbox* mb,
                              hipStream_t stream) {
    using namespace host;
    uint32_t* partials = cv.limbs((size_t)kMaxPartialBlocks * 3);
    uint32_t* ticket = (uint32_t*)cv.take(256);
    if (!partials || !ticket) return ZK_E_BUFSZ;
    launch_fill_u32(ticket, 1, 0u, stream);
    const size_t pstride = (size_t)kMaxPartialBlocks * 3;
    F r_prev = zero();
    bool claim_done = false;
    if (claim) {
        to_bytes(claim_bytes, *claim);
        tr.absorb("claim", claim_bytes, 32);
        claim_done = true;
    }
    auto emit_round = [&](const F& g0, const F& g1, const F& lead) {
        if (!claim_done) {
            to_bytes(claim_bytes, add(g0, g1));
            tr.absorb("claim", claim_bytes, 32);
            claim_done = true;
        }
        F g2 = add(sub(add(g1, g1), g0), add(lead, lead));
        to_bytes(out, g0);
        to_bytes(out + 32, g1);
        to_bytes(out + 64, g2);
        tr.absorb("g", out, 96);
        out += 96;
        r_prev = tr.challenge("r");
    };
    F r_last[3] = {zero(), zero(), zero()};
    auto bound = [&] {
        r_last[0] = r_last[1];
        r_last[1] = r_last[2];
        r_last[2] = r_prev;
    };
    int k = 0, pending = 0;  // pending: the last challenges that the arrays have yet to be bound to
    for (; d - k > kPassVars; ++k) {
        const size_t half = (size_t)1 << (d - k - 1);
        size_t span = half / kMaxPartialBlocks;
        if (span < (size_t)kBlock * 4) span = (size_t)kBlock * 4;
        if (span > half) span = half;
        const unsigned blocks = (unsigned)(half / span);
        ProductRoundArgs g;
        g.a = PairArray{a, as, a, as};
        g.b = PairArray{b, bs, b, bs};
        g.half = half;
        g.block_span = span;
        g.r_prev = to_dev(r_prev);
        g.partials = partials;
        g.pstride = pstride;
        if (k > 0) hipLaunchKernelGGL(k_round_product<true>, dim3(blocks), dim3(kBlock), 0, stream, g);
        else hipLaunchKernelGGL(k_round_product<false>, dim3(blocks), dim3(kBlock), 0, stream, g);
        const uint32_t seq = mb->next_seq();
        launch_final_sum(partials, pstride, blocks, 3, mb->words, mb->words, seq, ticket, stream);
        ZK_HIP_TRY(hipGetLastError());
        ZK_TRY(mailbox_wait(mb, seq, stream));
        emit_round(from_dev(mb->words), from_dev(mb->words + 8), from_dev(mb->words + 16));
        bound();
        pending = 1;
    }
    F ha[2 * kHostPairs], hb[2 * kHostPairs];
    size_t shipped;
    if (d == kHostVars + 1) {
        shipped = (size_t)1 << kHostVars;
        ProductTailArgs g{};
        g.a = a; g.as = as; g.b = b; g.bs = bs;
        g.half = (uint32_t)shipped;
        TailGuard guard{mb, stream};
        ZK_TRY(product_tail_launch(g, mb, device_spin_limit(), stream));
        guard.armed = true;
        ZK_TRY(mailbox_wait(mb, g.out_seq[0], stream));
        emit_round(from_dev(mb->words), from_dev(mb->words + 8), from_dev(mb->words + 16));
        mailbox_send_challenge(mb, g.cmd_seq, to_dev(r_prev).l);
        ZK_TRY(mailbox_wait(mb, g.out_seq[1], stream));
        guard.armed = false;
    } else {
        while (d - k > kHostVars) {
            const int left = d - k, vars = (left - kHostVars - 1) % kGridVars + 1;
            GridPass pass;
            pass.challenges(r_last);
            if (pending) {
                pass.add_fold(a, as, a, as, (size_t)1 << left, pending);
                pass.add_fold(b, bs, b, bs, (size_t)1 << left, pending);
            }
            pass.add(a, as, b, bs, vars, kGridPlain, (size_t)1 << (left - vars), EqSplit{nullptr, 0, 0, 0, 0, 0});
            const uint32_t seq = mb->next_seq();
            ZK_TRY(pass.launch(mb, zero(), partials, mb->words + kMailboxGrid, seq, ticket, stream));
            ZK_TRY(mailbox_wait(mb, seq, stream));
            HostGrid grid;
            grid.read(mb->words + kMailboxGrid, vars);
            for (int v = 0; v < vars; ++v, ++k) {
                F sums[3];
                grid.sums(sums, nullptr);
                emit_round(sums[0], sums[1], sums[2]);
                grid.bind(r_prev);
                bound();
            }
            pending = vars;
        }
        GridPass pass;
        pass.challenges(r_last);
        shipped = (size_t)1 << (d - k);
        pass.add_fold(a, as, mb->words + kMailboxShip, 0, shipped, pending, true);
        pass.add_fold(b, bs, mb->words + kMailboxShip + 8 * shipped, 0, shipped, pending, true);
        const uint32_t seq = mb->next_seq();
        ZK_TRY(pass.launch_folds(mb, seq, ticket, stream));
        ZK_TRY(mailbox_wait(mb, seq, stream));
    }
    ZK_HIP_TRY(hipStreamSynchronize(stream));  // everything of this call has left the device
    // the host's rounds, on the arrays it has been handed
    const uint32_t* at = mb->words + kMailboxShip;
    for (size_t j = 0; j < shipped; ++j, at += 8) ha[j] = from_dev(at);
    for (size_t j = 0; j < shipped; ++j, at += 8) hb[j] = from_dev(at);
    for (size_t half = shipped / 2; half >= 1; half >>= 1) {
        F g0 = zero(), g1 = zero(), lead = zero();
        for (size_t p = 0; p < half; ++p) {
            g0 = add(g0, mul(ha[p], hb[p]));
            g1 = add(g1, mul(ha[p + half], hb[p + half]));
            lead = add(lead, mul(sub(ha[p + half], ha[p]), sub(hb[p + half], hb[p])));
        }
        emit_round(g0, g1, lead);
        for (size_t p = 0; p < half; ++p) {
            ha[p] = add(ha[p], mul(r_prev, sub(ha[p + half], ha[p])));
            hb[p] = add(hb[p], mul(r_prev, sub(hb[p + half], hb[p])));
        }
    }
    if (!claim_done) {  // d == 0: the sum is the single product
        to_bytes(claim_bytes, mul(ha[0], hb[0]));
        tr.absorb("claim", claim_bytes, 32);
    }
    to_bytes(out, ha[0]);
    to_bytes(out + 32, hb[0]);
    tr.absorb("final", out, 64);
    return ZK_OK;
}

// Host replay of d product rounds.  el: d*3 round values then 2 final values.
static bool product_rounds_check(host::Transcript& tr, const uint8_t* body, int d, host::F claim, host::F* point,
                                 host::F fin[2]) {
    using namespace host;
    for (int k = 0; k < d; ++k) {
        F g[3];
        for (int X = 0; X < 3; ++X)
            if (!from_bytes(&g[X], body + 96 * k + 32 * X)) return false;
        if (!equal(add(g[0], g[1]), claim)) return false;
        tr.absorb("g", body + 96 * k, 96);
        point[k] = tr.challenge("r");
        claim = interpolate_at(g, 3, point[k]);
    }
    if (!from_bytes(&fin[0], body + 96 * d) || !from_bytes(&fin[1], body + 96 * d + 32)) return false;
    tr.absorb("final", body + 96 * d, 64);
    return equal(mul(fin[0], fin[1]), claim);
}

// ---- partial evaluations of a matrix -------------------------------------------------------

// part[c][k] = sum over rows i of chunk c of e[i] * X[i][k]; thread per column.
__global__ void __launch_bounds__(kBlock) k_colsum_partial(const uint32_t* __restrict__ X, size_t xs, size_t D0,
                                                           size_t D1, const uint32_t* __restrict__ e, size_t es,
                                                           size_t rows_per_chunk, uint32_t* __restrict__ part,
                                                           size_t ps, size_t P1) {
    size_t k = blockIdx.x * (size_t)kBlock + threadIdx.x;
    if (k >= D1) return;
    size_t i0 = blockIdx.y * rows_per_chunk, i1 = i0 + rows_per_chunk;
    if (i1 > D0) i1 = D0;
    FrWide acc = fr_wide_zero();
    size_t i = i0;
    for (; i + 2 <= i1; i += 2) {  // two rows at a time: their loads are in flight together
        const Fr x0 = fr_load(X, xs, i * D1 + k), x1 = fr_load(X, xs, (i + 1) * D1 + k);
        fr_wide_mac(acc, x0, fr_load(e, es, i));
        fr_wide_mac(acc, x1, fr_load(e, es, i + 1));
    }
    if (i < i1) fr_wide_mac(acc, fr_load(X, xs, i * D1 + k), fr_load(e, es, i));
    fr_store(part, ps, blockIdx.y * P1 + k, fr_wide_reduce(acc));
}

// a[k] = sum_c part[c][k] for k < D1, zero for D1 <= k < P1.  Eight threads per
// column, an eighth of the chunks each (one thread's chain of 64 loads and additions
// took 26 us).
static const int kReduceColumns = kBlock / 8;
__global__ void __launch_bounds__(kBlock) k_colsum_reduce(uint32_t* __restrict__ a, size_t as,
                                                          const uint32_t* __restrict__ part, size_t ps, size_t chunks,
                                                          size_t D1, size_t P1) {
    __shared__ uint32_t lds[8 * kBlock];
    const int col = threadIdx.x % kReduceColumns, share = threadIdx.x / kReduceColumns;
    const size_t k = blockIdx.x * (size_t)kReduceColumns + col;
    Fr acc = fr_zero();
    if (k < D1) {
        size_t c = share;
        for (; c + 24 < chunks; c += 32) {
            Fr v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = fr_load(part, ps, (c + 8 * q) * P1 + k);
#pragma unroll
            for (int q = 0; q < 4; ++q) acc = fr_add(acc, v[q]);
        }
        for (; c < chunks; c += 8) acc = fr_add(acc, fr_load(part, ps, c * P1 + k));
    }
    for (int step = 4; step >= 1; step >>= 1) {
#pragma unroll
        for (int q = 0; q < 8; ++q) lds[q * kBlock + threadIdx.x] = acc.l[q];
        __syncthreads();
        if (share < step) {
            Fr o;
#pragma unroll
            for (int q = 0; q < 8; ++q) o.l[q] = lds[q * kBlock + threadIdx.x + step * kReduceColumns];
            acc = fr_add(acc, o);
        }
        __syncthreads();
    }
    if (share == 0 && k < P1) fr_store(a, as, k, acc);
}

// b[k] = sum_j W[k][j] e[j]; rows D1 <= k < P1 are zero.  One workgroup per row: matrices
// of few rows, or so small that what counts is the length of a workgroup's chain.
__global__ void __launch_bounds__(kBlock) k_rowdot_short(uint32_t* __restrict__ b, size_t bs, const uint32_t* __restrict__ W,
                                                         size_t ws, size_t D1, size_t D2, const uint32_t* __restrict__ e,
                                                         size_t es) {
    __shared__ uint32_t lds[4 * 8];
    const size_t k = blockIdx.x;
    Fr tot[1] = {fr_zero()};
    if (k < D1) {
        FrWide acc = fr_wide_zero();
        for (size_t j = threadIdx.x; j < D2; j += kBlock) fr_wide_mac(acc, fr_load(W, ws, k * D2 + j), fr_load(e, es, j));
        tot[0] = fr_wide_reduce(acc);
    }
    block_sum<1, 4>(tot, lds);
    if (threadIdx.x == 0) fr_store(b, bs, k, tot[0]);
}

// The same for larger ones (rowdot_run).  A workgroup takes four rows, its
// wavefronts every fourth batch of 64 columns; the products are added up on the matrix
// cores (outer_dev.h), 4096 columns between two reductions.  Bound by HBM: 5120 x 5120
// elements 150 us, 5.6 TB/s (202 with 512-bit sums on the vector ALU, 290 with a reduction for every
// product).
static const int kDotRows = 4;
__global__ void __launch_bounds__(kBlock) k_rowdot(uint32_t* __restrict__ b, size_t bs, const uint32_t* __restrict__ W,
                                                   size_t ws, size_t D1, size_t D2, const uint32_t* __restrict__ e,
                                                   size_t es, size_t P1) {
    __shared__ __attribute__((aligned(16))) int sums[kDotRows * 1024];
    __shared__ uint32_t tot[kDotRows][8];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint8_t* const stage = (uint8_t*)sums + wave * kOuterStage;
    const size_t k = (size_t)blockIdx.x * kDotRows;
    if (threadIdx.x < kDotRows * 8) tot[threadIdx.x >> 3][threadIdx.x & 7] = 0;
    size_t row[kDotRows];
#pragma unroll
    for (int r = 0; r < kDotRows; ++r) row[r] = (k + r < D1 ? k + r : D1 - 1) * D2;
#pragma unroll 1
    for (size_t j0 = 0; j0 < D2 && k < D1; j0 += kOuterMaxSpan) {
        const size_t end = D2 - j0 < kOuterMaxSpan ? D2 : j0 + kOuterMaxSpan;
        v16i acc[kDotRows];
#pragma unroll
        for (int r = 0; r < kDotRows; ++r) outer_clear(acc[r]);
        size_t j = j0 + (size_t)wave * kOuterBatch;
        if (j < end) {
            auto count = [&](size_t at) { return (uint32_t)(end - at < (size_t)kOuterBatch ? end - at : (size_t)kOuterBatch); };
            uint32_t v[kDotRows][8], ev[8];  // asked for a turn ahead
            outer_load_part(ev, e, es, j, count(j));
#pragma unroll
            for (int r = 0; r < kDotRows; ++r) outer_load_part(v[r], W, ws, row[r] + j, count(j));
#pragma unroll 1
            for (; j < end; j += 4 * kOuterBatch) {
                const size_t next = j + 4 * kOuterBatch < end ? j + 4 * kOuterBatch : j;
                uint32_t d[8];
                balanced_digits(d, ev);
                if ((threadIdx.x & 63) >= count(j)) {
#pragma unroll
                    for (int q = 0; q < 8; ++q) d[q] = 0;
                }
                outer_load_part(ev, e, es, next, count(next));
                __builtin_amdgcn_sched_barrier(0);
                const OuterOperand w = outer_stage(d, stage);
#pragma unroll
                for (int r = 0; r < kDotRows; ++r) {
                    balanced_digits(d, v[r]);
                    outer_load_part(v[r], W, ws, row[r] + next, count(next));
                    __builtin_amdgcn_sched_barrier(0);
                    outer_mac(acc[r], w, outer_stage(d, stage));
                }
            }
        }
        outer_close<kDotRows, 32>(acc, sums, [&](int r, int, const Fr& x) {
            Fr t;
#pragma unroll
            for (int q = 0; q < 8; ++q) t.l[q] = tot[r][q];
            t = fr_add(t, x);
#pragma unroll
            for (int q = 0; q < 8; ++q) tot[r][q] = t.l[q];
        });
        __syncthreads();  // the sums are read: the next columns are staged where they lie
    }
    if (threadIdx.x < kDotRows * 8) {
        const size_t r = threadIdx.x >> 3, q = threadIdx.x & 7;
        if (k + r < P1) b[q * bs + k + r] = k + r < D1 ? tot[r][q] : 0u;
    }
}

__global__ void __launch_bounds__(kBlock) k_dot_partial(const uint32_t* __restrict__ x, size_t xs,
                                                        const uint32_t* __restrict__ y, size_t ys, size_t n,
                                                        uint32_t* __restrict__ partials, size_t pstride) {
    __shared__ uint32_t lds[4 * 8];
    Fr acc[1] = {fr_zero()};
    for (size_t i = blockIdx.x * (size_t)kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock)
        acc[0] = fr_add(acc[0], fr_mul(fr_load(x, xs, i), fr_load(y, ys, i)));
    block_sum<1, 4>(acc, lds);
    if (threadIdx.x == 0) fr_store(partials, pstride, blockIdx.x, acc[0]);
}

// ---- the same for matrices of small integers -----------------------------------------------
//
// Quantised activations and weights are 16-bit integers.  With x' = x + 2^15 (so
// 0 <= x' < 2^16) a sum  sum_i e_i x_i  of field elements times matrix entries is
// sum_i e_i x'_i - 2^15 sum_i e_i.  A product e_i x'_i is eight 32x32-bit products
// of at most 48 bits, added limb by limb into 64-bit accumulators with no carries
// and no reduction (2^16 terms fit); the sums leave the kernels as plain 288-bit
// integers ("raw", nine 32-bit limbs, limb-major) and one small kernel reduces
// them mod r and subtracts the constant.  Per matrix entry that is eight
// multiply-adds and two bytes of traffic instead of a field multiplication and 32.
static const int kRawLimbs = 9;
static const size_t kSmallTermsMax = 1 << 15;  // terms per accumulator: 2^48 * 2^15 = 2^63

__device__ __forceinline__ void small_mac(uint64_t (&acc)[8], const Fr& e, int16_t x) {
    const uint32_t xp = (uint32_t)((int)x + 32768);
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] += (uint64_t)e.l[j] * xp;
}

// sum_j acc[j] 2^(32 j) as nine 32-bit limbs (acc[j] < 2^63).
__device__ __forceinline__ void small_normalize(uint32_t (&out)[kRawLimbs], const uint64_t (&acc)[8]) {
    uint64_t carry = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        uint64_t s = (acc[j] & 0xffffffffu) + (carry & 0xffffffffu);
        out[j] = (uint32_t)s;
        carry = (acc[j] >> 32) + (carry >> 32) + (s >> 32);
    }
    out[8] = (uint32_t)carry;  // the sum is below 2^288
}

// raw part[c][limb][k] = sum over rows i of chunk c of e[i] * (X[i][k] + 2^15); thread per column.
__global__ void __launch_bounds__(kBlock) k_colsum_partial_i16(const int16_t* __restrict__ X, size_t D0, size_t D1,
                                                               const uint32_t* __restrict__ e, size_t es,
                                                               size_t rows_per_chunk, uint32_t* __restrict__ part,
                                                               size_t P1) {
    size_t k = blockIdx.x * (size_t)kBlock + threadIdx.x;
    if (k >= D1) return;
    size_t i0 = blockIdx.y * rows_per_chunk, i1 = i0 + rows_per_chunk;
    if (i1 > D0) i1 = D0;
    uint64_t acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0;
    size_t i = i0;
    for (; i + 4 <= i1; i += 4) {  // four rows at a time: their loads are in flight together
        int16_t x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = X[(i + q) * D1 + k];
#pragma unroll
        for (int q = 0; q < 4; ++q) small_mac(acc, fr_load(e, es, i + q), x[q]);
    }
    for (; i < i1; ++i) small_mac(acc, fr_load(e, es, i), X[i * D1 + k]);
    uint32_t raw[kRawLimbs];
    small_normalize(raw, acc);
#pragma unroll
    for (int j = 0; j < kRawLimbs; ++j) part[((size_t)blockIdx.y * kRawLimbs + j) * P1 + k] = raw[j];
}

// raw rows[limb][k] = sum_j (W[k][j] + 2^15) e[j]; one wavefront per four rows, lanes over j.
static const int kRowsPerWave = 4;
__global__ void __launch_bounds__(64) k_rowdot_i16(uint32_t* __restrict__ raw_out, size_t P1, const int16_t* __restrict__ W,
                                                   size_t D1, size_t D2, const uint32_t* __restrict__ e, size_t es) {
    const size_t k0 = (size_t)blockIdx.x * kRowsPerWave;
    if (k0 >= D1) return;
    uint64_t acc[kRowsPerWave][8];
#pragma unroll
    for (int r = 0; r < kRowsPerWave; ++r)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[r][j] = 0;
    const int rows = D1 - k0 < (size_t)kRowsPerWave ? (int)(D1 - k0) : kRowsPerWave;
    size_t j = 0;
    if ((D2 & 3) == 0 && (es & 3) == 0 && (reinterpret_cast<uintptr_t>(W) & 7) == 0 && (reinterpret_cast<uintptr_t>(e) & 15) == 0) {
        // four consecutive columns per lane: eight 16-byte loads bring four elements of e
        // (limb-major: limb k of columns j..j+3 is one uint4) and one 8-byte load per row four entries of W
        for (j = 4 * (size_t)threadIdx.x; j + 3 < D2; j += 4 * 64) {
            uint4 el[8];
            uint2 xw[kRowsPerWave];
#pragma unroll
            for (int k = 0; k < 8; ++k) el[k] = *reinterpret_cast<const uint4*>(e + k * es + j);
#pragma unroll
            for (int r = 0; r < kRowsPerWave; ++r)
                xw[r] = r < rows ? *reinterpret_cast<const uint2*>(W + (k0 + r) * D2 + j) : make_uint2(0x80008000u, 0x80008000u);
            Fr ej[4];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                ej[0].l[k] = el[k].x;
                ej[1].l[k] = el[k].y;
                ej[2].l[k] = el[k].z;
                ej[3].l[k] = el[k].w;
            }
#pragma unroll
            for (int r = 0; r < kRowsPerWave; ++r) {
                small_mac(acc[r], ej[0], (int16_t)(xw[r].x & 0xffffu));
                small_mac(acc[r], ej[1], (int16_t)(xw[r].x >> 16));
                small_mac(acc[r], ej[2], (int16_t)(xw[r].y & 0xffffu));
                small_mac(acc[r], ej[3], (int16_t)(xw[r].y >> 16));
            }
        }
        j = D2;  // D2 is a multiple of four: the loop above has covered every column
    }
    for (j += threadIdx.x; j < D2; j += 64) {
        const Fr ej = fr_load(e, es, j);
#pragma unroll
        for (int r = 0; r < kRowsPerWave; ++r)
            if (r < rows) small_mac(acc[r], ej, W[(k0 + r) * D2 + j]);
    }
    // the wavefront's sum of a limb is below 2^48 * D2 <= 2^63 (the caller keeps D2 <= 2^15)
#pragma unroll
    for (int r = 0; r < kRowsPerWave; ++r) {
#pragma unroll
        for (int limb = 0; limb < 8; ++limb) {
            uint64_t v = acc[r][limb];
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) v += __shfl_down(v, off, 64);
            acc[r][limb] = v;
        }
    }
    if (threadIdx.x == 0) {
#pragma unroll
        for (int r = 0; r < kRowsPerWave; ++r) {
            if (k0 + r >= D1) break;
            uint32_t raw[kRawLimbs];
            small_normalize(raw, acc[r]);
#pragma unroll
            for (int limb = 0; limb < kRawLimbs; ++limb) raw_out[(size_t)limb * P1 + k0 + r] = raw[limb];
        }
    }
}

// dst[k] = (sum over `chunks` raw values of entry k) mod r - 2^15 * (*esum), zero for
// k >= count: both products' sums in one launch (blockIdx.y).
struct SmallFinishArgs {
    struct Job {
        uint32_t* dst;
        const uint32_t* raw;
        size_t chunks, count;
        const uint32_t* esum;
    } job[2];
    size_t P;
};
__global__ void __launch_bounds__(kBlock) k_small_finish(SmallFinishArgs g) {
    const auto& job = g.job[blockIdx.y];
    uint32_t* const dst = job.dst;
    const uint32_t* const raw = job.raw;
    const uint32_t* const esum = job.esum;
    const size_t P = g.P, ds = g.P, chunks = job.chunks, count = job.count;
    size_t k = blockIdx.x * (size_t)kBlock + threadIdx.x;
    if (k >= P) return;
    if (k >= count) {
        fr_store(dst, ds, k, fr_zero());
        return;
    }
    uint64_t limb[kRawLimbs];
#pragma unroll
    for (int j = 0; j < kRawLimbs; ++j) limb[j] = 0;
    size_t c = 0;
    for (; c + 8 <= chunks; c += 8) {  // eight chunks per trip: 72 loads in flight
        uint32_t v[8][kRawLimbs];
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int j = 0; j < kRawLimbs; ++j) v[q][j] = raw[((c + q) * kRawLimbs + j) * P + k];
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int j = 0; j < kRawLimbs; ++j) limb[j] += v[q][j];
    }
    for (; c < chunks; ++c)
#pragma unroll
        for (int j = 0; j < kRawLimbs; ++j) limb[j] += raw[(c * kRawLimbs + j) * P + k];
    // carry: the total is below 2^288 * chunks, chunks <= 2^16
    Fr lo, hi = fr_zero();
    uint64_t carry = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        uint64_t s = limb[j] + carry;
        lo.l[j] = (uint32_t)s;
        carry = s >> 32;
    }
    uint64_t top = limb[8] + carry;
    hi.l[0] = (uint32_t)top;
    hi.l[1] = (uint32_t)(top >> 32);
    // lo (any value below 2^256) mod r = lo * 2^512 / 2^256 / 2^256; hi * 2^256 mod r = hi * 2^512 / 2^256
    Fr one_raw = fr_zero();
    one_raw.l[0] = 1;
    Fr sum = fr_add(fr_mul(fr_mul(lo, fr_rr()), one_raw), fr_mul(hi, fr_rr()));
    Fr shift = fr_zero();
    shift.l[0] = 32768;
    shift = fr_mul(shift, fr_rr());  // 2^15 in Montgomery form
    fr_store(dst, ds, k, fr_sub(sum, fr_mul(shift, fr_load(esum, 1, 0))));
}

// out[8 b .. 8 b + 7] (Montgomery limbs of one element) = sum_{i < n_b} e_b[i], workgroup b = 0, 1.
__global__ void __launch_bounds__(1024) k_sum_two(uint32_t* __restrict__ out, const uint32_t* __restrict__ e0, size_t es0, size_t n0,
                                                  const uint32_t* __restrict__ e1, size_t es1, size_t n1) {
    __shared__ uint32_t lds[16 * 8];
    const uint32_t* const e = blockIdx.x ? e1 : e0;
    const size_t es = blockIdx.x ? es1 : es0, n = blockIdx.x ? n1 : n0;
    Fr acc[1] = {fr_zero()};
    for (size_t i = threadIdx.x; i < n; i += 1024) acc[0] = fr_add(acc[0], fr_load(e, es, i));
    block_sum<1, 16>(acc, lds);
    if (threadIdx.x == 0) fr_store(out + 8 * blockIdx.x, 1, 0, acc[0]);
}

static const size_t kColChunks = 64;

struct MatmulWs {
    uint32_t *eu, *ev, *a, *b, *part, *dot;
    size_t P0, P1, P2;
};

static void carve_matmul(MatmulWs& w, Carver& cv, size_t D0, size_t D1, size_t D2) {
    w.P0 = (size_t)1 << log2_ceil(D0);
    w.P1 = (size_t)1 << log2_ceil(D1);
    w.P2 = (size_t)1 << log2_ceil(D2);
    w.eu = cv.limbs(w.P0);
    w.ev = cv.limbs(w.P2);
    w.a = cv.limbs(w.P1);
    w.b = cv.limbs(w.P1);
    size_t widest = w.P1 > w.P2 ? w.P1 : w.P2;
    // chunk sums as field elements (8 words each) or raw (9 words each, plus one element)
    w.part = cv.limbs(2 * kColChunks * widest + 8);
    w.dot = cv.limbs(kMaxPartialBlocks);
}

// a_k = sum_i e0[i] M[i][k] over an R x C row-major matrix, into `a` (PC entries, zero padded).
static void colsum_run(uint32_t* a, size_t PC, const uint32_t* M, size_t ms, size_t R, size_t C, const uint32_t* e0,
                       size_t e0s, uint32_t* part, hipStream_t stream) {
    size_t rows_per_chunk = div_up(R, kColChunks);
    size_t chunks = div_up(R, rows_per_chunk);
    hipLaunchKernelGGL(k_colsum_partial, dim3((unsigned)div_up(C, kBlock), (unsigned)chunks), dim3(kBlock), 0, stream, M,
                       ms, R, C, e0, e0s, rows_per_chunk, part, kColChunks * PC, PC);
    hipLaunchKernelGGL(k_colsum_reduce, dim3((unsigned)div_up(PC, kReduceColumns)), dim3(kBlock), 0, stream, a, PC, part,
                       kColChunks * PC, chunks, C, PC);
}

// a_k = sum_i eu[i] X[i][k] over R x C and b_k = sum_j W[k][j] ev[j] over C x C2, 16-bit entries, into a and b (PC entries).
// scratch: kColChunks raw chunks of the first, one of the second, the two sums of weights.
static void small_products_run(uint32_t* a, uint32_t* b, size_t PC, const int16_t* X, size_t R, size_t C, const uint32_t* eu,
                               size_t eus, const int16_t* W, size_t C2, const uint32_t* ev, size_t evs, uint32_t* scratch,
                               hipStream_t stream) {
    const size_t rows_per_chunk = div_up(R, kColChunks), chunks = div_up(R, rows_per_chunk);
    uint32_t* raw_a = scratch;
    uint32_t* raw_b = raw_a + kColChunks * kRawLimbs * PC;
    uint32_t* esums = raw_b + kRawLimbs * PC;
    hipLaunchKernelGGL(k_sum_two, dim3(2), dim3(1024), 0, stream, esums, eu, eus, R, ev, evs, C2);
    hipLaunchKernelGGL(k_colsum_partial_i16, dim3((unsigned)div_up(C, kBlock), (unsigned)chunks), dim3(kBlock), 0, stream, X,
                       R, C, eu, eus, rows_per_chunk, raw_a, PC);
    hipLaunchKernelGGL(k_rowdot_i16, dim3((unsigned)div_up(C, kRowsPerWave)), dim3(64), 0, stream, raw_b, PC, W, C, C2, ev, evs);
    SmallFinishArgs g;
    g.job[0] = {a, raw_a, chunks, C, esums};
    g.job[1] = {b, raw_b, 1, C, esums + 8};
    g.P = PC;
    hipLaunchKernelGGL(k_small_finish, dim3((unsigned)div_up(PC, kBlock), 2), dim3(kBlock), 0, stream, g);
}

static void rowdot_run(uint32_t* b, size_t PR, const uint32_t* M, size_t ms, size_t R, size_t C, const uint32_t* e1,
                       size_t e1s, hipStream_t stream) {
    // A workgroup of k_rowdot does four rows: of few rows it leaves compute units idle, of short ones there is nothing to
    // gain.  Whole proofs with eight rows of X, a workgroup per row of W and four rows per workgroup: 128 x 32768: 164 and
    // 228 us, 512 x 32768: 266 and 281, 768 x 32768: 313 and 289, 5120 x 5120: 314 and 289, 1024 x 4096: 142 and 132,
    // 1024 x 1024: 119 and 116, 768 x 1024: alike, 1024 x 128: alike
    if (R < 768 || R * C < (size_t)1 << 20)
        hipLaunchKernelGGL(k_rowdot_short, dim3((unsigned)PR), dim3(kBlock), 0, stream, b, PR, M, ms, R, C, e1, e1s);
    else hipLaunchKernelGGL(k_rowdot, dim3((unsigned)div_up(PR, kDotRows)), dim3(kBlock), 0, stream, b, PR, M, ms, R, C, e1, e1s, PR);
}

static int dot_run(const uint32_t* x, size_t xs, const uint32_t* y, size_t ys, size_t n, uint32_t* partials,
                   uint32_t* out_words, hipStream_t stream) {
    unsigned blocks = grid_for(n, kBlock * 4, kMaxPartialBlocks);
    hipLaunchKernelGGL(k_dot_partial, dim3(blocks), dim3(kBlock), 0, stream, x, xs, y, ys, n, partials,
                       (size_t)kMaxPartialBlocks);
    launch_final_sum(partials, kMaxPartialBlocks, blocks, 1, out_words, out_words, 0, nullptr, stream);
    ZK_HIP_TRY(hipGetLastError());
    return ZK_OK;
}

}  // namespace zkmi

using namespace zkmi;

extern "C" {

size_t sumcheck_product_proof_bytes(size_t n) { return 16 + 32 + (size_t)log2_floor(n ? n : 1) * 96 + 64; }
size_t sumcheck_product_workspace_bytes(size_t) { return product_scratch_bytes(); }

int sumcheck_prove_product(const uint8_t seed[32], fr_vec a, fr_vec b, const fr_t* claim, uint8_t* proof, size_t cap,
                           size_t* len, void* ws, size_t ws_bytes, void* stream) {
    const size_t n = a.n;
    if (!seed || !claim || !is_pow2(n) || b.n != n || !vec_ok(a, n) || !vec_ok(b, n)) return ZK_E_BADARG;
    if (n > ((size_t)1 << 31) || !host::canonical_in_range(*claim)) return ZK_E_BADARG;
    const int d = log2_floor(n);
    const size_t need = sumcheck_product_proof_bytes(n);
    if (len) *len = need;
    if (!proof || cap < need) return ZK_E_BUFSZ;
    if (!ws || ws_bytes < product_scratch_bytes()) return ZK_E_BUFSZ;
    Mailbox* mb;
    ZK_TRY(mailbox_get(&mb));
    Carver cv(ws, ws_bytes);
    uint64_t dims[1] = {(uint64_t)d};
    host::Transcript tr("zkmi/sumcheck-product/v1", seed, dims, 1);
    memcpy(proof, "ZKSP\x01\0\0\0", 8);
    host::put_le64(proof + 8, (uint64_t)d);
    host::F c = host::from_canonical(*claim);
    return product_rounds_run(tr, a.limbs, a.stride, b.limbs, b.stride, d, &c, proof + 16, proof + 48, cv, mb,
                              as_stream(stream));
}

int sumcheck_verify_product(const uint8_t seed[32], const uint8_t* proof, size_t len, size_t n, fr_t final_claims[2],
                            fr_t* point) {
    if (!seed || !proof || !is_pow2(n) || n > ((size_t)1 << 31)) return ZK_E_BADARG;
    const int d = log2_floor(n);
    if (len != sumcheck_product_proof_bytes(n)) return ZK_E_REJECT;
    if (memcmp(proof, "ZKSP\x01\0\0\0", 8) != 0 || host::get_le64(proof + 8) != (uint64_t)d) return ZK_E_REJECT;
    host::F claim;
    if (!host::from_bytes(&claim, proof + 16)) return ZK_E_REJECT;
    uint64_t dims[1] = {(uint64_t)d};
    host::Transcript tr("zkmi/sumcheck-product/v1", seed, dims, 1);
    tr.absorb("claim", proof + 16, 32);
    host::F pt[32], fin[2];
    if (!product_rounds_check(tr, proof + 48, d, claim, pt, fin)) return ZK_E_REJECT;
    if (final_claims) {
        final_claims[0] = host::to_canonical(fin[0]);
        final_claims[1] = host::to_canonical(fin[1]);
    }
    if (point)
        for (int k = 0; k < d; ++k) point[k] = host::to_canonical(pt[k]);
    return ZK_OK;
}

size_t matmul_proof_bytes(size_t D1) { return 32 + 32 + (size_t)log2_ceil(D1 ? D1 : 1) * 96 + 64; }

size_t matmul_workspace_bytes(size_t D0, size_t D1, size_t D2) {
    if (!D0 || !D1 || !D2) return 0;
    Carver cv(nullptr, 0);
    MatmulWs w;
    carve_matmul(w, cv, D0, D1, D2);
    cv.limbs((size_t)kMaxPartialBlocks * 3);  // round partial sums (prover)
    cv.take(256);                             // ticket of the final sums
    cv.limbs(w.P2);                           // column sums of Y (verifier)
    cv.limbs(w.P1);                           // e~(r, .) (verifier)
    return cv.used();
}

static bool matmul_dims_ok(size_t D0, size_t D1, size_t D2) {
    const size_t lim = (size_t)1 << 31;
    return D0 && D1 && D2 && D0 <= lim && D1 <= lim && D2 <= lim && D0 * D1 / D1 == D0 && D1 * D2 / D2 == D1;
}

// X, W as field vectors, or (X16, W16 non-null) as row-major 16-bit integers.
static int matmul_prove_any(const uint8_t seed[32], fr_vec X, const int16_t* X16, size_t D0, size_t D1, fr_vec W,
                            const int16_t* W16, size_t D2, uint8_t* proof, size_t cap, size_t* len, void* ws,
                            size_t ws_bytes, void* stream_v) {
    const bool small = X16 != nullptr;
    if (!seed || !matmul_dims_ok(D0, D1, D2)) return ZK_E_BADARG;
    if (small ? !W16 : (!vec_ok(X, D0 * D1) || !vec_ok(W, D1 * D2))) return ZK_E_BADARG;
    const int n0 = log2_ceil(D0), n1 = log2_ceil(D1), n2 = log2_ceil(D2);
    const size_t need = matmul_proof_bytes(D1);
    if (len) *len = need;
    if (!proof || cap < need) return ZK_E_BUFSZ;
    if (!ws || ws_bytes < matmul_workspace_bytes(D0, D1, D2)) return ZK_E_BUFSZ;
    hipStream_t stream = as_stream(stream_v);
    Mailbox* mb;
    ZK_TRY(mailbox_get(&mb));
    Carver cv(ws, ws_bytes);
    MatmulWs w;
    carve_matmul(w, cv, D0, D1, D2);
    uint64_t dims[3] = {D0, D1, D2};
    host::Transcript tr("zkmi/matmul/v1", seed, dims, 3);
    host::F u[32], v[32];
    for (int t = 0; t < n0; ++t) u[t] = tr.challenge("u");
    for (int t = 0; t < n2; ++t) v[t] = tr.challenge("v");
    const EqTable tables[2] = {{w.eu, w.P0, u, n0}, {w.ev, w.P2, v, n2}};
    ZK_TRY(eq_tables_run(tables, 2, stream));
    if (small) {
        // entries per accumulator: rows of X per chunk, columns of W per lane
        if (D0 > kColChunks * kSmallTermsMax || D2 > kSmallTermsMax) return ZK_E_BADARG;
        small_products_run(w.a, w.b, w.P1, X16, D0, D1, w.eu, w.P0, W16, D2, w.ev, w.P2, w.part, stream);
    } else {
        colsum_run(w.a, w.P1, X.limbs, X.stride, D0, D1, w.eu, w.P0, w.part, stream);
        rowdot_run(w.b, w.P1, W.limbs, W.stride, D1, D2, w.ev, w.P2, stream);
    }
    ZK_HIP_TRY(hipGetLastError());
    memcpy(proof, "ZKMM\x01\0\0\0", 8);
    host::put_le64(proof + 8, D0);
    host::put_le64(proof + 16, D1);
    host::put_le64(proof + 24, D2);
    return product_rounds_run(tr, w.a, w.P1, w.b, w.P1, n1, nullptr, proof + 32, proof + 64, cv, mb, stream);
}

int zkmi_selftest_resident_wait(void* ws, size_t ws_bytes, void* stream_v) {
    // The kernel waits for the host's answer to its sums.  Here the host never gives one: with a bound of a few polls
    // the kernel must give up by itself, having published the sums and nothing after them.
    if (!ws || ws_bytes < 4 * 32 * 4 + 512) return ZK_E_BUFSZ;
    hipStream_t stream = as_stream(stream_v);
    Mailbox* mb;
    ZK_TRY(mailbox_get(&mb));
    Carver cv(ws, ws_bytes);
    uint32_t* a = cv.limbs(4);
    uint32_t* b = cv.limbs(4);
    launch_fill_u32(a, 32, 1u, stream);
    launch_fill_u32(b, 32, 1u, stream);
    ProductTailArgs g{};
    g.a = a; g.as = 4; g.b = b; g.bs = 4;
    g.half = 2;
    ZK_TRY(product_tail_launch(g, mb, 8, stream));
    ZK_TRY(mailbox_wait(mb, g.out_seq[0], stream));          // the sums arrive
    ZK_HIP_TRY(hipStreamSynchronize(stream));                 // and the kernel ends without an answer
    const uint32_t flag = mb->words[kMailboxFlag];
    if (flag != g.out_seq[0]) return ZK_E_HIP;                // nothing was published after them
    // A call that ends early leaves an abort in the channel.  The next kernel must
    // not see it: this one is answered and has to run to its end.
    mailbox_send_abort(mb);
    TailGuard guard{mb, stream};
    ZK_TRY(product_tail_launch(g, mb, device_spin_limit(), stream));
    guard.armed = true;
    ZK_TRY(mailbox_wait(mb, g.out_seq[0], stream));
    mailbox_send_challenge(mb, g.cmd_seq, to_dev(host::one()).l);
    ZK_TRY(mailbox_wait(mb, g.out_seq[1], stream));
    guard.armed = false;
    ZK_HIP_TRY(hipStreamSynchronize(stream));
    return ZK_OK;
}

int matmul_sumcheck_prove(const uint8_t seed[32], fr_vec X, size_t D0, size_t D1, fr_vec W, size_t D2, uint8_t* proof,
                          size_t cap, size_t* len, void* ws, size_t ws_bytes, void* stream) {
    return matmul_prove_any(seed, X, nullptr, D0, D1, W, nullptr, D2, proof, cap, len, ws, ws_bytes, stream);
}

int matmul_sumcheck_prove_i16(const uint8_t seed[32], const int16_t* X, size_t D0, size_t D1, const int16_t* W, size_t D2,
                              uint8_t* proof, size_t cap, size_t* len, void* ws, size_t ws_bytes, void* stream) {
    if (!X || !W) return ZK_E_BADARG;
    fr_vec none = {nullptr, 0, 0};
    return matmul_prove_any(seed, none, X, D0, D1, none, W, D2, proof, cap, len, ws, ws_bytes, stream);
}

size_t matmul_verify_workspace_bytes(size_t D0, size_t D1, size_t D2) { return matmul_workspace_bytes(D0, D1, D2); }

int matmul_sumcheck_verify(const uint8_t seed[32], const uint8_t* proof, size_t len, size_t D0, size_t D1, size_t D2,
                           fr_vec Y, fr_vec X, fr_vec W, void* ws, size_t ws_bytes, void* stream_v) {
    using namespace host;
    if (!seed || !proof || !matmul_dims_ok(D0, D1, D2)) return ZK_E_BADARG;
    const int n0 = log2_ceil(D0), n1 = log2_ceil(D1), n2 = log2_ceil(D2);
    if (len != matmul_proof_bytes(D1) || memcmp(proof, "ZKMM\x01\0\0\0", 8) != 0) return ZK_E_REJECT;
    if (get_le64(proof + 8) != D0 || get_le64(proof + 16) != D1 || get_le64(proof + 24) != D2) return ZK_E_REJECT;
    F claim;
    if (!from_bytes(&claim, proof + 32)) return ZK_E_REJECT;
    uint64_t dims[3] = {D0, D1, D2};
    Transcript tr("zkmi/matmul/v1", seed, dims, 3);
    F u[32], v[32], r[32], fin[2];
    for (int t = 0; t < n0; ++t) u[t] = tr.challenge("u");
    for (int t = 0; t < n2; ++t) v[t] = tr.challenge("v");
    tr.absorb("claim", proof + 32, 32);
    if (!product_rounds_check(tr, proof + 64, n1, claim, r, fin)) return ZK_E_REJECT;
    const bool want_Y = Y.limbs != nullptr, want_X = X.limbs != nullptr, want_W = W.limbs != nullptr;
    if (!want_Y && !want_X && !want_W) return ZK_OK;
    if ((want_Y && !vec_ok(Y, D0 * D2)) || (want_X && !vec_ok(X, D0 * D1)) || (want_W && !vec_ok(W, D1 * D2)))
        return ZK_E_BADARG;
    if (!ws || ws_bytes < matmul_workspace_bytes(D0, D1, D2)) return ZK_E_BUFSZ;
    hipStream_t stream = as_stream(stream_v);
    Mailbox* mb;
    ZK_TRY(mailbox_get(&mb));
    Carver cv(ws, ws_bytes);
    MatmulWs w;
    carve_matmul(w, cv, D0, D1, D2);
    const EqTable tables[2] = {{w.eu, w.P0, u, n0}, {w.ev, w.P2, v, n2}};
    ZK_TRY(eq_tables_run(tables, 2, stream));
    // Y~(u,v) = sum_j (sum_i e~(u,i) Y[i][j]) e~(v,j)
    if (want_Y) {
        uint32_t* ycols = cv.limbs(w.P2);
        if (!ycols) return ZK_E_BUFSZ;
        colsum_run(ycols, w.P2, Y.limbs, Y.stride, D0, D2, w.eu, w.P0, w.part, stream);
        ZK_TRY(dot_run(ycols, w.P2, w.ev, w.P2, D2, w.dot, mb->words, stream));
        ZK_HIP_TRY(hipStreamSynchronize(stream));
        if (!equal(from_dev(mb->words), claim)) return ZK_E_REJECT;
    }
    if (want_X || want_W) {
        uint32_t* er = cv.limbs(w.P1);
        if (!er) return ZK_E_BUFSZ;
        ZK_TRY(eq_table_run(er, w.P1, r, n1, stream));
        if (want_X) {
            colsum_run(w.a, w.P1, X.limbs, X.stride, D0, D1, w.eu, w.P0, w.part, stream);
            ZK_TRY(dot_run(w.a, w.P1, er, w.P1, D1, w.dot, mb->words, stream));
            ZK_HIP_TRY(hipStreamSynchronize(stream));
            if (!equal(from_dev(mb->words), fin[0])) return ZK_E_REJECT;
        }
        if (want_W) {
            rowdot_run(w.b, w.P1, W.limbs, W.stride, D1, D2, w.ev, w.P2, stream);
            ZK_TRY(dot_run(w.b, w.P1, er, w.P1, D1, w.dot, mb->words, stream));
            ZK_HIP_TRY(hipStreamSynchronize(stream));
            if (!equal(from_dev(mb->words), fin[1])) return ZK_E_REJECT;
        }
    }
    return ZK_OK;
}

}  // extern "C"

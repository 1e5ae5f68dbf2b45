// Sums, eq tables, folding and multilinear evaluation (Section 3.3 of the paper:
// tensors as functions on the Boolean cube and their multilinear extensions).
#include <mutex>

#include "internal.h"
#include "mfma_dev.h"
#include "mle_dev.h"
#include "reduce_dev.h"

namespace zkmi {

// ---- sums -------------------------------------------------------------------

__global__ void k_fill_words(uint32_t* p, size_t n, uint32_t v) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

void launch_fill_u32(uint32_t* p, size_t n, uint32_t v, hipStream_t stream) {
    if (n == 0) return;
    hipLaunchKernelGGL(k_fill_words, dim3(grid_for(n)), dim3(kBlock), 0, stream, p, n, v);
}

__global__ void __launch_bounds__(kBlock) k_sum_partial(const uint32_t* __restrict__ a, size_t stride, size_t n,
                                                        uint32_t* __restrict__ partials, size_t pstride) {
    __shared__ uint32_t lds[4 * 8];
    Fr acc[1] = {fr_zero()};
    for (size_t i = blockIdx.x * (size_t)kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock)
        acc[0] = fr_add(acc[0], fr_load(a, stride, i));
    block_sum<1, 4>(acc, lds);
    if (threadIdx.x == 0) fr_store(partials, pstride, blockIdx.x, acc[0]);
}

// Adds up the per-workgroup partial values of a round, one workgroup per value
// (the first nv1 values come from the first array, the rest from the second;
// value v of workgroup b sits at element b*nv + v of its array).  Totals go out as
// raw Montgomery limbs, value q at out_words[8q..8q+7].  The workgroup that
// finishes last (a ticket counter in device memory, left at zero again) publishes
// completion.
static const int kFinalThreads = 1024;

__global__ void __launch_bounds__(kFinalThreads) k_final_sum2(const uint32_t* __restrict__ part1, size_t pstride1, int nv1,
                                                              const uint32_t* __restrict__ part2, size_t pstride2, int nv2,
                                                              unsigned nblocks, uint32_t* out_words, uint32_t* words,
                                                              uint32_t seq, uint32_t* ticket, const uint32_t* note,
                                                              uint32_t* note_out) {
    __shared__ uint32_t lds[16 * 8];
    const int q = blockIdx.x;
    const bool first = q < nv1;
    const uint32_t* part = first ? part1 : part2;
    const size_t pstride = first ? pstride1 : pstride2;
    const int nv = first ? nv1 : nv2, qq = first ? q : q - nv1;
    Fr acc[1] = {fr_zero()};
    for (unsigned b = threadIdx.x; b < nblocks; b += kFinalThreads)
        acc[0] = fr_add(acc[0], fr_load(part, pstride, (size_t)b * nv + qq));
    block_sum<1, 16>(acc, lds);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < 8; ++k) out_words[8 * q + k] = acc[0].l[k];
        if (note && q == 0) {
            note_out[0] = note[0];
            note_out[1] = note[1];
        }
        mailbox_written();
        if (seq != 0) {
            unsigned done = atomicAdd(ticket, 1u);
            if (done == gridDim.x - 1) {
                *ticket = 0;
                mailbox_publish(words, seq);
            }
        }
    }
}

void launch_final_sum2(const uint32_t* part1, size_t pstride1, int nv1, const uint32_t* part2, size_t pstride2, int nv2,
                       unsigned nblocks, uint32_t* out_words, uint32_t* words, uint32_t seq, uint32_t* ticket,
                       hipStream_t stream, const uint32_t* note, uint32_t* note_out) {
    hipLaunchKernelGGL(k_final_sum2, dim3(nv1 + nv2), dim3(kFinalThreads), 0, stream, part1, pstride1, nv1, part2, pstride2,
                       nv2, nblocks, out_words, words, seq, ticket, note, note_out);
}

void launch_final_sum(const uint32_t* partials, size_t pstride, unsigned nblocks, int nv, uint32_t* out_words,
                      uint32_t* words, uint32_t seq, uint32_t* ticket, hipStream_t stream) {
    launch_final_sum2(partials, pstride, nv, nullptr, 0, 0, nblocks, out_words, words, seq, ticket, stream);
}

size_t sum_scratch_bytes(size_t) {
    Carver cv(nullptr, 0);
    cv.limbs(kMaxPartialBlocks);
    cv.take(256);  // ticket
    return cv.used();
}

int sum_run(const uint32_t* a, size_t stride, size_t n, Carver& cv, Mailbox* mb, uint32_t seq, hipStream_t stream) {
    uint32_t* partials = cv.limbs(kMaxPartialBlocks);
    uint32_t* ticket = (uint32_t*)cv.take(256);
    if (!partials || !ticket) return ZK_E_BUFSZ;
    launch_fill_u32(ticket, 1, 0u, stream);
    unsigned blocks = grid_for(n, kBlock * 8, kMaxPartialBlocks);
    hipLaunchKernelGGL(k_sum_partial, dim3(blocks), dim3(kBlock), 0, stream, a, stride, n, partials,
                       (size_t)kMaxPartialBlocks);
    launch_final_sum(partials, kMaxPartialBlocks, blocks, 1, mb->words, mb->words, seq, ticket, stream);
    ZK_HIP_TRY(hipGetLastError());
    return ZK_OK;
}

// ---- the sum for callers that cannot allocate ---------------------------------------
//
// fr_sum_noalloc keeps its per-workgroup partial sums in an array that is part of
// the library's image on every GPU instead of in a workspace.  The array's name
// is only a handle on the host: the address kernels can use is asked for once per
// device (hipGetSymbolAddress with that device current) and kept.

static const unsigned kStaticSumBlocks = 1024;
static __device__ __align__(256) uint32_t scratch[kStaticSumBlocks * 8];  // 32 KiB on every GPU the library runs on

static const int kStaticMaxDevices = 64;
static std::mutex g_scratch_mutex;
static uint32_t* g_scratch_ptr[kStaticMaxDevices];  // device address of `scratch`, per device

static int scratch_of_current_device(uint32_t** out) {
    int dev = -1;
    ZK_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kStaticMaxDevices) return ZK_E_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return ZK_E_HIP;
        g_scratch_ptr[dev] = (uint32_t*)p;
    }
    *out = g_scratch_ptr[dev];
    return ZK_OK;
}

// Adds up nblocks partial sums (limb-major, stride pstride) and writes the total
// as the canonical integer, eight little-endian words, to out (device memory).
__global__ void __launch_bounds__(kFinalThreads) k_sum_finish_canonical(const uint32_t* __restrict__ partials,
                                                                        size_t pstride, unsigned nblocks,
                                                                        uint32_t* __restrict__ out) {
    __shared__ uint32_t lds[16 * 8];
    Fr acc[1] = {fr_zero()};
    for (unsigned b = threadIdx.x; b < nblocks; b += kFinalThreads) acc[0] = fr_add(acc[0], fr_load(partials, pstride, b));
    block_sum<1, 16>(acc, lds);
    if (threadIdx.x == 0) {
        const Fr c = fr_from_mont(acc[0]);
#pragma unroll
        for (int k = 0; k < 8; ++k) out[k] = c.l[k];
    }
}

// ---- eq tables ----------------------------------------------------------------

// Up to two tables in one launch.  The factors of an entry's first and last four
// variables come from small tables the host has made, those in between are multiplied
// up.
//
// A short table takes a thread per entry: its chain of products is what counts (two
// tables of 2^11 and 2^13 entries: 43 us as launches of their own with a thread for
// sixteen entries, 9 us so).  With many entries per lane it is the products themselves,
// one per variable and entry: from kEqSharedVars variables on a thread makes the product
// of all but the first four variables once for the sixteen entries that differ in those.
// Measured, whole calls by entry and shared: 2^17 entries 17.3 and 23.9 us, 2^18 30.1 and
// 25.2, 2^22 496 and 75, 2^25 4640 and 546 (bound by issue: some 2.4 products per entry).
static const int kEqEdge = 4;
static const int kEqSharedVars = 18;
struct EqJob {
    uint32_t* dst;
    size_t stride;
    Fr u[32 - 2 * kEqEdge];  // the variables in between
    Fr top[1 << kEqEdge], low[1 << kEqEdge];
    int nvars, ntop, nlow;
    int shared;  // a thread per entry of all but the first kEqEdge variables
    uint32_t blocks;
};
struct EqArgs {
    EqJob job[2];
};

__global__ void __launch_bounds__(kBlock) k_eq_table(EqArgs args) {
    const int second = blockIdx.x >= args.job[0].blocks;
    const EqJob& g = args.job[second];
    const size_t first = (blockIdx.x - (second ? args.job[0].blocks : 0u)) * (size_t)kBlock + threadIdx.x;
    const int rest = g.nvars - g.ntop;  // the variables behind the first few
    const size_t count = (size_t)1 << (g.shared ? rest : g.nvars);
    const Fr one = fr_one();
    for (size_t x = first; x < count; x += (size_t)g.blocks * kBlock) {
        Fr acc = g.shared ? g.low[x & ((1u << g.nlow) - 1)] : g.top[x >> rest];
        if (!g.shared && g.nlow) acc = fr_mul(acc, g.low[x & ((1u << g.nlow) - 1)]);
        for (int t = g.ntop; t < g.nvars - g.nlow; ++t) {
            const unsigned bit = (unsigned)(x >> (g.nvars - 1 - t)) & 1u;
            acc = fr_mul(acc, bit ? g.u[t - g.ntop] : fr_sub(one, g.u[t - g.ntop]));
        }
        if (!g.shared) {
            fr_store(g.dst, g.stride, x, acc);
            continue;
        }
        for (int hi = 0; hi < 1 << kEqEdge; ++hi) fr_store(g.dst, g.stride, ((size_t)hi << rest) + x, fr_mul(acc, g.top[hi]));
    }
}

static void eq_edge(Fr* out, const host::F* u, int vars) {
    host::F e[1 << kEqEdge];
    e[0] = host::one();
    for (int t = 0; t < vars; ++t) {
        // append variable t below the ones already in the table
        for (int x = (1 << t) - 1; x >= 0; --x) {
            const host::F hi = host::mul(e[x], u[t]);
            e[2 * x + 1] = hi;
            e[2 * x] = host::sub(e[x], hi);
        }
    }
    for (int x = 0; x < (1 << vars); ++x) out[x] = to_dev(e[x]);
}

int eq_tables_run(const EqTable* tables, int count, hipStream_t stream) {
    if (count < 1 || count > 2) return ZK_E_BADARG;
    EqArgs args;
    memset(&args, 0, sizeof args);
    uint32_t blocks = 0;
    for (int q = 0; q < count; ++q) {
        const EqTable& t = tables[q];
        if (t.nvars < 0 || t.nvars > 31) return ZK_E_BADARG;
        EqJob& j = args.job[q];
        j.dst = t.dst;
        j.stride = t.stride;
        j.nvars = t.nvars;
        j.ntop = t.nvars < kEqEdge ? t.nvars : kEqEdge;
        j.nlow = t.nvars - j.ntop < kEqEdge ? t.nvars - j.ntop : kEqEdge;
        eq_edge(j.top, t.u, j.ntop);
        eq_edge(j.low, t.u + (t.nvars - j.nlow), j.nlow);
        for (int v = j.ntop; v < t.nvars - j.nlow; ++v) j.u[v - j.ntop] = to_dev(t.u[v]);
        j.shared = t.nvars >= kEqSharedVars;
        j.blocks = grid_for((size_t)1 << (t.nvars - (j.shared ? kEqEdge : 0)));
        blocks += j.blocks;
    }
    hipLaunchKernelGGL(k_eq_table, dim3(blocks), dim3(kBlock), 0, stream, args);
    ZK_HIP_TRY(hipGetLastError());
    return ZK_OK;
}

int eq_table_run(uint32_t* dst, size_t stride, const host::F* u, int nvars, hipStream_t stream) {
    const EqTable t{dst, stride, u, nvars};
    return eq_tables_run(&t, 1, stream);
}

// ---- evaluation ----------------------------------------------------------------------

__global__ void k_emit(const uint32_t* __restrict__ a, size_t stride, size_t index, uint32_t* out, uint32_t* words, uint32_t seq) {
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < 8; ++k) out[k] = a[k * stride + index];
        mailbox_written();
        mailbox_publish(words, seq);
    }
}

// Multilinear evaluation: the variables are bound up to six at a time (64 constants
// per output, on the matrix cores), so that 2^22 elements take four passes, of
// which only the first is long and bound by the reading of its input.  One variable
// per pass, as before, took 22 dependent launches of some 12 us.  Measured: a lookup
// proof of 2^22 entries verified against its tensors (five evaluations, two digests)
// 1.27 -> 0.58 ms, with the evaluations in the same launches and one wait for all.
static const int kMleStageVars = 6;

static int mle_stage_count(int nvars) { return (nvars + kMleStageVars - 1) / kMleStageVars; }
// Variables stage t of s binds: nvars split as evenly as it goes, the longer stages first.
static int mle_stage_vars(int nvars, int s, int t) { return nvars / s + (t < nvars % s ? 1 : 0); }

// The matrices of all stages' constants of up to two points, in one launch: thread
// (entry, k) makes column k of one entry's matrix.
struct MleTableArgs {
    Fr u[2][32];
    int nvars[2];
    uint32_t first[2];    // entries of point q start here in the table
    uint32_t total;       // entries in all
    uint8_t* table;
};

__global__ void __launch_bounds__(kBlock) k_mle_table(MleTableArgs args) {
    const uint32_t g = blockIdx.x * kBlock + threadIdx.x;
    const uint32_t entry = g >> 5;
    if (entry >= args.total) return;
    const int pt = entry >= args.first[1] ? 1 : 0;
    uint32_t x = entry - args.first[pt];
    const int nv = args.nvars[pt], stages = (nv + kMleStageVars - 1) / kMleStageVars;
    int v0 = 0, vars = 0;
    for (int t = 0; t < stages; ++t) {
        vars = nv / stages + (t < nv % stages ? 1 : 0);
        if (x < (1u << vars)) break;
        x -= 1u << vars;
        v0 += vars;
    }
    const Fr one = fr_one();
    Fr e = one;
    for (int t = 0; t < vars; ++t) {
        const Fr u = args.u[pt][v0 + t];
        const Fr f = (x >> (vars - 1 - t)) & 1u ? u : fr_sub(one, u);
        e = t == 0 ? f : fr_mul(e, f);
    }
    uint32_t digits[8];
    toeplitz_column(digits, e, (int)(g & 31));
    toeplitz_store(args.table + (size_t)entry * kToepBytes, digits, (int)(g & 31));
}

__global__ void __launch_bounds__(kBlock) k_mle_stage(MleStageArgs args) {
    __shared__ MleParts part;
    mle_stage_block(args, blockIdx.x, part);
    if (args.seq) {
        __syncthreads();
        if (threadIdx.x != 0) return;
        if (gridDim.x == 1) {  // one evaluation: nobody to wait for
            mailbox_publish(args.words, args.seq);
        } else if (atomicAdd(args.ticket, 1u) == gridDim.x - 1) {
            *args.ticket = 0;
            mailbox_publish(args.words, args.seq);
        }
    }
}

// Scratch of one evaluation: its stages' outputs.
static size_t mle_outputs(int nvars) {
    const int s = mle_stage_count(nvars);
    size_t total = 0;
    for (int t = 0, left = nvars; t + 1 < s; ++t) {
        left -= mle_stage_vars(nvars, s, t);
        total += (size_t)1 << left;
    }
    return total;
}
static uint32_t mle_table_entries(int nvars) {
    const int s = mle_stage_count(nvars);
    uint32_t total = 0;
    for (int t = 0; t < s; ++t) total += 1u << mle_stage_vars(nvars, s, t);
    return total;
}

// Room for jobs of at most these lengths at (at most) two points, whose lengths are
// at most those of jobs 0 and njobs - 1.  Monotonic in the lengths: a stage is counted
// with all its 64 constants.
size_t mle_scratch_bytes_many(const int* nvars, int njobs) {
    Carver cv(nullptr, 0);
    for (int q = 0; q < njobs; ++q) cv.limbs(mle_outputs(nvars[q]));
    const int stages = mle_stage_count(nvars[0]) + (njobs > 1 ? mle_stage_count(nvars[njobs - 1]) : 0);
    cv.take((size_t)stages * (kToepBytes << kMleStageVars));
    cv.take(256);
    return cv.used();
}
size_t mle_scratch_bytes(int nvars) { return mle_scratch_bytes_many(&nvars, 1); }

// C0 mod r plus 4096 C r (the weights e~(point, c) add up to one).
static ToepBias mle_bias(uint32_t C) {
    ToepBias b;
    // C0 = 0x8080..80 is r + kC0: below 2 r
    static const uint32_t c0_mod_r[8] = {0x8080807fu, 0x80808081u, 0x80822481u, 0x2cc2dc7du, 0x76dea87bu, 0x4d46a878u, 0x56e30338u, 0x0c92d92du};
    static const uint32_t r32[8] = {ZK_R0, ZK_R1, ZK_R2, ZK_R3, ZK_R4, ZK_R5, ZK_R6, ZK_R7};
    uint64_t acc = 0;
    for (int k = 0; k < 8; ++k) {
        acc += (uint64_t)r32[k] * (4096u * C) + c0_mod_r[k];
        b.w[k] = (uint32_t)acc;
        acc >>= 32;
    }
    b.w[8] = (uint32_t)acc;
    return b;
}

int mle_eval_begin(MlePlan& plan, const MleJob* jobs, int njobs, Carver& cv, Mailbox* mb, uint32_t seq, hipStream_t stream) {
    if (njobs < 1 || njobs > kMleMaxJobs) return ZK_E_BADARG;
    // the points: at most two different ones (a lookup's tensor and its table)
    MleTableArgs targs;
    memset(&targs, 0, sizeof targs);
    const host::F* points[2] = {nullptr, nullptr};
    int npoints = 0, point_of[kMleMaxJobs], most_stages = 0;
    for (int q = 0; q < njobs; ++q) {
        int at = -1;
        for (int p = 0; p < npoints; ++p)
            if (points[p] == jobs[q].point && targs.nvars[p] == jobs[q].nvars) at = p;
        if (at < 0) {
            if (npoints == 2) return ZK_E_BADARG;
            at = npoints++;
            points[at] = jobs[q].point;
            targs.nvars[at] = jobs[q].nvars;
            for (int t = 0; t < jobs[q].nvars; ++t) targs.u[at][t] = to_dev(jobs[q].point[t]);
        }
        point_of[q] = at;
        const int s = mle_stage_count(jobs[q].nvars);
        if (s > most_stages) most_stages = s;
    }
    if (most_stages > kMleMaxSteps) return ZK_E_BADARG;
    memset(&plan, 0, sizeof plan);
    plan.steps = most_stages;
    plan.njobs = njobs;
    plan.seq = seq;
    for (int q = 0; q < njobs; ++q) plan.jobs[q] = jobs[q];
    if (most_stages == 0) return ZK_OK;  // single elements are their own values: no scratch is asked for
    targs.first[0] = 0;
    targs.first[1] = mle_table_entries(targs.nvars[0]);
    targs.total = targs.first[1] + (npoints == 2 ? mle_table_entries(targs.nvars[1]) : 0);
    if (npoints < 2) targs.first[1] = 0xffffffffu;
    uint32_t* outs[kMleMaxJobs];
    for (int q = 0; q < njobs; ++q) {
        outs[q] = cv.limbs(mle_outputs(jobs[q].nvars));
        if (!outs[q]) return ZK_E_BUFSZ;
    }
    targs.table = (uint8_t*)cv.take((size_t)targs.total * kToepBytes);
    uint32_t* ticket = (uint32_t*)cv.take(256);
    if (!targs.table || !ticket) return ZK_E_BUFSZ;
    if (njobs > 1) launch_fill_u32(ticket, 1, 0u, stream);
    hipLaunchKernelGGL(k_mle_table, dim3(grid_for((size_t)targs.total * 32)), dim3(kBlock), 0, stream, targs);
    // every job's last stage in the last launch, so that one flag stands for all
    ToepSource cur[kMleMaxJobs];
    int left[kMleMaxJobs];
    const uint4* table[kMleMaxJobs];
    for (int q = 0; q < njobs; ++q) {
        cur[q].p = jobs[q].a;
        cur[q].stride = jobs[q].stride;
        left[q] = jobs[q].nvars;
        table[q] = (const uint4*)(targs.table + (size_t)(point_of[q] ? targs.first[1] : 0) * kToepBytes);
    }
    for (int step = 0; step < most_stages; ++step) {
        MleStageArgs& args = plan.step[step];
        uint32_t& blocks = plan.blocks[step];
        for (int q = 0; q < njobs; ++q) {
            const int s = mle_stage_count(jobs[q].nvars), t = step - (most_stages - s);
            if (s == 0 || t < 0) continue;
            const int vars = mle_stage_vars(jobs[q].nvars, s, t);
            left[q] -= vars;
            MleStageJob& j = args.job[args.njobs++];
            j.C = 1u << vars;
            j.P = (size_t)1 << left[q];
            j.src = cur[q];
            j.src.vec = j.P % 4 == 0 && j.src.stride % 4 == 0 && ((uintptr_t)j.src.p & 15) == 0;
            j.table = table[q];
            j.bias = mle_bias(j.C);
            j.first_block = blocks;
            if (t == s - 1) {
                j.dst = jobs[q].out_words;
                j.dst_stride = 1;
            } else {
                j.dst = outs[q];
                j.dst_stride = j.P;
                outs[q] += 8 * j.P;
            }
            cur[q].p = j.dst;
            cur[q].stride = j.dst_stride;
            table[q] += (size_t)j.C * (kToepBytes / 16);
            blocks += (uint32_t)div_up(j.P, 128);
        }
        if (step == most_stages - 1) {
            args.words = mb->words;
            args.ticket = ticket;
            args.seq = seq;
        }
    }
    ZK_HIP_TRY(hipGetLastError());
    return ZK_OK;
}

int mle_eval_rest(const MlePlan& plan, int first, Mailbox* mb, hipStream_t stream) {
    for (int step = first; step + 1 < plan.steps; ++step)
        hipLaunchKernelGGL(k_mle_stage, dim3(plan.blocks[step]), dim3(kBlock), 0, stream, plan.step[step]);
    for (int q = 0; q < plan.njobs; ++q) {  // a single element: its value
        const MleJob& j = plan.jobs[q];
        if (j.nvars == 0)
            hipLaunchKernelGGL(k_emit, dim3(1), dim3(64), 0, stream, j.a, j.stride, (size_t)0, j.out_words, mb->words,
                               plan.steps == 0 && q + 1 == plan.njobs ? plan.seq : 0u);
    }
    if (plan.steps) {
        const int last = plan.steps - 1;
        hipLaunchKernelGGL(k_mle_stage, dim3(plan.blocks[last]), dim3(kBlock), 0, stream, plan.step[last]);
    }
    ZK_HIP_TRY(hipGetLastError());
    return ZK_OK;
}

int mle_eval_launch(const MleJob* jobs, int njobs, Carver& cv, Mailbox* mb, uint32_t seq, hipStream_t stream) {
    MlePlan plan;
    ZK_TRY(mle_eval_begin(plan, jobs, njobs, cv, mb, seq, stream));
    return mle_eval_rest(plan, 0, mb, stream);
}

int mle_eval_run(const uint32_t* a, size_t stride, int nvars, const host::F* point, Carver& cv, Mailbox* mb,
                 uint32_t seq, hipStream_t stream) {
    const MleJob job{a, stride, nvars, point, mb->words};
    return mle_eval_launch(&job, 1, cv, mb, seq, stream);
}

}  // namespace zkmi

using namespace zkmi;

extern "C" {

size_t fr_sum_workspace_bytes(size_t n) { return sum_scratch_bytes(n); }

int fr_sum(fr_t* out, fr_vec a, void* ws, size_t ws_bytes, void* stream) {
    if (!out || (a.n && !vec_ok(a, a.n))) return ZK_E_BADARG;
    if (a.n == 0) {
        memset(out, 0, sizeof *out);
        return ZK_OK;
    }
    if (!ws || ws_bytes < sum_scratch_bytes(a.n)) return ZK_E_BUFSZ;
    Mailbox* mb;
    ZK_TRY(mailbox_get(&mb));
    Carver cv(ws, ws_bytes);
    uint32_t seq = mb->next_seq();
    ZK_TRY(sum_run(a.limbs, a.stride, a.n, cv, mb, seq, as_stream(stream)));
    ZK_TRY(mailbox_wait(mb, seq, as_stream(stream)));
    ZK_HIP_TRY(hipStreamSynchronize(as_stream(stream)));
    *out = host::to_canonical(from_dev(mb->words));
    return ZK_OK;
}

int fr_sum_noalloc(uint32_t* out, fr_vec a, void* stream) {
    if (!out || a.n > FR_SUM_NOALLOC_MAX || (a.n && !vec_ok(a, a.n))) return ZK_E_BADARG;
    uint32_t* partials = nullptr;
    ZK_TRY(scratch_of_current_device(&partials));
    // every workgroup writes its partial sum before the closing kernel reads exactly
    // that many: nothing in the array has to start at zero
    unsigned blocks = 0;
    if (a.n) {
        blocks = grid_for(a.n, kBlock * 8, kStaticSumBlocks);
        hipLaunchKernelGGL(k_sum_partial, dim3(blocks), dim3(kBlock), 0, as_stream(stream), a.limbs, a.stride, a.n, partials,
                           (size_t)kStaticSumBlocks);
    }
    hipLaunchKernelGGL(k_sum_finish_canonical, dim3(1), dim3(kFinalThreads), 0, as_stream(stream), partials,
                       (size_t)kStaticSumBlocks, blocks, out);
    ZK_HIP_TRY(hipGetLastError());
    return ZK_OK;
}

int fr_eq_table(fr_vec dst, const fr_t* u, int nvars, void* stream) {
    if (nvars < 0 || nvars > 31 || (nvars && !u) || !vec_ok(dst, (size_t)1 << nvars)) return ZK_E_BADARG;
    host::F um[32];
    for (int t = 0; t < nvars; ++t) {
        if (!host::canonical_in_range(u[t])) return ZK_E_BADARG;
        um[t] = host::from_canonical(u[t]);
    }
    return eq_table_run(dst.limbs, dst.stride, um, nvars, as_stream(stream));
}

size_t fr_mle_eval_workspace_bytes(int nvars) { return mle_scratch_bytes(nvars); }

int fr_mle_eval(fr_t* out, fr_vec a, const fr_t* point, int nvars, void* ws, size_t ws_bytes, void* stream) {
    if (!out || nvars < 0 || nvars > 31 || (nvars && !point) || !vec_ok(a, (size_t)1 << nvars)) return ZK_E_BADARG;
    if (nvars && (!ws || ws_bytes < mle_scratch_bytes(nvars))) return ZK_E_BUFSZ;
    host::F pm[32];
    for (int t = 0; t < nvars; ++t) {
        if (!host::canonical_in_range(point[t])) return ZK_E_BADARG;
        pm[t] = host::from_canonical(point[t]);
    }
    Mailbox* mb;
    ZK_TRY(mailbox_get(&mb));
    Carver cv(ws, ws_bytes);
    uint32_t seq = mb->next_seq();
    ZK_TRY(mle_eval_run(a.limbs, a.stride, nvars, pm, cv, mb, seq, as_stream(stream)));
    ZK_TRY(mailbox_wait(mb, seq, as_stream(stream)));
    ZK_HIP_TRY(hipStreamSynchronize(as_stream(stream)));
    *out = host::to_canonical(from_dev(mb->words));
    return ZK_OK;
}

}  // extern "C"

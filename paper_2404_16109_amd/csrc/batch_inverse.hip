// Batched inversion by the product trick, arranged for a GPU:
//
//   down pass  : every thread multiplies up its K elements (stride 256 within a
//                block, so loads stay coalesced), storing the running products,
//                and emits its total into the next, K times smaller, level;
//   top        : one workgroup scans the last level (<= 256 values); the host
//                inverts the single grand total (the only field inversion);
//   up pass    : each thread receives the inverse of its own total and walks
//                back over its elements: out_j = inv * prefix_{j-1}, inv *= x_j.
//
// A level that is short enough (<= 2^20 elements, a first level of 2561 to 2^17) is
// reduced by whole workgroups instead: the threads' totals are multiplied up within the
// workgroup (a scan in LDS), so the next level is 256*K times smaller and fits
// the top.  That saves dependent launches, which is all the small levels cost:
// eight for 2^25 elements instead of twelve, four for a table of 2^16.  (Longer
// levels stay with the threads: there the scans cost more than the launches they
// save.)
//
// Cost: about 3 multiplications per element plus a geometric tail.  A zero
// anywhere makes the grand total zero, which is how it is detected.
#include "internal.h"

namespace zkmi {

static const int kBiK = 16;  // elements per thread per level

// A level can be the concatenation of two vectors (the tensor and the table of a
// lookup, inverted in one go): elements from n1 on belong to the second, which
// has its own source and its own prefix/result buffer.  n1 is a multiple of the
// elements one workgroup covers, so a workgroup lies in one of them.
struct BiSecond {
    const uint32_t* src;
    size_t ss;
    uint32_t* p;
    size_t ps;
    size_t n1;  // SIZE_MAX: no second vector
};

__device__ __forceinline__ Fr bi_load(const uint32_t* __restrict__ src, size_t ss, size_t i, bool shifted,
                                      const Fr& shift) {
    Fr x = fr_load(src, ss, i);
    return shifted ? fr_add(x, shift) : x;
}

// prefix_i = product of this thread's elements up to and including i; the
// thread's total goes to next[tid].
__global__ void __launch_bounds__(kBlock) k_bi_down(const uint32_t* __restrict__ src, size_t ss, size_t n, int shifted,
                                                    Fr shift, uint32_t* __restrict__ prefix, size_t ps,
                                                    uint32_t* __restrict__ next, size_t ns, BiSecond second) {
    size_t tid = blockIdx.x * (size_t)kBlock + threadIdx.x;
    size_t base = blockIdx.x * (size_t)kBlock * kBiK + threadIdx.x;
    if (blockIdx.x * (size_t)kBlock * kBiK >= second.n1) {  // the whole workgroup is in the second vector
        src = second.src;
        ss = second.ss;
        prefix = second.p;
        ps = second.ps;
        base -= second.n1;
        n -= second.n1;
    } else if (n > second.n1) {
        n = second.n1;
    }
    Fr acc = fr_one();
    bool first = true;
    for (int j = 0; j < kBiK; ++j) {
        size_t i = base + (size_t)j * kBlock;
        if (i < n) {
            Fr x = bi_load(src, ss, i, shifted, shift);
            acc = first ? x : fr_mul(acc, x);
            first = false;
            fr_store(prefix, ps, i, acc);
        }
    }
    fr_store(next, ns, tid, acc);
}

// inv_next[tid] = inverse of this thread's total.  out may be the prefix buffer.
__global__ void __launch_bounds__(kBlock) k_bi_up(const uint32_t* __restrict__ src, size_t ss, size_t n, int shifted,
                                                  Fr shift, const uint32_t* prefix, size_t ps,
                                                  const uint32_t* __restrict__ inv_next, size_t is, uint32_t* out,
                                                  size_t os, BiSecond second) {
    size_t tid = blockIdx.x * (size_t)kBlock + threadIdx.x;
    size_t base = blockIdx.x * (size_t)kBlock * kBiK + threadIdx.x;
    if (blockIdx.x * (size_t)kBlock * kBiK >= second.n1) {  // prefix and out are the same buffer (see batch_inverse_end)
        src = second.src;
        ss = second.ss;
        prefix = second.p;
        ps = second.ps;
        out = second.p;
        os = second.ps;
        base -= second.n1;
        n -= second.n1;
    } else if (n > second.n1) {
        n = second.n1;
    }
    Fr inv = fr_load(inv_next, is, tid);
    for (int j = kBiK - 1; j >= 0; --j) {
        size_t i = base + (size_t)j * kBlock;
        if (i < n) {
            if (j > 0) {
                Fr before = fr_load(prefix, ps, i - kBlock);
                Fr x = bi_load(src, ss, i, shifted, shift);
                fr_store(out, os, i, fr_mul(inv, before));
                inv = fr_mul(inv, x);
            } else {
                fr_store(out, os, i, inv);
            }
        }
    }
}

// Inclusive scan of products over one workgroup of THREADS threads (Hillis-Steele in LDS, 8*THREADS words).
template <int THREADS>
__device__ __forceinline__ Fr block_scan_mul(Fr v, uint32_t* lds, bool reverse) {
    const int t = threadIdx.x;
    for (int off = 1; off < THREADS; off <<= 1) {
#pragma unroll
        for (int k = 0; k < 8; ++k) lds[k * THREADS + t] = v.l[k];
        __syncthreads();
        int partner = reverse ? t + off : t - off;
        if (partner >= 0 && partner < THREADS) {
            Fr o;
#pragma unroll
            for (int k = 0; k < 8; ++k) o.l[k] = lds[k * THREADS + partner];
            v = fr_mul(v, o);
        }
        __syncthreads();
    }
    return v;
}

// Inclusive products from both ends over THREADS values, by a workgroup of twice as
// many threads: thread t < THREADS gets v_0 .. v_t, thread THREADS + t v_t .. v_last
// (v: value t % THREADS in both), and from these everybody's neighbours: what comes
// before, respectively after, value t.  One chain of eight dependent products where the
// two scans one after the other are sixteen (a workgroup of 256 values: 16 -> 13.7 us).
// lds: 16 * THREADS words.
template <int THREADS>
__device__ __forceinline__ Fr block_scan_both(Fr v, uint32_t* lds) {
    const int t = threadIdx.x & (THREADS - 1);
    const bool back = threadIdx.x >= THREADS;
    uint32_t* mine = lds + (back ? 8 * THREADS : 0);
    for (int off = 1; off < THREADS; off <<= 1) {
#pragma unroll
        for (int k = 0; k < 8; ++k) mine[k * THREADS + t] = v.l[k];
        __syncthreads();
        const int partner = back ? t + off : t - off;
        if (partner >= 0 && partner < THREADS) {
            Fr o;
#pragma unroll
            for (int k = 0; k < 8; ++k) o.l[k] = mine[k * THREADS + partner];
            v = fr_mul(v, o);
        }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) mine[k * THREADS + t] = v.l[k];
    __syncthreads();
    Fr o = fr_one();
    const int partner = back ? t + 1 : t - 1;
    if (partner >= 0 && partner < THREADS) {
#pragma unroll
        for (int k = 0; k < 8; ++k) o.l[k] = mine[k * THREADS + partner];
    }
    __syncthreads();
    return o;
}

// The scanned value of the thread before (reverse: after) this one, or one at the end of the line.
template <int THREADS>
__device__ __forceinline__ Fr block_neighbour(const Fr& scanned, uint32_t* lds, bool reverse) {
    const int t = threadIdx.x;
#pragma unroll
    for (int k = 0; k < 8; ++k) lds[k * THREADS + t] = scanned.l[k];
    __syncthreads();
    Fr o = fr_one();
    const int partner = reverse ? t + 1 : t - 1;
    if (partner >= 0 && partner < THREADS) {
#pragma unroll
        for (int k = 0; k < 8; ++k) o.l[k] = lds[k * THREADS + partner];
    }
    __syncthreads();
    return o;
}

// A level reduced by whole workgroups, down: as k_bi_down, then the product of the
// workgroup's thread totals goes to next[blockIdx.x].
template <int kPer>
__global__ void __launch_bounds__(kBlock) k_bi_down_wg(const uint32_t* __restrict__ src, size_t ss, size_t n, int shifted,
                                                       Fr shift, uint32_t* __restrict__ prefix, size_t ps,
                                                       uint32_t* __restrict__ next, size_t ns) {
    __shared__ uint32_t lds[8 * kBlock];
    const size_t base = blockIdx.x * (size_t)kBlock * kPer + threadIdx.x;
    Fr x[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const size_t i = base + (size_t)j * kBlock;
        x[j] = i < n ? bi_load(src, ss, i, shifted, shift) : fr_one();
    }
    Fr acc = x[0];
    if (base < n) fr_store(prefix, ps, base, acc);
#pragma unroll
    for (int j = 1; j < kPer; ++j) {
        const size_t i = base + (size_t)j * kBlock;
        if (i < n) {
            acc = fr_mul(acc, x[j]);
            fr_store(prefix, ps, i, acc);
        }
    }
    const Fr total = block_scan_mul<kBlock>(acc, lds, false);
    if (threadIdx.x == kBlock - 1) fr_store(next, ns, blockIdx.x, total);
}

// Up: inv_next[blockIdx.x] is the inverse of the workgroup's product; a thread's
// own inverse is that times the totals of all other threads of the workgroup.
template <int kPer>
__global__ void __launch_bounds__(kBlock) k_bi_up_wg(const uint32_t* __restrict__ src, size_t ss, size_t n, int shifted,
                                                     Fr shift, const uint32_t* prefix, size_t ps,
                                                     const uint32_t* __restrict__ inv_next, size_t is, uint32_t* out,
                                                     size_t os) {
    __shared__ uint32_t lds[8 * kBlock];
    const size_t base = blockIdx.x * (size_t)kBlock * kPer + threadIdx.x;
    // how many elements this thread has; its total is the last of its running products
    int count = 0;
    if (base < n) {
        const size_t left = (n - base + kBlock - 1) / kBlock;
        count = left < (size_t)kPer ? (int)left : kPer;
    }
    const Fr total = count ? fr_load(prefix, ps, base + (size_t)(count - 1) * kBlock) : fr_one();
    const Fr pre = block_scan_mul<kBlock>(total, lds, false);
    const Fr suf = block_scan_mul<kBlock>(total, lds, true);
    const Fr others = fr_mul(block_neighbour<kBlock>(pre, lds, false), block_neighbour<kBlock>(suf, lds, true));
    Fr inv = fr_mul(fr_load(inv_next, is, blockIdx.x), others);
    // back over the elements, at most eight at a time: their loads do not depend on the chain of products
    constexpr int kStep = kPer < 8 ? kPer : 8;
#pragma unroll
    for (int part = kPer / kStep - 1; part >= 0; --part) {
        Fr x[kStep], before[kStep];
#pragma unroll
        for (int q = 0; q < kStep; ++q) {
            const int j = part * kStep + q;
            const size_t i = base + (size_t)j * kBlock;
            x[q] = j > 0 && j < count ? bi_load(src, ss, i, shifted, shift) : fr_one();
            before[q] = j > 0 && j < count ? fr_load(prefix, ps, i - kBlock) : fr_one();
        }
#pragma unroll
        for (int q = kStep - 1; q >= 0; --q) {
            const int j = part * kStep + q;
            if (j < count) {
                const size_t i = base + (size_t)j * kBlock;
                if (j > 0) {
                    fr_store(out, os, i, fr_mul(inv, before[q]));
                    inv = fr_mul(inv, x[q]);
                } else {
                    fr_store(out, os, i, inv);
                }
            }
        }
    }
}

// The last levels of all inversions of a call, a workgroup each: its chain of eight products
// is what such a level costs (three inversions one after the other 24 and 38 us, together 8
// and 13).
struct BiTop {
    const uint32_t* src;
    size_t ss, n;
    int shifted;
    uint32_t* total_words;
    uint32_t* out;
    size_t os;
    Fr inv_total;
};
template <int NJ>
struct BiTopArgs {
    BiTop job[NJ];
    Fr shift;
    uint32_t* flag_words;
    uint32_t* ticket;  // (more than one job)
    uint32_t seq;
};

// Grand totals of the last levels (n <= THREADS) to total_words (Montgomery limbs).
template <int THREADS, int NJ>
__global__ void __launch_bounds__(THREADS) k_bi_top_total(BiTopArgs<NJ> args) {
    __shared__ uint32_t lds[8 * THREADS];
    const BiTop& g = args.job[NJ == 1 ? 0 : blockIdx.x];
    Fr x = threadIdx.x < g.n ? bi_load(g.src, g.ss, threadIdx.x, g.shifted, args.shift) : fr_one();
    Fr p = block_scan_mul<THREADS>(x, lds, false);
    if (threadIdx.x == THREADS - 1) {
#pragma unroll
        for (int k = 0; k < 8; ++k) g.total_words[k] = p.l[k];
        mailbox_written();
        if (gridDim.x == 1) {
            mailbox_publish(args.flag_words, args.seq);
        } else if (atomicAdd(args.ticket, 1u) == gridDim.x - 1) {
            *args.ticket = 0;
            mailbox_publish(args.flag_words, args.seq);
        }
    }
}

// out_t = inv_total * (product of the others) for the last levels.
template <int THREADS, int NJ>
__global__ void __launch_bounds__(2 * THREADS) k_bi_top_finish(BiTopArgs<NJ> args) {
    __shared__ uint32_t lds[16 * THREADS];
    const BiTop& g = args.job[NJ == 1 ? 0 : blockIdx.x];
    const uint32_t* __restrict__ const src = g.src;
    const size_t ss = g.ss, n = g.n, os = g.os;
    const int shifted = g.shifted;
    const Fr shift = args.shift, inv_total = g.inv_total;
    uint32_t* const out = g.out;
    const int t = threadIdx.x & (THREADS - 1);
    const Fr x = (size_t)t < n ? bi_load(src, ss, t, shifted, shift) : fr_one();
    Fr others = block_scan_both<THREADS>(x, lds);
    if (threadIdx.x >= THREADS) {
#pragma unroll
        for (int k = 0; k < 8; ++k) lds[k * THREADS + t] = others.l[k];
    } else {
        others = fr_mul(others, inv_total);
    }
    __syncthreads();
    if (threadIdx.x < THREADS && (size_t)t < n) {
        Fr after;
#pragma unroll
        for (int k = 0; k < 8; ++k) after.l[k] = lds[k * THREADS + t];
        fr_store(out, os, t, fr_mul(others, after));
    }
}

static const size_t kBiTopMax = kBlock;  // values the top kernels take

// Whether level `depth` of length n is reduced by whole workgroups, how many
// elements a thread then takes (as few as still leave the top at most kBiTopMax
// values: the chain of products is what such a level costs), and the next level's length.
static bool bi_by_workgroups(int depth, size_t n) {
    if (depth >= 1) return n <= kBiTopMax * kBlock * kBiK;
    // the threads of one workgroup leave the top its 256 values straight away; their chain, one product per 256 elements
    // there and two back, costs less than the workgroups' scans up to ten of them (whole calls by threads and by
    // workgroups: 512 elements 57.6 and 76.4 us, 2048 71.4 and 77.3, 2560 76.0 and 77.9, 3072 80.5 and 78.2)
    return n > (size_t)kBlock * 10 && n <= kBiTopMax * kBlock * 2;
}
static int bi_wg_per_thread(size_t n) {
    int per = 2;
    while (per < kBiK && div_up(n, (size_t)kBlock * per) > kBiTopMax) per *= 2;
    return per;
}
static size_t bi_next_size(int depth, size_t n) {
    if (bi_by_workgroups(depth, n)) return div_up(n, (size_t)kBlock * bi_wg_per_thread(n));
    return div_up(n, (size_t)kBlock * kBiK) * kBlock;
}

template <int kPer>
static void bi_launch_wg(bool down, unsigned blocks, hipStream_t stream, const BatchInverseJob::Level& lv, const Fr& shift,
                         uint32_t* next_or_inv, size_t ns) {
    if (down)
        hipLaunchKernelGGL(k_bi_down_wg<kPer>, dim3(blocks), dim3(kBlock), 0, stream, lv.x, lv.xs, lv.n, lv.shifted, shift,
                           lv.p, lv.ps, next_or_inv, ns);
    else
        hipLaunchKernelGGL(k_bi_up_wg<kPer>, dim3(blocks), dim3(kBlock), 0, stream, lv.x, lv.xs, lv.n, lv.shifted, shift, lv.p,
                           lv.ps, next_or_inv, ns, lv.p, lv.ps);
}
static void bi_launch_wg_level(bool down, hipStream_t stream, const BatchInverseJob::Level& lv, const Fr& shift,
                               uint32_t* next_or_inv, size_t ns) {
    const int per = bi_wg_per_thread(lv.n);
    const unsigned blocks = (unsigned)div_up(lv.n, (size_t)kBlock * per);
    if (per == 2) bi_launch_wg<2>(down, blocks, stream, lv, shift, next_or_inv, ns);
    else if (per == 4) bi_launch_wg<4>(down, blocks, stream, lv, shift, next_or_inv, ns);
    else if (per == 8) bi_launch_wg<8>(down, blocks, stream, lv, shift, next_or_inv, ns);
    else bi_launch_wg<16>(down, blocks, stream, lv, shift, next_or_inv, ns);
}

size_t batch_inverse_scratch_bytes(size_t n) {
    Carver cv(nullptr, 0);
    size_t m = n;
    for (int depth = 0; m > kBiTopMax; ++depth) {
        m = bi_next_size(depth, m);
        cv.limbs(m);  // level values
        cv.limbs(m);  // level prefixes, then inverses
    }
    return cv.used();
}

static BiSecond bi_second_of(const BatchInverseJob& job, int depth) {
    if (depth == 0 && job.n2) return BiSecond{job.src2, job.src2_stride, job.dst2, job.dst2_stride, job.lv[0].n - job.n2};
    return BiSecond{nullptr, 0, nullptr, 0, SIZE_MAX};
}

bool batch_inverse_can_join(size_t n1, size_t n2) {
    return n1 % ((size_t)kBlock * kBiK) == 0 && !bi_by_workgroups(0, n1 + n2);
}

int batch_inverse_begin(BatchInverseJob& job, uint32_t* dst, size_t dst_stride, const uint32_t* src, size_t src_stride,
                        size_t n, const host::F& shift, Carver& cv, uint32_t* total_words, hipStream_t stream, uint32_t* dst2, size_t dst2_stride, const uint32_t* src2,
                        size_t src2_stride, size_t n2) {
    typedef BatchInverseJob::Level Level;
    if (n2 && !batch_inverse_can_join(n, n2)) return ZK_E_BADARG;
    job.depth = 0;
    job.shift = to_dev(shift);
    job.n2 = n2;
    job.src2 = src2;
    job.src2_stride = src2_stride;
    job.dst2 = dst2;
    job.dst2_stride = dst2_stride;
    job.total_words = total_words;
    int shifted0 = host::is_zero(shift) ? 0 : 1;
    job.lv[0] = Level{src, src_stride, dst, dst_stride, n + n2, shifted0};
    while (job.lv[job.depth].n > kBiTopMax) {
        const Level& cur = job.lv[job.depth];
        const size_t m = bi_next_size(job.depth, cur.n);
        const unsigned blocks = (unsigned)div_up(cur.n, (size_t)kBlock * kBiK);
        uint32_t* x = cv.limbs(m);
        uint32_t* p = cv.limbs(m);
        if (!x || !p) return ZK_E_BUFSZ;
        if (bi_by_workgroups(job.depth, cur.n))
            bi_launch_wg_level(true, stream, cur, job.shift, x, m);
        else
            hipLaunchKernelGGL(k_bi_down, dim3(blocks), dim3(kBlock), 0, stream, cur.x, cur.xs, cur.n, cur.shifted,
                               job.shift, cur.p, cur.ps, x, m, bi_second_of(job, job.depth));
        ++job.depth;
        job.lv[job.depth] = Level{x, m, p, m, m, 0};
    }
    ZK_HIP_TRY(hipGetLastError());
    return ZK_OK;
}

template <int NJ>
static BiTopArgs<NJ> bi_tops(const BatchInverseJob* const* jobs, int njobs) {
    BiTopArgs<NJ> args;
    memset(&args, 0, sizeof args);
    args.shift = jobs[0]->shift;
    for (int q = 0; q < njobs; ++q) {
        const BatchInverseJob::Level& top = jobs[q]->lv[jobs[q]->depth];
        BiTop& g = args.job[q];
        g.src = top.x;
        g.ss = top.xs;
        g.n = top.n;
        g.shifted = top.shifted;
        g.total_words = jobs[q]->total_words;
        g.out = top.p;
        g.os = top.ps;
    }
    return args;
}

int batch_inverse_totals(const BatchInverseJob* const* jobs, int njobs, uint32_t* flag_words, uint32_t seq, uint32_t* ticket,
                         hipStream_t stream) {
    if (njobs < 1 || njobs > kBatchInverseMaxJobs || (njobs > 1 && !ticket)) return ZK_E_BADARG;
    const auto launch = [&](auto args) {
        args.flag_words = flag_words;
        args.ticket = ticket;
        args.seq = seq;
        hipLaunchKernelGGL((k_bi_top_total<kBlock, sizeof args.job / sizeof(BiTop)>), dim3(njobs), dim3(kBlock), 0, stream, args);
    };
    if (njobs == 1) launch(bi_tops<1>(jobs, 1));  // (few arguments where few do)
    else launch(bi_tops<kBatchInverseMaxJobs>(jobs, njobs));
    ZK_HIP_TRY(hipGetLastError());
    return ZK_OK;
}

int batch_inverse_end(const BatchInverseJob* const* jobs, const host::F* inv_totals, int njobs, hipStream_t stream) {
    typedef BatchInverseJob::Level Level;
    if (njobs < 1 || njobs > kBatchInverseMaxJobs) return ZK_E_BADARG;
    const auto launch = [&](auto args) {
        for (int q = 0; q < njobs; ++q) args.job[q].inv_total = to_dev(inv_totals[q]);
        hipLaunchKernelGGL((k_bi_top_finish<kBlock, sizeof args.job / sizeof(BiTop)>), dim3(njobs), dim3(2 * kBlock), 0, stream, args);
    };
    if (njobs == 1) launch(bi_tops<1>(jobs, 1));
    else launch(bi_tops<kBatchInverseMaxJobs>(jobs, njobs));
    for (int q = 0; q < njobs; ++q) {
        const BatchInverseJob& job = *jobs[q];
        for (int d = job.depth - 1; d >= 0; --d) {
            const Level& cur = job.lv[d];
            const Level& up = job.lv[d + 1];
            const unsigned blocks = (unsigned)div_up(cur.n, (size_t)kBlock * kBiK);
            if (bi_by_workgroups(d, cur.n))
                bi_launch_wg_level(false, stream, cur, job.shift, up.p, up.ps);
            else
                hipLaunchKernelGGL(k_bi_up, dim3(blocks), dim3(kBlock), 0, stream, cur.x, cur.xs, cur.n, cur.shifted, job.shift,
                                   cur.p, cur.ps, up.p, up.ps, cur.p, cur.ps, bi_second_of(job, d));
        }
    }
    ZK_HIP_TRY(hipGetLastError());
    return ZK_OK;
}

int batch_inverse_run(uint32_t* dst, size_t dst_stride, const uint32_t* src, size_t src_stride, size_t n,
                      const host::F& shift, Carver& cv, Mailbox* mb, hipStream_t stream) {
    if (n == 0) return ZK_OK;
    BatchInverseJob job;
    uint32_t seq = mb->next_seq();
    ZK_TRY(batch_inverse_begin(job, dst, dst_stride, src, src_stride, n, shift, cv, mb->words + kMailboxInvA,
                               stream, nullptr, 0, nullptr, 0, 0));
    const BatchInverseJob* const jobs[1] = {&job};
    ZK_TRY(batch_inverse_totals(jobs, 1, mb->words, seq, nullptr, stream));
    ZK_TRY(mailbox_wait(mb, seq, stream));
    host::F total = from_dev(mb->words + kMailboxInvA);
    if (host::is_zero(total)) {
        ZK_HIP_TRY(hipStreamSynchronize(stream));  // error codes that depend on data come from an idle stream
        return ZK_E_ZERO_DENOM;
    }
    const host::F inv_total = host::inv(total);
    return batch_inverse_end(jobs, &inv_total, 1, stream);
}

}  // namespace zkmi

using namespace zkmi;

extern "C" {

size_t fr_batch_inverse_workspace_bytes(size_t n) { return batch_inverse_scratch_bytes(n); }

int fr_batch_inverse(fr_vec dst, fr_vec src, void* ws, size_t ws_bytes, void* stream) {
    size_t n = dst.n;
    if (!vec_ok(dst, n) || !vec_ok(src, n)) return ZK_E_BADARG;
    if (n == 0) return ZK_OK;
    if (dst.limbs == src.limbs) return ZK_E_BADARG;
    if (!ws || ws_bytes < batch_inverse_scratch_bytes(n)) return ZK_E_BUFSZ;
    Mailbox* mb;
    ZK_TRY(mailbox_get(&mb));
    Carver cv(ws, ws_bytes);
    ZK_TRY(batch_inverse_run(dst.limbs, dst.stride, src.limbs, src.stride, n, host::zero(), cv, mb, as_stream(stream)));
    ZK_HIP_TRY(hipStreamSynchronize(as_stream(stream)));
    return ZK_OK;
}

}  // extern "C"

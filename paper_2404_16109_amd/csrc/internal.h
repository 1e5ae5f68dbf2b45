// Launchers shared between the translation units of the library.
#pragma once
#include "common.h"
#include "small_dev.h"

namespace zkmi {

// ---- batch inversion ------------------------------------------------------
// dst_i = 1 / (src_i + shift) for i < n (shift in Montgomery form; pass zero for
// a plain inverse).  dst must not overlap src.  Scratch comes from `cv`.
// Synchronises the stream once (the single field inversion is done on the host).
size_t batch_inverse_scratch_bytes(size_t n);
int batch_inverse_run(uint32_t* dst, size_t dst_stride, const uint32_t* src, size_t src_stride, size_t n,
                      const host::F& shift, Carver& cv, Mailbox* mb, hipStream_t stream);

// The same in parts, so that several inversions (of one shift) can share launches and one
// wait: `begin` runs an inversion's down passes, `totals` leaves all grand totals
// (Montgomery limbs) at their total_words and publishes `seq` (`ticket`: one zeroed word
// of device memory, left zero; may be null for one job), `end` takes the inverses of those
// totals and runs the up passes.
static const int kBatchInverseMaxJobs = 16;
struct BatchInverseJob {
    struct Level {
        const uint32_t* x;
        size_t xs;
        uint32_t* p;
        size_t ps;
        size_t n;
        int shifted;
    };
    Level lv[16];
    int depth = 0;
    Fr shift;
    // a second vector inverted together with the first (its elements follow the first's)
    size_t n2 = 0;
    const uint32_t* src2 = nullptr;
    size_t src2_stride = 0;
    uint32_t* dst2 = nullptr;
    size_t dst2_stride = 0;
    uint32_t* total_words = nullptr;
};
// src2 (n2 elements, may be none: n2 = 0) is inverted into dst2 by the same passes,
// shifted like src; needs batch_inverse_can_join(n, n2) and scratch for n + n2 elements.
bool batch_inverse_can_join(size_t n, size_t n2);
int batch_inverse_begin(BatchInverseJob& job, uint32_t* dst, size_t dst_stride, const uint32_t* src, size_t src_stride,
                        size_t n, const host::F& shift, Carver& cv, uint32_t* total_words, hipStream_t stream, uint32_t* dst2, size_t dst2_stride, const uint32_t* src2,
                        size_t src2_stride, size_t n2);
int batch_inverse_totals(const BatchInverseJob* const* jobs, int njobs, uint32_t* flag_words, uint32_t seq, uint32_t* ticket,
                         hipStream_t stream);
int batch_inverse_end(const BatchInverseJob* const* jobs, const host::F* inv_totals, int njobs, hipStream_t stream);

// ---- sums -----------------------------------------------------------------
// Partial sums buffer for reductions: up to kMaxPartialBlocks blocks.
static const unsigned kMaxPartialBlocks = 4096;

// Adds up `nv` interleaved per-block partial values (block b, value q at
// element b*nv + q of `partials`, limb-major with stride pstride) and writes
// the nv totals, Montgomery limbs, to out_words (device-visible host memory
// or device memory): value q at out_words[8q .. 8q+8).
// `words` is the mailbox the flag lives in; seq != 0 publishes completion, for
// which `ticket` (one zeroed word of device memory, left zero) is needed.
void launch_final_sum(const uint32_t* partials, size_t pstride, unsigned nblocks, int nv, uint32_t* out_words,
                      uint32_t* words, uint32_t seq, uint32_t* ticket, hipStream_t stream);

// Same for two partial arrays at once: nv1 values per block from the first, then
// nv2 from the second (nv2 may be 0); totals at out_words[8q..], first array first.
// note: two words of device memory that go out beside them, to note_out, if not null.
void launch_final_sum2(const uint32_t* part1, size_t pstride1, int nv1, const uint32_t* part2, size_t pstride2, int nv2,
                       unsigned nblocks, uint32_t* out_words, uint32_t* words, uint32_t seq, uint32_t* ticket,
                       hipStream_t stream, const uint32_t* note = nullptr, uint32_t* note_out = nullptr);

// sum_i a_i into mailbox words [0, 8).
size_t sum_scratch_bytes(size_t n);
int sum_run(const uint32_t* a, size_t stride, size_t n, Carver& cv, Mailbox* mb, uint32_t seq, hipStream_t stream);

// ---- eq tables --------------------------------------------------------------
// dst_x = prod_{t < nvars} (u_t x_t + (1-u_t)(1-x_t)), x in {0,1}^nvars, first
// variable = top bit.  u: host, Montgomery.
int eq_table_run(uint32_t* dst, size_t stride, const host::F* u, int nvars, hipStream_t stream);
struct EqTable {
    uint32_t* dst;
    size_t stride;
    const host::F* u;
    int nvars;
};
int eq_tables_run(const EqTable* tables, int count, hipStream_t stream);  // one or two, in one launch

// ---- multilinear evaluation ---------------------------------------------------
// a~(point) into out_words[0, 8) (Montgomery); a is not modified.
size_t mle_scratch_bytes(int nvars);
// Up to kMleMaxJobs evaluations at up to two points in the same launches; job q's
// value goes to its out_words (eight Montgomery words in device-visible memory).
static const int kMleMaxJobs = 5;
struct MleJob {
    const uint32_t* a;
    size_t stride;
    int nvars;
    const host::F* point;  // jobs with the same pointer and length share their constants
    uint32_t* out_words;
};
size_t mle_scratch_bytes_many(const int* nvars, int njobs);
int mle_eval_launch(const MleJob* jobs, int njobs, Carver& cv, Mailbox* mb, uint32_t seq, hipStream_t stream);
int mle_eval_run(const uint32_t* a, size_t stride, int nvars, const host::F* point, Carver& cv, Mailbox* mb,
                 uint32_t seq, hipStream_t stream);

// p[0..n) = v (a kernel, so that it can sit in a captured graph).
void launch_fill_u32(uint32_t* p, size_t n, uint32_t v, hipStream_t stream);

}  // namespace zkmi

// A stage of multilinear evaluations, whose launches are laid out by mle_eval_begin (poly.hip).
// Its workgroups also run beside others in one launch (k_leaves_beside).
#pragma once
#include "internal.h"
#include "mfma_dev.h"

namespace zkmi {

// One stage of up to kMleMaxJobs evaluations: workgroup b of a job makes outputs
// 128 b .. 128 b + 127, its wavefronts sharing the constants (each adds a quarter of
// them up; the column sums meet in LDS), so that the short last stages are not one
// wavefront's chain of 64 loads.
struct MleStageJob {
    ToepSource src;
    uint32_t* dst;
    size_t dst_stride;
    size_t P;
    const uint4* table;
    uint32_t C;
    uint32_t first_block;
    ToepBias bias;
};
struct MleStageArgs {
    MleStageJob job[kMleMaxJobs];
    int njobs;
    uint32_t* words;   // the mailbox, if this launch publishes
    uint32_t* ticket;
    uint32_t seq;
};

typedef int MleParts[4][4][16][64];  // [from wavefront][tile][row][lane]
__device__ __forceinline__ void mle_stage_block(const MleStageArgs& args, uint32_t block, MleParts& part) {
    int q = 0;
    while (q + 1 < args.njobs && block >= args.job[q + 1].first_block) ++q;
    const MleStageJob& job = args.job[q];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 31;
    const size_t base = (size_t)(block - job.first_block) * 128;
    v16i acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0;
    const unsigned c0 = job.C * wave / 4, c1 = job.C * (wave + 1) / 4;
    if (job.src.vec) toeplitz_accumulate<true>(acc, job.src, job.P, base, job.table, c0, c1);
    else toeplitz_accumulate<false>(acc, job.src, job.P, base, job.table, c0, c1);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) part[wave][j][r][lane] = acc[j][r];
    __syncthreads();
    if (wave < 2) {
        // tiles (wave, wave + 2) with 16-byte places: lanes 0..31 then hold element 4 i + wave, the others 4 i + 2 + wave;
        // otherwise tiles (2 wave, 2 wave + 1): element 64 wave + lane
        const int ta = job.src.vec ? wave : 2 * wave, tb = job.src.vec ? wave + 2 : 2 * wave + 1;
        v16i a, b;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            a[r] = part[0][ta][r][lane] + part[1][ta][r][lane] + part[2][ta][r][lane] + part[3][ta][r][lane];
            b[r] = part[0][tb][r][lane] + part[1][tb][r][lane] + part[2][tb][r][lane] + part[3][tb][r][lane];
        }
        const Fr v = toeplitz_finish(a, b, job.bias);
        const size_t e = job.src.vec ? base + 4 * (size_t)i + 2 * (lane >> 5) + wave : base + 64 * (size_t)wave + lane;
        if (e < job.P) {
            fr_store(job.dst, job.dst_stride, e, v);
            if (args.seq) mailbox_written();
        }
    }
}

// What is left to launch of some evaluations: step t's workgroups, the last step's results going to the mailbox.
static const int kMleMaxSteps = 6;  // of six variables each, 32 at most
struct MlePlan {
    MleStageArgs step[kMleMaxSteps];
    uint32_t blocks[kMleMaxSteps];
    int steps;
    MleJob jobs[kMleMaxJobs];
    int njobs;
    uint32_t seq;
};
// Lays them out and makes the constants.
int mle_eval_begin(MlePlan& plan, const MleJob* jobs, int njobs, Carver& cv, Mailbox* mb, uint32_t seq, hipStream_t stream);
// Launches the steps from `first` on.
int mle_eval_rest(const MlePlan& plan, int first, Mailbox* mb, hipStream_t stream);

}  // namespace zkmi

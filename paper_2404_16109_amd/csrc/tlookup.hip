// tlookup prover and verifier (Section 4 of the paper, Protocol 1), host
// orchestration.  All arithmetic on tensors runs in the kernels of
// tlookup_kernels.h, batch_inverse.hip and poly.hip; the host only drives the
// Fiat-Shamir transcript and turns the handful of sums a round returns into
// the round polynomial.
//
// How a round is computed.  With x = (X, rest) after binding k variables,
//   e~(u, x) = c_k * e~(u_k, X) * e_rest(rest),   c_k = prod_{t<k} e~(u_t, r_t),
// so the data side of g_k is  alpha c_k e~(u_k, X) q(X) + sA(X)  with
//   q(X) = sum_rest e_rest A(X,rest) (S(X,rest)+beta)   (degree 2 in X),
//   sA(X) = sum_rest A(X,rest)                          (degree 1),
// and e_rest never has to be folded: it is looked up in two small tables (low
// and high remaining variables).  The table side is the constant
// 2^-(k+1) * c_B while the variable being bound is not one of the table's, and
// 2^-h (alpha^2 c'_k e~(u_k,X) qT(X) - bm(X)) afterwards.
//
// What computes a round's sums is decided by plan_round.  From a vector of field
// elements the first pass over A and S yields the sums of the first TWO rounds
// (k_round_first_two) and the third round's kernel binds both variables at once; in the
// large folding rounds the kernel sums one side of the round (X = 0 or X = 1) and
// the other side follows here from the running claim; the rounds of the last
// variables come several from one pass (grid_dev.h), the very last are the host's.
#include "internal.h"
#include "tlookup_kernels.h"
#include "tlookup_round29.h"
#include "tlookup_rows.h"
#include "grid_dev.h"
#include "long_host.h"
#include "transcript.h"

#include <algorithm>
#include <memory>
#include <new>

namespace zkmi {

static const int kLoBits = 12;  // low eq table covers up to this many variables

// Pool of eq tables for a point u of n variables.
//   suffix[s], s = 0..min(kLoBits, n-1): e~ over the last s variables;
//   suffix29[s]: the same times 2^10, for the rounds on 29-bit limbs, whose
//                multiplication divides by 2^261 instead of 2^256 (twice on the way
//                into a sum of products);
//   high[k], for rounds k with n-k-1 > kLoBits: e~ over variables k+1 .. n-kLoBits-1.
struct EqPool {
    uint32_t* pool = nullptr;
    size_t stride = 0;
    uint32_t suffix_off[kLoBits + 1];
    uint32_t suffix29_off[kLoBits + 1];  // within pool29
    uint32_t high_off[32];
    uint4* pool29 = nullptr;  // the scaled suffix tables as 29-bit limbs, three planes of count29 elements
    size_t count29 = 0;
    int n = 0;

    static size_t entries29(int n) {
        size_t total = 0;
        int smax = n - 1 < kLoBits ? n - 1 : kLoBits;
        for (int s = 0; s <= smax; ++s) total += (size_t)1 << s;
        return total ? total : 1;
    }

    static size_t entries(int n) {
        size_t total = 0;
        int smax = n - 1 < kLoBits ? n - 1 : kLoBits;
        for (int s = 0; s <= smax; ++s) total += (size_t)2 << s;
        for (int k = 0; k < n; ++k) {
            int rest = n - k - 1;
            if (rest > kLoBits) total += (size_t)1 << (rest - kLoBits);
        }
        return total ? total : 1;
    }

    // Weights of round k (remaining variables k+1 .. n-1).
    EqSplit round(int k) const {
        int rest = n - k - 1;
        EqSplit e;
        e.pool = pool;
        e.stride = stride;
        e.lbits = rest < kLoBits ? rest : kLoBits;
        e.lo_off = suffix_off[e.lbits];
        e.has_hi = rest > kLoBits;
        e.hi_off = e.has_hi ? high_off[k] : 0;
        return e;
    }
};

static int eq_pool_build(EqPool& ep, const host::F* u, int n, Carver& cv, hipStream_t stream) {
    ep.n = n;
    ep.stride = EqPool::entries(n);
    ep.pool = cv.limbs(ep.stride);
    ep.count29 = EqPool::entries29(n);
    ep.pool29 = (uint4*)cv.take(ep.count29 * 36);
    if (!ep.pool || !ep.pool29) return ZK_E_BUFSZ;
    EqPoolArgs args;
    memset(&args, 0, sizeof args);
    for (int t = 0; t < n; ++t) args.u[t] = to_dev(u[t]);
    int q = 0;
    uint32_t off = 0;
    int smax = n - 1 < kLoBits ? n - 1 : kLoBits;
    for (int s = 0; s <= smax; ++s) {
        ep.suffix_off[s] = off;
        args.offset[q] = off;
        args.var0[q] = (uint8_t)(n - s);
        args.nvars[q] = (uint8_t)s;
        off += 1u << s;
        ++q;
    }
    if (n == 0) ep.suffix_off[0] = 0;
    args.scale = to_dev(host::from_u64(1024));
    args.pool29 = ep.pool29;
    args.count29 = ep.count29;
    args.first29 = off;
    for (int s = 0; s <= smax; ++s) {
        ep.suffix29_off[s] = off - args.first29;
        args.offset[q] = off;
        args.var0[q] = (uint8_t)(n - s);
        args.nvars[q] = (uint8_t)s;
        args.scaled[q] = 1;
        off += 1u << s;
        ++q;
    }
    for (int k = 0; k < n; ++k) {
        int rest = n - k - 1;
        if (rest <= kLoBits) continue;
        ep.high_off[k] = off;
        args.offset[q] = off;
        args.var0[q] = (uint8_t)(k + 1);
        args.nvars[q] = (uint8_t)(rest - kLoBits);
        off += 1u << (rest - kLoBits);
        ++q;
    }
    args.ntables = q;
    args.total = off;
    if (q > 64) return ZK_E_BADARG;
    if (off) {
        launch_eq_pool(ep.pool, ep.stride, args, stream);
        ZK_HIP_TRY(hipGetLastError());
    }
    return ZK_OK;
}

// Quadratic through value(0), value(1) and leading coefficient, at X = 0..3.
static void quad_values(host::F out[4], const host::F& v0, const host::F& v1, const host::F& lead) {
    using namespace host;
    out[0] = v0;
    out[1] = v1;
    F lead2 = add(lead, lead);
    out[2] = add(sub(add(v1, v1), v0), lead2);                                 // 2 v1 - v0 + 2 lead
    out[3] = add(sub(add(add(v1, v1), v1), add(v0, v0)), add(add(lead2, lead2), lead2));  // 3 v1 - 2 v0 + 6 lead
}

// Line through value(0), value(1) at X = 0..3.
static void line_values(host::F out[4], const host::F& v0, const host::F& v1) {
    using namespace host;
    F d = sub(v1, v0);
    out[0] = v0;
    out[1] = v1;
    out[2] = add(v1, d);
    out[3] = add(out[2], d);
}

// ---- workspace layout -------------------------------------------------------------

struct ProveWs {
    uint32_t* A;        // D
    uint32_t* Sf;       // D/2
    uint4* A29;         // folded A and S while they are held in 29-bit limbs: D/2 elements of 36 bytes each
    uint4* S29;
    uint32_t* B;        // N
    uint32_t* Bf;       // N/2: B is folded back and forth between B and Bf
    uint32_t* Tf;       // N/2
    uint32_t* M;        // N
    uint32_t* m;        // N counts
    uint32_t* slots;    // hash of T
    uint32_t cap_mask;
    uint32_t* canon;    // N
    uint4* rows;        // N rows of T, eight words each
    uint4* rows_b;      // N rows of B, sixteen words each (k_rows_of)
    uint32_t* found;    // D: the row of every S_i, found while counting (calls without hints), else null
    uint32_t* hist;     // per-workgroup histograms (tables of up to 2^16 rows), else null
    uint32_t hist_parts;
    uint32_t* flags;    // [0] duplicate flag, [1] ticket of the final sums, [2..3] smallest bad index (64-bit)
    SmallFold4* fold4;  // constants of the first fold when S comes as small integers (tlookup_prove_small)
    uint32_t nleaves;
    uint32_t* dig_rows;    // the shorter rows of A's tree above kTreeChunk leaves
    uint32_t* dig_rows_b;  // the same for B
    size_t part_blocks; // capacity of the two partial-sum buffers, in workgroups
    uint32_t* partD;    // part_blocks * 5
    uint32_t* partT;    // part_blocks * 6
};

// Most workgroups a round kernel can be launched with: spans never shrink below
// 2^kLoBits pairs while high weight tables are in use.
static size_t round_blocks_max(size_t D) {
    size_t by_span = (D / 2) >> kLoBits;
    return by_span > kMaxPartialBlocks ? by_span : kMaxPartialBlocks;
}

static const size_t kLdsHistMaxRows = (size_t)1 << 16;  // packed 16-bit counters: 128 KiB of LDS
static const uint32_t kHistParts = 256;                // one workgroup per compute unit

// ---- digest of a vector (stand-in for its commitment) ----------------------------------
// Scratch: the leaf digests and, for rows longer than kTreeChunk, the rows above
// them (each at most 1/kTreeChunk of the one below: twice the first is room for all).
static size_t vec_digest_leaves(size_t n) { return n / kVecLeaf ? n / kVecLeaf : 1; }
static size_t vec_digest_row_digests(size_t n) {
    const size_t first = vec_digest_leaves(n) / kTreeChunk;
    return first ? 2 * first : 1;
}

// Enqueues the hash trees over up to kDigestMaxJobs vectors (n elements each, powers
// of two): their last rows (at most kTreeHostRow digests) go to pinned host memory,
// and the last launch publishes `seq` if it is not zero (`ticket`: one zeroed word of
// device memory, left zero).  The host then finishes each tree (vec_digest_finish); to_host
// (host_leaves): it gets the leaves' bytes and hashes them itself.
// leaves: room for the sum of vec_digest_leaves(n); rows: vec_digest_row_digests(n)
// digests each.
struct VecDigestJob {
    uint32_t* v;  // only read, unless `from` says that it is made here
    size_t stride, n;
    uint32_t* rows;
    LeafGather from;
    const uint32_t* host_row = nullptr;  // set by the launch: the row handed to the host
    uint32_t host_count = 0;
    uint8_t* shipped = nullptr;          // or the leaves' bytes, leaf_bytes each
    size_t leaf_bytes = 0;
};

// Whether the host hashes a call's leaves: they are few, and it has the instructions for it.
static bool host_leaves(size_t leaves, bool sha_instructions) { return leaves <= kHostLeaves && sha_instructions; }

template <int MODE>
static void launch_leaves(const VecLeavesArgs& lv, hipStream_t stream) {
    if (leaves_in_pairs<MODE>(lv.groups))
        hipLaunchKernelGGL(k_vec_leaves_piped<MODE>, dim3((lv.groups + 1) / 2), dim3(256), 0, stream, lv);
    else hipLaunchKernelGGL(k_vec_leaves<MODE>, dim3(lv.groups), dim3(64), 0, stream, lv);
}

template <int MODE>
static void launch_leaves_to_host(const VecLeavesArgs& lv, hipStream_t stream) {
    hipLaunchKernelGGL(k_leaves_to_host<MODE>, dim3((unsigned)div_up(lv.groups, kBlock)), dim3(kBlock), 0, stream, lv);
}

// What may run in the launch of a verification's leaves.
struct LeavesBeside {
    LeafDigestJob counts;
    const MleStageArgs* stage;
    uint32_t stage_blocks;
    bool launched;  // it has: the leaves are not the host's
};

// The jobs that have rows (LeafGather) all compare them with S, or all with the
// integers, or none: by `ints` and whether they have an S; those that are only hashed do not.
static int vec_digest_launch(VecDigestJob* jobs, int njobs, bool to_host, uint32_t* leaves, Mailbox* mb, uint32_t seq, uint32_t* ticket,
                             hipStream_t stream, const SmallSource* ints = nullptr, const BadWords& bad = BadWords{},
                             LeavesBeside* beside = nullptr) {
    if (njobs < 1 || njobs > kDigestMaxJobs) return ZK_E_BADARG;
    ZK_TRY(mailbox_bulk(mb, 0));
    VecLeavesArgs lv{};
    if (ints) lv.ints = *ints;
    lv.bad = bad;
    lv.njobs = njobs;
    lv.words = mb->words;
    lv.ticket = ticket;
    const uint32_t* in[kDigestMaxJobs];
    size_t cnt[kDigestMaxJobs];
    uint32_t* rows[kDigestMaxJobs];
    size_t total = 0;
    uint32_t blocks = 0;
    bool more = false;
    for (int q = 0; q < njobs; ++q) {
        VecDigestJob& j = jobs[q];
        cnt[q] = vec_digest_leaves(j.n);
        rows[q] = j.rows;
        uint32_t* host_row = (uint32_t*)mb->bulk + (size_t)q * kTreeHostRow * 8;
        j.host_row = host_row;
        uint32_t* out = cnt[q] <= kTreeHostRow ? host_row : leaves + total * 8;
        if (cnt[q] > kTreeHostRow) {
            total += cnt[q];
            more = true;
        }
        lv.job[q] = VecLeavesJob{j.v, j.stride, j.n, cnt[q], out, blocks, j.from, out == host_row};
        in[q] = out;
        blocks += (uint32_t)div_up(cnt[q], 64);
    }
    lv.seq = more ? 0 : seq;
    lv.groups = blocks;
    int mode = kLeafPlain;
    for (int q = 0; q < njobs; ++q) {
        const LeafGather& from = jobs[q].from;
        if (from.hash_only && mode == kLeafPlain) mode = kLeafRowsHash;
        else if (from.rows && !from.hash_only) mode = from.S ? kLeafRowsCheck : ints ? kLeafRowsInts : kLeafRows;
    }
    if (to_host) {
        if (mode == kLeafRowsHash) return ZK_E_BADARG;  // cannot happen: what the host hashes is made on its way there (hash_plan)
        static_assert(kHostLeaves * kVecLeaf * 32 <= kBulkDigests, "the leaves take the place of the digests");
        uint32_t elements = 0;
        for (int q = 0; q < njobs; ++q) {
            VecDigestJob& j = jobs[q];
            uint8_t* const at = mb->bulk + (size_t)elements * 32;
            lv.job[q].out = (uint32_t*)at;
            lv.job[q].first_group = elements;
            j.shipped = at;
            j.leaf_bytes = j.n / cnt[q] * 32;
            j.host_count = (uint32_t)cnt[q];
            elements += (uint32_t)j.n;
        }
        lv.groups = elements;
        lv.seq = seq;
        if (mode == kLeafRowsCheck) launch_leaves_to_host<kLeafRowsCheck>(lv, stream);
        else if (mode == kLeafRowsInts) launch_leaves_to_host<kLeafRowsInts>(lv, stream);
        else if (mode == kLeafRows) launch_leaves_to_host<kLeafRows>(lv, stream);
        else launch_leaves_to_host<kLeafPlain>(lv, stream);
        ZK_HIP_TRY(hipGetLastError());
        return ZK_OK;
    }
    if (mode == kLeafRowsCheck || mode == kLeafRowsInts) return ZK_E_BADARG;  // cannot happen: k_make_a or the rounds compare (hash_plan)
    if (mode == kLeafRows) launch_leaves<kLeafRows>(lv, stream);
    else if (mode == kLeafRowsHash) launch_leaves<kLeafRowsHash>(lv, stream);
    else if (beside) {
        LeavesBesideArgs args;
        memset(&args, 0, sizeof args);
        args.leaves = lv;
        args.counts = beside->counts;
        args.count_blocks = (uint32_t)div_up(beside->counts.nleaves, 128);
        args.stage = *beside->stage;
        if (lv.seq || args.stage.seq) return ZK_E_BADARG;  // cannot happen: neither is the last
        hipLaunchKernelGGL(k_leaves_beside, dim3((lv.groups + 1) / 2 + args.count_blocks + beside->stage_blocks), dim3(kBlock), 0, stream, args);
        beside->launched = true;
    } else launch_leaves<kLeafPlain>(lv, stream);
    // up the trees, all rows in one launch, a factor of up to kTreeChunk per launch
    while (more) {
        DigestTreeArgs tr;
        memset(&tr, 0, sizeof tr);
        tr.words = mb->words;
        tr.ticket = ticket;
        tr.bad = bad;
        blocks = 0;
        more = false;
        for (int q = 0; q < njobs; ++q) {
            if (cnt[q] <= kTreeHostRow) continue;
            uint32_t chunk = 4;
            while (chunk < kTreeChunk && cnt[q] / chunk > kTreeHostRow) chunk *= 4;
            cnt[q] /= chunk;
            uint32_t* out = cnt[q] <= kTreeHostRow ? const_cast<uint32_t*>(jobs[q].host_row) : rows[q];
            tr.job[tr.njobs++] = DigestTreeJob{in[q], out, chunk, blocks, out == jobs[q].host_row};
            in[q] = out;
            blocks += (uint32_t)cnt[q];
            if (cnt[q] > kTreeHostRow) {
                rows[q] += cnt[q] * 8;
                more = true;
            }
        }
        tr.seq = more ? 0 : seq;
        hipLaunchKernelGGL(k_digest_tree, dim3(blocks), dim3(kBlock), 0, stream, tr);
    }
    for (int q = 0; q < njobs; ++q) jobs[q].host_count = (uint32_t)cnt[q];
    ZK_HIP_TRY(hipGetLastError());
    return ZK_OK;
}

// The rest of a tree, from the row the device has handed over: consecutive fours
// (a last pair in twos) down to one digest.  Leaves' bytes are the caller's witness: they do
// not stay in memory that outlives the call (1 us for 32 leaves).
static void vec_digest_finish(uint8_t out[32], const VecDigestJob& job) {
    uint8_t row[kTreeHostRow * 32];
    uint32_t cnt = job.host_count;
    if (job.shipped) {
        host::Sha256::hash_each(row, job.shipped, job.leaf_bytes, cnt);
        memset(job.shipped, 0, job.leaf_bytes * cnt);
    }
    for (uint32_t i = 0; i < cnt * 8 && !job.shipped; ++i) {
        const uint32_t v = __builtin_bswap32(job.host_row[i]);  // hash-state words: big-endian words of the digest's bytes
        memcpy(row + 4 * i, &v, 4);
    }
    while (cnt >= 4) {
        cnt /= 4;
        host::Sha256::hash_fours(row, row, cnt);
    }
    if (cnt == 2) {
        host::Sha256 h;
        h.update(row, 64);
        h.finish(row);
    }
    memcpy(out, row, 32);
}

static uint32_t hash_capacity(size_t N) {
    size_t cap = 64;
    while (cap < 2 * N) cap <<= 1;
    return (uint32_t)cap;
}

// Whether A is read off B by row (LeafGather) without being asked to: always with the tables whose rows stay in the L2.
static bool gather_by_default(size_t N) { return N <= kLdsHistMaxRows; }

static int carve_prove(ProveWs& w, Carver& cv, size_t D, size_t N) {
    w.A = cv.limbs(D);
    w.Sf = cv.limbs(D / 2 ? D / 2 : 1);
    w.A29 = (uint4*)cv.take((D / 2 ? D / 2 : 1) * 36);
    w.S29 = (uint4*)cv.take((D / 2 ? D / 2 : 1) * 36);
    w.Bf = cv.limbs(N / 2 ? N / 2 : 1);
    w.Tf = cv.limbs(N / 2 ? N / 2 : 1);
    // B's rows are read by what makes and hashes A only, before anything is folded: they lie where the folded arrays will be (Sf to
    // Tf, one after the other: 52 D + 32 N bytes, and N <= D)
    w.rows_b = (uint4*)w.Sf;
    w.B = cv.limbs(N);
    w.M = cv.limbs(N);
    w.m = (uint32_t*)cv.take(N * 4);
    uint32_t cap = hash_capacity(N);
    w.cap_mask = cap - 1;
    w.slots = (uint32_t*)cv.take((size_t)cap * 4);
    w.canon = (uint32_t*)cv.take(N * 4);
    w.rows = (uint4*)cv.take(N * 32);
    w.found = gather_by_default(N) ? (uint32_t*)cv.take(D * 4) : nullptr;
    w.hist_parts = N <= kLdsHistMaxRows ? kHistParts : 0;
    w.hist = w.hist_parts ? (uint32_t*)cv.take((size_t)w.hist_parts * N * 4) : nullptr;
    w.flags = (uint32_t*)cv.take(64);
    w.fold4 = (SmallFold4*)cv.take(sizeof(SmallFold4));
    w.nleaves = (uint32_t)div_up(N, kLeafCounts);
    w.dig_rows = (uint32_t*)cv.take(vec_digest_row_digests(D) * 32);
    w.dig_rows_b = (uint32_t*)cv.take(vec_digest_row_digests(N) * 32);
    w.part_blocks = round_blocks_max(D);
    w.partD = cv.limbs(w.part_blocks * 5);
    w.partT = cv.limbs(w.part_blocks * 6);
    return ZK_OK;
}

// Leaf digests of the hash trees over the K instances' A and B.
static size_t dig_leaves_bytes(const size_t* D, const size_t* N, size_t K) {
    size_t total = 0;
    for (size_t i = 0; i < K; ++i) total += vec_digest_leaves(D[i]) + vec_digest_leaves(N[i]);
    return total * 32;
}

// K instances: their buffers, one pool of weight tables per distinct length of
// the tensors, and the scratch of the 2K inversions that are in flight together.
// The order here is the order prove_core carves in.
static size_t prove_ws_bytes_shapes(const size_t* D, const size_t* N, size_t K) {
    Carver cv(nullptr, 0);
    for (size_t i = 0; i < K; ++i) {
        ProveWs w;
        carve_prove(w, cv, D[i], N[i]);
    }
    cv.take(dig_leaves_bytes(D, N, K));
    for (size_t i = 0; i < K; ++i) {
        bool seen = false;
        for (size_t j = 0; j < i; ++j) seen = seen || D[j] == D[i];
        if (seen) continue;
        cv.limbs(EqPool::entries(log2_floor(D[i])));
        cv.take(EqPool::entries29(log2_floor(D[i])) * 36);
    }
    for (size_t i = 0; i < K; ++i) {
        if (gather_by_default(N[i])) {
            cv.take(batch_inverse_scratch_bytes(N[i]));
            continue;
        }
        size_t apart = batch_inverse_scratch_bytes(D[i]) + batch_inverse_scratch_bytes(N[i]),
               joined = batch_inverse_scratch_bytes(D[i] + N[i]);
        cv.take(apart > joined ? apart : joined);
    }
    return cv.used();
}

static size_t prove_ws_bytes(size_t D, size_t N, size_t K = 1) {
    size_t Ds[kMailboxMaxInstances], Ns[kMailboxMaxInstances];
    if (K > kMailboxMaxInstances) K = kMailboxMaxInstances;
    for (size_t i = 0; i < K; ++i) {
        Ds[i] = D;
        Ns[i] = N;
    }
    return prove_ws_bytes_shapes(Ds, Ns, K);
}

// What counting hands to the host: the four flag words, then the digests of m's leaves or (host_counts) the counts, for
// which there is then room beside that of digests.  A call's, of tables no longer than those zkmi_thread_init was told of,
// fits what that has reserved.
static size_t counted_bytes(const ProveWs& w, size_t N, bool to_host) {
    return 16 + std::max((size_t)w.nleaves * 32, to_host ? align_up(N * 4, 16) : 0);
}
static_assert(kHostCountLeaves * kLeafCounts * 4 == kBulkCounts, "");
// Smallest i with S_i not in T (all ones: none), once that has arrived.
static uint64_t counted_bad(const uint8_t* staged) {
    uint64_t bad;
    memcpy(&bad, staged + 8, 8);
    return bad;
}

// Whether the comparison of S with hinted rows can be left to the caller (workgroup histograms in use).
static bool can_defer_check(size_t D, size_t N, bool hints) { return N <= kLdsHistMaxRows && hints && D > (size_t)kBlock; }

// One tensor's counting.
struct CountJob {
    ProveWs* w;
    fr_vec S;
    const uint32_t* idx;
    fr_vec T;
    size_t D, N;
    uint8_t* staged;   // pinned, counted_bytes: receives the flags and the digests of m's leaves or the counts
    bool defer_check;  // the hints are taken as they are; S_i = T[idx_i] is then checked by the caller
    uint32_t* found;   // without hints the rows are left here, if the caller wants them
};

static TableJob table_job(const ProveWs& w, const fr_vec& T, size_t N) {
    return TableJob{T.limbs, T.stride, (uint32_t)N, w.slots, w.cap_mask, w.flags, w.canon, w.rows, w.m, w.hist, w.hist_parts, w.M, w.B, nullptr, nullptr, nullptr};
}

// Whether the host hashes a call's leaves of m: they are few, the counts come from workgroups' histograms.  Decided once:
// what counting stages, how it is read and whether it is cleared go by the same value.
static bool host_counts(const size_t* N, size_t K, bool sha_instructions) {
    size_t leaves = 0;
    for (size_t i = 0; i < K; ++i) {
        if (N[i] > kLdsHistMaxRows) return false;
        leaves += div_up(N[i], kLeafCounts);
    }
    return leaves <= kHostCountLeaves && sha_instructions;
}

// Enqueues the multiplicities of up to kMaxTables tensors into their w.m; `seq` (not zero)
// is published once all that they stage is there.  to_host: host_counts' answer, for all of the call's tables.
template <int NT>
static int count_rows_of(const CountJob* jobs, int njobs, bool to_host, uint32_t seq, Mailbox* mb, hipStream_t stream, bool counts_as_fr) {
    CountsOutArgs<NT> out{};
    TableJobs<NT>& tables = out.tables;
    LeafDigestArgs<NT> lf{};
    size_t most = 0;
    uint32_t most_leaves = 0, most_parts = 0;
    for (int q = 0; q < njobs; ++q) {
        const CountJob& j = jobs[q];
        if (j.defer_check && !can_defer_check(j.D, j.N, j.idx != nullptr)) return ZK_E_BADARG;
        tables.job[q] = table_job(*j.w, j.T, j.N);
        out.out[q] = (uint32_t*)j.staged;
        lf.job[q] = LeafDigestJob{(uint32_t*)(j.staged + 16), j.w->m, (uint32_t)j.N, j.w->nleaves, j.w->flags, (uint32_t*)j.staged};
        most = std::max(most, j.N);
        most_leaves = std::max(most_leaves, j.w->nleaves);
        most_parts = std::max(most_parts, j.w->hist_parts);
    }
    const unsigned ny = (unsigned)njobs;
    if (most <= kSmallTable) {
        hipLaunchKernelGGL(k_table_small<NT>, dim3(1, ny), dim3(1024), 0, stream, tables);
    } else {
        hipLaunchKernelGGL(k_count_init<NT>, dim3(grid_for(hash_capacity(most) + most + 4), ny), dim3(kBlock), 0, stream, tables);
        hipLaunchKernelGGL(k_hash_build<NT>, dim3(grid_for(most), ny), dim3(kBlock), 0, stream, tables);
        hipLaunchKernelGGL(k_canon_rows<NT>, dim3(grid_for(most), ny), dim3(kBlock), 0, stream, tables);
    }
    for (int q = 0; q < njobs; ++q) {
        const CountJob& j = jobs[q];
        const ProveWs& w = *j.w;
        const uint32_t* idx = j.idx;
        if (!w.hist) {
            hipLaunchKernelGGL(k_count, dim3(grid_for(j.D, kBlock, 8192)), dim3(kBlock), 0, stream, w.m, j.S.limbs, j.S.stride, j.D,
                               idx, j.T.limbs, j.T.stride, w.rows, (uint32_t)j.N, w.slots, w.cap_mask, w.canon, w.flags,
                               (unsigned long long*)(w.flags + 2));
            continue;
        }
        // LDS histograms: every workgroup takes a contiguous share of S
        static thread_local bool lds_limit_raised = false;
        const size_t lds_bytes = ((j.N + 1) / 2) * 4;
        if (!lds_limit_raised) {
            ZK_HIP_TRY(hipFuncSetAttribute((const void*)k_count_lds<true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)(((kLdsHistMaxRows + 1) / 2) * 4)));
            ZK_HIP_TRY(hipFuncSetAttribute((const void*)k_count_lds<false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)(((kLdsHistMaxRows + 1) / 2) * 4)));
            lds_limit_raised = true;
        }
        // equal chunks, as few passes per workgroup as the 16-bit counters allow
        const size_t passes = div_up(div_up(j.D, w.hist_parts), (size_t)kHistPass);
        const size_t per_block = align_up(div_up(j.D, w.hist_parts * passes), kHistThreads);
        const bool find = !idx && j.found;
        if (find) {
            hipLaunchKernelGGL(k_find_rows, dim3((unsigned)div_up(j.D, kBlock)), dim3(kBlock), 0, stream, j.found, j.S.limbs, j.S.stride, j.D,
                               w.rows, (uint32_t)j.N, w.slots, w.cap_mask, (unsigned long long*)(w.flags + 2));
            idx = j.found;
        }
        if (j.defer_check || find)
            hipLaunchKernelGGL(k_count_lds<false>, dim3(w.hist_parts), dim3(kHistThreads), lds_bytes, stream, w.m, w.hist,
                               j.S.limbs, j.S.stride, j.D, per_block, idx, j.T.limbs, j.T.stride, w.rows, (uint32_t)j.N, w.slots,
                               w.cap_mask, w.canon, w.flags, (unsigned long long*)(w.flags + 2));
        else
            hipLaunchKernelGGL(k_count_lds<true>, dim3(w.hist_parts), dim3(kHistThreads), lds_bytes, stream, w.m, w.hist,
                               j.S.limbs, j.S.stride, j.D, per_block, idx, j.T.limbs, j.T.stride, w.rows, (uint32_t)j.N, w.slots,
                               w.cap_mask, w.canon, w.flags, (unsigned long long*)(w.flags + 2));
    }
    if (to_host) {
        out.words = mb->words;
        out.ticket = jobs[0].w->flags + 1;
        out.seq = seq;
        hipLaunchKernelGGL(k_counts_out<NT>, dim3((unsigned)div_up(most, 64), ny), dim3(1024), 0, stream, out);
        ZK_HIP_TRY(hipGetLastError());
        return ZK_OK;
    }
    if (most_parts) {
        const uint32_t group = 16;
        size_t rows = 0;  // of the tables that have histograms
        for (int q = 0; q < njobs; ++q)
            if (jobs[q].w->hist) rows = std::max(rows, jobs[q].N);
        hipLaunchKernelGGL(k_hist_reduce<NT>, dim3((unsigned)div_up(rows, kBlock), (unsigned)div_up(most_parts, group), ny), dim3(kBlock), 0,
                           stream, tables, group);
    }
    lf.words = mb->words;
    lf.ticket = jobs[0].w->flags + 1;
    lf.seq = seq;
    hipLaunchKernelGGL(k_leaf_digests<NT>, dim3((unsigned)div_up(most_leaves, 64), ny), dim3(128), 0, stream, lf);
    // the counts as field elements (w.M), while the host is busy with the digest
    if (counts_as_fr) hipLaunchKernelGGL(k_counts_to_fr<NT>, dim3(grid_for(most), ny), dim3(kBlock), 0, stream, tables);
    ZK_HIP_TRY(hipGetLastError());
    return ZK_OK;
}
static int count_rows(const CountJob* jobs, int njobs, bool to_host, uint32_t seq, Mailbox* mb, hipStream_t stream,
                      bool counts_as_fr = false) {
    return njobs == 1 ? count_rows_of<1>(jobs, 1, to_host, seq, mb, stream, counts_as_fr)
                      : count_rows_of<kMaxTables>(jobs, njobs, to_host, seq, mb, stream, counts_as_fr);
}

static void digest_of_leaves(uint8_t out[32], const uint8_t* leaves, uint32_t nleaves) {
    host::Sha256 h;
    h.update(leaves, (size_t)nleaves * 32);
    h.finish(out);
}

// Counts are the caller's witness: they do not stay in memory that outlives the call.
static void forget_counts(const CountJob* jobs, int njobs, bool to_host) {
    if (!to_host) return;
    for (int q = 0; q < njobs; ++q) memset(jobs[q].staged + 16, 0, jobs[q].N * 4);
}

// The digest of m from what counting has staged.
static void digest_of_counts(uint8_t out[32], const CountJob& j, bool to_host) {
    if (!to_host) {
        digest_of_leaves(out, j.staged + 16, j.w->nleaves);
        return;
    }
    uint8_t leaves[kHostCountLeaves * 32];
    host::Sha256::hash_each(leaves, j.staged + 16, std::min(j.N, (size_t)kLeafCounts) * 4, j.w->nleaves);
    digest_of_leaves(out, leaves, j.w->nleaves);
}

static const size_t kHostPairs = kMailboxShipEntries / 2;

struct HostTail {
    host::F A[kMailboxShipEntries], S[kMailboxShipEntries], B[kMailboxShipEntries], M[kMailboxShipEntries],
        T[kMailboxShipEntries];
    host::F W[kHostPairs];  // this round's weights e~(u_rest, p), p < half

    // e~((u_0 .. u_{m-1}), p) for p < 2^m, u_0 belonging to the top bit of p
    void weights(const host::F* u, int m) {
        using namespace host;
        W[0] = one();
        for (int t = 0; t < m; ++t) {
            for (size_t e = (size_t)1 << t; e-- > 0;) {
                const F hi = mul(W[e], u[t]);
                W[2 * e] = sub(W[e], hi);
                W[2 * e + 1] = hi;
            }
        }
    }
    // the round's eleven sums in the order the kernels report them: q0, q1, qinf, sA0, sA1, then the table side's
    // t0, t1, tinf, m0, m1, minf (zero unless a table variable is being bound)
    void sums(size_t half, bool table_round, const host::F& beta, host::F out[11]) const {
        using namespace host;
        for (int q = 0; q < 11; ++q) out[q] = zero();
        for (size_t p = 0; p < half; ++p) {
            const F wa0 = mul(W[p], A[p]), wa1 = mul(W[p], A[p + half]);
            out[0] = add(out[0], mul(wa0, add(S[p], beta)));
            out[1] = add(out[1], mul(wa1, add(S[p + half], beta)));
            out[2] = add(out[2], mul(sub(wa1, wa0), sub(S[p + half], S[p])));
            out[3] = add(out[3], A[p]);
            out[4] = add(out[4], A[p + half]);
            if (!table_round) continue;
            const F wb0 = mul(W[p], B[p]), wb1 = mul(W[p], B[p + half]);
            out[5] = add(out[5], mul(wb0, add(T[p], beta)));
            out[6] = add(out[6], mul(wb1, add(T[p + half], beta)));
            out[7] = add(out[7], mul(sub(wb1, wb0), sub(T[p + half], T[p])));
            out[8] = add(out[8], mul(B[p], M[p]));
            out[9] = add(out[9], mul(B[p + half], M[p + half]));
            out[10] = add(out[10], mul(sub(B[p + half], B[p]), sub(M[p + half], M[p])));
        }
    }
    // binds the round's variable to r and moves the weights on to the next round
    void fold(size_t half, bool table_round, const host::F& r) {
        using namespace host;
        auto bind = [&](F* x) {
            for (size_t p = 0; p < half; ++p) x[p] = add(x[p], mul(r, sub(x[p + half], x[p])));
        };
        bind(A);
        bind(S);
        if (table_round) {
            bind(B);
            bind(M);
            bind(T);
        }
        for (size_t p = 0; p < half / 2; ++p) W[p] = add(W[p], W[p + half / 2]);  // the next variable summed out
    }
};

// Positions per workgroup of a long pass (k_round_pair): as many as its weights' shared factor and its sums allow, but
// at least 512 workgroups, two per compute unit, while a batch of 64 is left for each.
static size_t pair_span(size_t P) {
    size_t span = P / 512;
    if (span < (size_t)kOuterBatch) span = (size_t)kOuterBatch;
    return span < kOuterMaxSpan ? span : kOuterMaxSpan;
}

// ---- prover --------------------------------------------------------------------------------------
//
// One routine proves K instances with a single sumcheck over
//   f = sum_i lambda^i f_i,   claim_0 = (sum_i lambda^i)(alpha + alpha^2),
// f_i the tlookup summand of instance i; beta, alpha, u and the round challenges
// are shared.  tlookup_prove is K = 1 without lambda and with its own transcript
// label and proof header.  Per instance the device work is exactly that of a
// single proof: every round launches the instance's kernels one after the other
// on the stream, each instance's sums land in its own part of the mailbox, only
// the last launch of a round publishes, and the host adds the instances' round
// polynomials weighted by lambda^i.
//
// Shapes may differ (tlookup_prove_multi).  The sumcheck then has n = max_i n_i
// variables, instance i lives on the last n_i of them (skip_i = n - n_i) and
//   f = sum_i lambda^i 2^-skip_i f_i(x_[skip_i:]),  f_i built with u_[skip_i:]:
// in a round k < skip_i the instance is a constant, (alpha + alpha^2) 2^(skip_i-k-1)
// before its weight, which the host adds without any device work; from round
// skip_i on it runs the rounds of a proof of its own ("local round" k - skip_i)
// with the shared challenges, and all instances reach their last round together.

// ---- what runs a round, and where it finds the arrays ---------------------------------
//
// Decided in one place, by a function of the shape and of what the rounds before have
// left behind, both plain numbers, so that the prover's schedule can be walked on the
// host without a GPU (zkmi_selftest_tlookup_plan) and checked against the pointers
// actually handed to a kernel before it is launched.
enum RoundKind {
    kRoundFirst = 0,     // k_round_data0: the first round, nothing to fold
    kRound29 = 1,        // k_round_data29: large folding rounds on 29-bit limbs (where the rounds do not go by row)
    kRoundBoth = 2,      // k_round_both: data and table side, the table's variables being bound
    kRoundFirstTwo = 5,  // k_round_first_two or, by row, k_first_two_rows: yields the sums of the first two rounds
    kRoundNoPass = 6,    // the second round after kRoundFirstTwo: the host has everything, nothing is launched
    kRoundHost = 7,      // the host's (HostTail); the first of them fetches the arrays
    kRoundGrid = 8,      // its sums come from the grid of a pass over several variables; the first of them runs the pass
    kRoundPair = 9       // the first round of a long pass over two variables (tlookup_rows.h); a second one is a kRoundGrid
};
enum SSource {
    kSFromCaller = 0,  // the caller's vector of field elements
    kSFromInts = 1,    // the caller's integer columns (tlookup_prove_small)
    kSFromWords = 2,   // the folded copy in the workspace, 32-bit words
    kSFromPlanes = 3,  // the folded copy in the workspace, planes of 29-bit limbs (kRound29) or of digits (kRoundPair)
    kSUnread = 4,      // the round reads no array
    kSFromRows = 5,    // the rows of the table (tlookup_rows.h)
    kSNowhere = -1     // a plan this library has no kernel for: never launched
};

// What the rounds of one instance so far have left behind.
struct RoundState {
    int lazy = 0;                           // folds since the data arrays were last fully reduced, if they are in 29-bit planes
    int pending = 0, pending_t = 0;         // last challenges that the arrays (the table's) have yet to be bound to
    bool s_moved = false, t_moved = false;  // S is in the workspace, T is (bound at least once)
    bool first_two = false;                 // the round before was kRoundFirstTwo
    int pass_left = 0;                      // rounds of the running pass that are still to come
    bool on_host = false;
};

struct RoundPlan {
    int kind;
    int s_source;
    bool table_round;  // the variable being bound is one of the table's
    bool in32, out32;  // kRound29: the data arrays arrive as / leave as 32-bit words (kRoundPair: leave)
    bool fold2;        // kRound29: binds the two previous variables at once (after kRoundFirstTwo, kRoundNoPass)
    // kRoundGrid, kRoundPair, kRoundHost
    bool starts;              // the pass, or the hand-over, is this round's
    int vars, tvars;          // variables (of the table) the pass serves, when it starts
    int left;                 // rounds of the pass from this one on
    int bind, bind_t;         // challenges the arrays (the table's) are bound to before it, when it starts
    bool s_moved, t_moved;    // where it finds S and T: the workspace or the caller's vectors
};

// The last rounds on the host.  A pass costs a trip to the host and back (some forty microseconds) whatever it
// computes; a round of 32 pairs is some six hundred multiplications, which the host does in a fraction of that.  So
// once few variables are left (host_vars), the device binds the last challenges, writes the five arrays (at most 64
// elements each) into the mailbox, and the host computes the remaining rounds' sums, folds and final claims from them:
// the same sums over the same arrays (Section 3.3's sumcheck, Section 4's summand), exact arithmetic, so the same bytes.
// Variables left to the host: six of a single proof (63 pairs of some 19 multiplications, 24 us), three of each of
// several (7 pairs each, and one more pass for all of them together).
static int host_vars(size_t K) { return K == 1 ? 6 : 3; }
// Passes serve the rounds of the last kPassVars variables.  At 2^16 entries three rounds by themselves take 140 us, most
// of it trips, and a pass over them 60; the rounds of longer arrays are what the 29-bit kernel is for.
static const int kPassVars = 16;
// The variables of a pass that starts with `left` of them unbound: up to the next of the places at which all passes
// of a call end (whatever the instances' lengths: they share the trips).  Zero: not in a pass.
static int plan_pass(int left, size_t K) {
    const int host = host_vars(K);
    if (left > kPassVars || left <= host) return 0;
    return (left - host - 1) % kGridVars + 1;
}

static const size_t kSmallPairs = 256;  // the 29-bit kernel's rounds have more pairs than this
static bool round_on_29_bits(int n, int h, int k) {
    return k >= 1 && k < h && ((size_t)1 << (n - k - 1)) > kSmallPairs;
}

// Whether the first pass over the data serves the first two rounds (k_round_first_two)
// and both variables are bound at once afterwards: the three rounds must all bind data
// variables only, and be long.
static bool first_two_rounds_share_a_pass(int n, int h, bool from_ints) {
    return !from_ints && h >= 3 && round_on_29_bits(n, h, 2);
}

// Whether the long rounds read the table's rows (tlookup_rows.h): the first pass serves two rounds and a pass over two
// variables follows, which needs three variables beyond those the last passes serve.  (With one or two, 2^17 and 2^18
// entries, the first of the last passes binds the first two variables, from vectors.)  Tables of up to 2^16 rows: the
// caches hold their rows, and all their variables are among the last ones.
static bool rounds_by_row(int n, int h) {
    return first_two_rounds_share_a_pass(n, h, false) && n - 2 > kPassVars && n - h <= kPassVars;
}

// What a pass, or the hand-over to the host, finds and leaves.
static void plan_bound(RoundPlan& pl, RoundState& st, int vars, int tvars) {
    pl.starts = true;
    pl.vars = vars;
    pl.tvars = tvars;
    pl.bind = st.pending;
    pl.bind_t = st.pending_t;
    pl.s_moved = st.s_moved;
    pl.t_moved = st.t_moved;
    pl.s_source = st.s_moved ? kSFromWords : kSFromCaller;
    if (st.pending) st.s_moved = true;
    if (st.pending_t) st.t_moved = true;
    st.pending = vars;
    st.pending_t = tvars;
}

// Round k of an instance of n variables, the last n - h of them the table's, in a call of K instances; moves the state on.
static RoundPlan plan_round(int n, int h, int k, size_t K, bool from_ints, RoundState& st) {
    RoundPlan pl{};
    const bool by_row = rounds_by_row(n, h);  // the entries are rows of the table, whatever the caller's tensor is
    const int left = n - k;
    pl.table_round = k >= h;
    pl.s_source = kSUnread;
    // integers are the first two rounds' business (but by row), and the second of two rounds that share a pass needs none
    const bool own = (from_ints && !by_row && k < 2) || st.first_two;
    if (st.on_host || (!own && left <= host_vars(K))) {
        pl.kind = kRoundHost;
        if (!st.on_host) plan_bound(pl, st, 0, 0);
        st.on_host = true;
        return pl;
    }
    if (st.pass_left > 0 || (!own && plan_pass(left, K) > 0)) {
        pl.kind = kRoundGrid;
        if (st.pass_left == 0) {
            const int vars = plan_pass(left, K), after = left - vars;
            plan_bound(pl, st, vars, std::max(0, std::min(vars, n - h - after)));
            st.pass_left = vars;
        }
        pl.left = st.pass_left--;
        return pl;
    }
    if (st.first_two) {
        pl.kind = kRoundNoPass;
        st.first_two = false;
        return pl;
    }
    if (by_row && k > 0) {
        // two variables, of which the second may be one of the last passes' (that many fewer for them) if it is not the
        // table's; one where it is
        plan_bound(pl, st, std::min(2, h - k), 0);
        pl.kind = kRoundPair;
        pl.s_source = k == 2 ? kSFromRows : kSFromPlanes;
        pl.out32 = left - pl.vars <= kPassVars;
        st.pass_left = pl.vars;
        pl.left = st.pass_left--;
        return pl;
    }
    pl.in32 = st.lazy == 0;
    int lazy_after = 0;
    if (k == 0) {
        st.first_two = by_row || first_two_rounds_share_a_pass(n, h, from_ints);
        pl.kind = st.first_two ? kRoundFirstTwo : kRoundFirst;
        pl.s_source = by_row ? kSFromRows : from_ints ? kSFromInts : kSFromCaller;
    } else if (pl.table_round) {
        pl.kind = kRoundBoth;
        pl.s_source = k > 1 ? kSFromWords : from_ints ? kSNowhere : kSFromCaller;
    } else if (round_on_29_bits(n, h, k)) {
        pl.kind = kRound29;
        pl.fold2 = st.pending == 2;
        // words for whatever is not a 29-bit round, and when the lazily reduced sums have grown enough
        lazy_after = st.lazy + (pl.fold2 ? 2 : 1);
        pl.out32 = !round_on_29_bits(n, h, k + 1) || plan_pass(left - 1, K) > 0 || lazy_after == kMaxLazyRounds;
        if (pl.out32) lazy_after = 0;
        pl.s_source = !pl.in32 ? kSFromPlanes : st.s_moved ? kSFromWords : from_ints ? kSFromInts : kSFromCaller;
    } else {
        pl.kind = kRoundFirst;
        pl.s_source = kSNowhere;  // a short round in the middle: never of the shapes that are accepted
    }
    st.lazy = lazy_after;
    st.pending = pl.kind == kRoundFirstTwo ? 2 : 1;
    st.pending_t = pl.table_round ? 1 : 0;
    st.s_moved = k >= 1;
    st.t_moved = k > h;
    return pl;
}

struct Instance {
    ProveWs w;
    fr_vec S, T;
    size_t D = 0, N = 0;             // its shape: n = log2 D, l = log2 N, h = n - l;
    int n = 0, l = 0, h = 0, skip = 0;  // skip: the rounds of the whole proof before its own first
    const EqPool* ep = nullptr;      // weight tables for u_[skip:]
    host::F cD, cT;                  // products of e~(u_t, r_t) over its bound variables (all / the table's)
    host::F half_pow;                // 2^-(local round + 1)
    host::F scale;                   // 2^-h
    host::F inv_den;                 // what the one-sided round's other side is divided by (this round)
    host::F pass01[9];               // kRoundFirstTwo's sums: c20, c21, qd, T, qe, then the sums of A_00, A_01, A_10, A_11
    const uint32_t* idx = nullptr;
    uint32_t* b_cur = nullptr;  // where B lives at the moment (it ping-pongs while folding)
    size_t b_cur_stride = 0;
    uint32_t* words = nullptr;  // this instance's round sums in the mailbox
    uint32_t* inv_words = nullptr;    // totals of its two inversions (B, then A)
    host::F sum_mB, cB, sum_A, lam;
    host::F claim;       // the running claim of this instance's own sumcheck: f_i's round polynomial at 0 plus at 1
    host::F fX[4];       // its last round polynomial at X = 0..3
    host::F sA_prev[2];  // its last round's sums of A at X = 0, 1
    uint8_t md[32], dA[32], dB[32];
    BatchInverseJob job_a, job_b;
    // the last rounds (passes over several variables, then the host's)
    HostGrid gq, gt, gm;         // the data side's products, the table side's
    host::F gs[1 << kGridVars];  // sums of A
    const uint32_t* grid_words = nullptr;  // where the running pass's values come out
    RoundState state;            // what its rounds so far have left behind
    HostTail* tail = nullptr;    // once the host has the arrays
    bool gather = false;    // A is B by row (all but kAInverted)
    bool by_row = false;    // A and S are the table's rows until a challenge has bound them (tlookup_rows.h): kANever
    bool apart = false;     // kAApart
    bool deferred = false;  // S_i = T[idx_i] is checked where A is made (by_row: in the first pass), not while counting
    bool unchecked = false; // that first pass has not run yet

    const uint32_t* rows() const { return idx ? idx : w.found; }
    // Where the rows lie: those of the two passes behind the folded planes of A and S, what the hash of A reads where the
    // words of folded S will be (rounds_by_row: N <= D / 8, so 8 D, 8 D and 4 D bytes at most).
    uint4* rows_first() const { return w.A29 + D / 2; }
    uint4* rows_pair() const { return w.S29 + D / 2; }
    uint4* rows_hash() const { return (uint4*)w.Sf; }
    DigitPlanes planes(uint4* base) const { return DigitPlanes{base, D / 4}; }
};

// Who makes, compares and hashes what of a call: decided once, from its shapes and options, and all launches go by it.
// With hints S_i = T[idx_i] is compared where A is made from the rows; all instances or none, so that the first instance
// at fault is the one reported.
enum AMaker {
    kAInverted = 0,     // the inversion of beta + S
    kAWhileHashed = 1,  // the leaves' hash, or what ships the leaves to the host: writes A, in the latter case compares too
    kAApart = 2,        // k_make_a, which compares; the hash only hashes
    kANever = 3         // rounds by row: hashed from the rows, compared by the first pass
};
struct HashPlan {
    bool leaves_to_host, counts_to_host;
    struct {
        AMaker maker;
        bool deferred;  // compared where A is made (kANever: by the first pass), not while counting
    } of[kMailboxMaxInstances];
};
static HashPlan hash_plan(const size_t* D, const size_t* N, const bool* hints, size_t K, bool check_upfront, bool by_rows,
                          bool sha_instructions) {
    HashPlan p;
    size_t leaves = 0;
    bool defer_all = !check_upfront;
    for (size_t i = 0; i < K; ++i) {
        leaves += vec_digest_leaves(D[i]) + vec_digest_leaves(N[i]);
        defer_all = defer_all && can_defer_check(D[i], N[i], hints[i]);
    }
    p.leaves_to_host = host_leaves(leaves, sha_instructions);
    p.counts_to_host = host_counts(N, K, sha_instructions);
    for (size_t i = 0; i < K; ++i) {
        const int n = log2_floor(D[i]), h = n - log2_floor(N[i]);
        p.of[i].maker = !(by_rows || gather_by_default(N[i])) ? kAInverted
                        : rounds_by_row(n, h)                 ? kANever
                        : p.leaves_to_host || D[i] > kMadeApart ? kAWhileHashed
                                                                : kAApart;
        p.of[i].deferred = defer_all && p.of[i].maker != kAInverted;
    }
    return p;
}

struct ProveCall {
    const uint8_t* seed = nullptr;
    size_t K = 1;
    const fr_vec* S = nullptr;
    const uint32_t* const* idx = nullptr;  // may be null, entries may be null
    const fr_vec* T = nullptr;
    bool batch = false;                    // batched transcript and proof layout
    bool multi = false;                    // batched, and the instances' shapes may differ (S[i].n, T[i].n)
    const fr_t* forced_beta = nullptr;
    bool by_rows = false;                  // A as B[idx_i] whatever the table's length
    bool check_upfront = false;            // compare every S_i with its hinted row while counting (no deferred check)
    // S_0 given as small integers x + rho y (K = 1, hints required, S ignored): see tlookup_prove_small
    const int32_t* ints_x = nullptr;
    const int32_t* ints_y = nullptr;
    const fr_t* ints_rho = nullptr;
    size_t ints_D = 0;
    uint8_t* proof = nullptr;
    size_t cap = 0;
    size_t* len = nullptr;
    tlookup_aux* aux = nullptr;            // single proof
    tlookup_batch_aux* baux = nullptr;     // batched proof
    void* ws = nullptr;
    size_t ws_bytes = 0;
    void* stream = nullptr;
};

// Whether a lookup of this shape can read S as small integers all the way: the
// multiplicities come from the hints alone (workgroup histograms); by row the first pass
// compares integers with the rows, otherwise the first round and the first fold are kernels
// of their own that read integers.
static bool small_source_shape_ok(size_t D, size_t N) {
    if (!is_pow2(D) || !is_pow2(N) || N > D || N > kLdsHistMaxRows || D <= (size_t)kBlock) return false;
    const int n = log2_floor(D), h = n - log2_floor(N);
    if (n < 2) return false;
    if (rounds_by_row(n, h)) return true;
    RoundState st;
    const RoundPlan p0 = plan_round(n, h, 0, 1, true, st);
    const RoundPlan p1 = plan_round(n, h, 1, 1, true, st);
    return p0.s_source == kSFromInts && p1.s_source == kSFromInts;
}

static __global__ void k_store_fold4(SmallFold4 v, SmallFold4* dst) {
    ((uint32_t*)dst)[threadIdx.x] = ((const uint32_t*)&v)[threadIdx.x];  // 64 words
}

static size_t batch_proof_bytes(size_t D, size_t K) {
    return 32 + 96 * K + (size_t)log2_floor(D ? D : 1) * 128 + 160 * K;
}

// "ZKTM" | u32 1 | LE64 K | K x (LE64 D_i, LE64 N_i) | K digests of m | K x [digest(A) digest(B)] | rounds | K x 5 claims
static size_t multi_proof_bytes(int n_max, size_t K) { return 16 + 16 * K + 96 * K + (size_t)n_max * 128 + 160 * K; }

static int prove_core(const ProveCall& c) {
    using namespace host;
    const size_t K = c.K;
    const bool from_ints = c.ints_x != nullptr;
    if (!c.seed || (!c.S && !from_ints) || !c.T || K == 0 || K > kMailboxMaxInstances) return ZK_E_BADARG;
    if (!c.batch && (K != 1 || c.multi)) return ZK_E_BADARG;
    if (from_ints && (K != 1 || c.batch || c.by_rows || !c.idx || !c.idx[0])) return ZK_E_BADARG;
    // shapes: one for all, unless the call says they may differ
    size_t Ds[kMailboxMaxInstances], Ns[kMailboxMaxInstances];
    int n = 0;  // variables of the sumcheck: those of the longest instance
    for (size_t i = 0; i < K; ++i) {
        Ds[i] = from_ints ? c.ints_D : c.S[c.multi ? i : 0].n;
        Ns[i] = c.T[c.multi ? i : 0].n;
        if (!is_pow2(Ds[i]) || !is_pow2(Ns[i]) || Ns[i] > Ds[i] || Ds[i] > ((size_t)1 << 31)) return ZK_E_BADARG;
        if (c.T[i].n != Ns[i] || !vec_ok(c.T[i], Ns[i])) return ZK_E_BADARG;
        if (!from_ints && (c.S[i].n != Ds[i] || !vec_ok(c.S[i], Ds[i]))) return ZK_E_BADARG;
        if (c.by_rows && !(c.idx && c.idx[i])) return ZK_E_BADARG;
        if (log2_floor(Ds[i]) > n) n = log2_floor(Ds[i]);
    }
    if (from_ints && !small_source_shape_ok(Ds[0], Ns[0])) return ZK_E_BADARG;
    if (from_ints && ((c.ints_y != nullptr) != (c.ints_rho != nullptr))) return ZK_E_BADARG;
    if (from_ints && c.ints_rho && !canonical_in_range(*c.ints_rho)) return ZK_E_BADARG;
    // the tensor as small integers, if it came that way
    SmallSource ints_src;
    memset(&ints_src, 0, sizeof ints_src);
    F ints_rho = zero();
    const F two64 = mul(from_u64((uint64_t)1 << 32), from_u64((uint64_t)1 << 32));
    if (from_ints) {
        if (c.ints_rho) ints_rho = from_canonical(*c.ints_rho);
        ints_src.x = c.ints_x;
        ints_src.y = c.ints_y;
        to_device_limbs(ints_src.plus_one, two64);
        to_device_limbs(ints_src.minus_one, neg(two64));
        to_device_limbs(ints_src.plus_rho, mul(ints_rho, two64));
        to_device_limbs(ints_src.minus_rho, neg(mul(ints_rho, two64)));
    }
    if (c.forced_beta && !canonical_in_range(*c.forced_beta)) return ZK_E_BADARG;
    const size_t need = c.multi ? multi_proof_bytes(n, K) : c.batch ? batch_proof_bytes(Ds[0], K) : tlookup_proof_bytes(Ds[0]);
    if (c.len) *c.len = need;
    if (!c.proof || c.cap < need) return ZK_E_BUFSZ;
    if (!c.ws || c.ws_bytes < prove_ws_bytes_shapes(Ds, Ns, K)) return ZK_E_BUFSZ;
    hipStream_t stream = as_stream(c.stream);
    Mailbox* mb;
    ZK_TRY(mailbox_get(&mb));
    Carver cv(c.ws, c.ws_bytes);
    Instance inst[kMailboxMaxInstances];
    const F inv2 = inv(from_u64(2));
    for (size_t i = 0; i < K; ++i) {
        Instance& I = inst[i];
        I.D = Ds[i];
        I.N = Ns[i];
        I.n = log2_floor(I.D);
        I.l = log2_floor(I.N);
        I.h = I.n - I.l;
        I.skip = n - I.n;
        carve_prove(I.w, cv, I.D, I.N);
        I.S = from_ints ? fr_vec{nullptr, I.D, I.D} : c.S[i];  // with integers there is no vector: every reader of I.S.limbs
        I.T = c.T[i];                                           // is gated by the round's plan (s_source)
        I.idx = c.idx ? c.idx[i] : nullptr;
        I.b_cur = I.w.B;
        I.b_cur_stride = I.N;
        I.words = mb->words + kMailboxSlot * i;
        I.inv_words = mb->words + kMailboxInvB + 16 * i;
        I.sum_mB = I.cB = I.sum_A = zero();
        I.cD = I.cT = I.half_pow = one();
        I.inv_den = zero();
        I.scale = one();
        for (int t = 0; t < I.h; ++t) I.scale = mul(I.scale, inv2);
    }
    uint32_t* dig_leaves = (uint32_t*)cv.take(dig_leaves_bytes(Ds, Ns, K));
    if (cv.overflow()) return ZK_E_BUFSZ;

    ProfileScope prof_total(kProfTotal, stream);

    // -- Prep: multiplicities and their digests -------------------------------------------------
    bool hints[kMailboxMaxInstances];
    for (size_t i = 0; i < K; ++i) hints[i] = inst[i].idx != nullptr;
    const HashPlan who = hash_plan(Ds, Ns, hints, K, c.check_upfront, c.by_rows, Sha256::has_instructions());
    for (size_t i = 0; i < K; ++i) {
        Instance& I = inst[i];
        I.gather = who.of[i].maker != kAInverted;
        I.by_row = who.of[i].maker == kANever;
        I.apart = who.of[i].maker == kAApart;
        I.deferred = who.of[i].deferred;
        I.unchecked = I.by_row && I.deferred;
    }
    if (from_ints && !inst[0].deferred) return ZK_E_BADARG;  // counting would read S as a vector
    {
        // all instances' counting, then one wait
        ProfileScope prof(kProfCount, stream);
        size_t total = 0, at[kMailboxMaxInstances];
        for (size_t i = 0; i < K; ++i) {
            at[i] = total;
            total += counted_bytes(inst[i].w, inst[i].N, who.counts_to_host);
        }
        ZK_TRY(mailbox_bulk(mb, total));
        uint8_t* const staged = mb->bulk + kBulkDigests;
        const uint32_t seq = mb->next_seq();
        CountJob counts[kMailboxMaxInstances];
        for (size_t i = 0; i < K; ++i) {
            Instance& I = inst[i];
            counts[i] = CountJob{&I.w, I.S, I.idx, I.T, I.D, I.N, staged + at[i], I.deferred, I.idx ? nullptr : I.w.found};
        }
        const bool to_host = who.counts_to_host;
        ZK_TRY(count_rows(counts, (int)K, to_host, seq, mb, stream, true));
        ZK_TRY(mailbox_wait(mb, seq, stream));
        for (size_t i = 0; i < K; ++i) {
            const uint64_t bad = counted_bad(staged + at[i]);
            if (bad != UINT64_MAX) {
                if (c.aux) c.aux->bad_index = bad;
                if (c.baux) {
                    c.baux->bad_instance = i;
                    c.baux->bad_index = bad;
                }
                forget_counts(counts, (int)K, to_host);
                ZK_HIP_TRY(hipStreamSynchronize(stream));
                return ZK_E_NOT_IN_TABLE;
            }
            digest_of_counts(inst[i].md, counts[i], to_host);
        }
        forget_counts(counts, (int)K, to_host);
    }

    uint64_t dims[1 + 2 * kMailboxMaxInstances];
    int ndims;
    if (c.multi) {
        dims[0] = K;
        for (size_t i = 0; i < K; ++i) {
            dims[1 + 2 * i] = inst[i].D;
            dims[2 + 2 * i] = inst[i].N;
        }
        ndims = 1 + 2 * (int)K;
    } else {
        dims[0] = inst[0].D;
        dims[1] = inst[0].N;
        dims[2] = K;
        ndims = c.batch ? 3 : 2;
    }
    Transcript tr(c.multi ? "zkmi/tlookup-multi/v1" : c.batch ? "zkmi/tlookup-batch/v2" : "zkmi/tlookup/v2", c.seed, dims, ndims);
    for (size_t i = 0; i < K; ++i) tr.absorb("m", inst[i].md, 32);

    unsigned table_shares = 0;  // of the table side's sums, where the host adds them up

    // -- Prove: beta, inverse vectors ---------------------------------------------------------------
    F beta = tr.challenge("beta");
    if (c.forced_beta) beta = from_canonical(*c.forced_beta);
    {
        // all inversions share one wait: the down passes, one round trip, one host
        // inversion (of the product of all grand totals), the up passes.  Usually the
        // table's are the only ones (see LeafGather); a table too long for that is
        // inverted together with its tensor, as one vector, if the tensor's length
        // allows (its small passes then cost nothing of their own).
        ProfileScope prof(kProfInverse, stream);
        Carver inv_cv = cv;
        const uint32_t seq = mb->next_seq();
        const BatchInverseJob* jobs[2 * kMailboxMaxInstances];
        const uint32_t* totals[2 * kMailboxMaxInstances];
        size_t njobs = 0;
        for (size_t i = 0; i < K; ++i) {
            Instance& I = inst[i];
            const size_t D = I.D, N = I.N;
            const bool joined = !I.gather && batch_inverse_can_join(D, N);
            if (!joined) {
                ZK_TRY(batch_inverse_begin(I.job_b, I.w.B, N, I.T.limbs, I.T.stride, N, beta, inv_cv, I.inv_words, stream,
                                           nullptr, 0, nullptr, 0, 0));
                jobs[njobs] = &I.job_b;
                totals[njobs++] = I.inv_words;
            }
            if (!I.gather) {
                ZK_TRY(batch_inverse_begin(I.job_a, I.w.A, D, I.S.limbs, I.S.stride, D, beta, inv_cv, I.inv_words + 8,
                                           stream, joined ? I.w.B : nullptr, N, I.T.limbs, I.T.stride,
                                           joined ? N : 0));
                jobs[njobs] = &I.job_a;
                totals[njobs++] = I.inv_words + 8;
            }
        }
        ZK_TRY(batch_inverse_totals(jobs, (int)njobs, mb->words, seq, inst[0].w.flags + 1, stream));
        ZK_TRY(mailbox_wait(mb, seq, stream));
        // inverse of each total from one inversion of their product
        F tot[2 * kMailboxMaxInstances], pre[2 * kMailboxMaxInstances + 1];
        pre[0] = one();
        for (size_t q = 0; q < njobs; ++q) {
            tot[q] = from_dev(totals[q]);
            if (is_zero(tot[q])) {
                ZK_HIP_TRY(hipStreamSynchronize(stream));
                return ZK_E_ZERO_DENOM;
            }
            pre[q + 1] = mul(pre[q], tot[q]);
        }
        F suffix_inv = inv(pre[njobs]);  // 1 / (tot_0 ... tot_q) while walking down
        for (size_t q = njobs; q-- > 0;) {
            pre[q] = mul(suffix_inv, pre[q]);
            suffix_inv = mul(suffix_inv, tot[q]);
        }
        ZK_TRY(batch_inverse_end(jobs, pre, (int)njobs, stream));
        TableJobs<kMaxTables> tables{};
        size_t rows = 0;
        for (size_t i = 0; i < K; ++i) {
            TableJob& t = tables.job[i] = table_job(inst[i].w, inst[i].T, inst[i].N);
            if (!inst[i].gather) continue;
            rows = std::max(rows, inst[i].N);
            t.rows_b = inst[i].by_row ? inst[i].rows_first() : inst[i].w.rows_b;
            if (inst[i].by_row) {
                t.rows_pair = inst[i].rows_pair();
                t.rows_hash = inst[i].rows_hash();
            }
        }
        if (rows && K == 1) hipLaunchKernelGGL(k_rows_of<1>, dim3(grid_for(rows)), dim3(kBlock), 0, stream, TableJobs<1>{{tables.job[0]}});
        else if (rows) hipLaunchKernelGGL(k_rows_of<kMaxTables>, dim3(grid_for(rows), (unsigned)K), dim3(kBlock), 0, stream, tables);
        ZK_HIP_TRY(hipGetLastError());
    }

    // What the comparisons of S with its rows have found, in the words that came with the last sums: the first instance
    // at fault is the one reported, so that the earlier ones whose first pass is yet to come are looked through now.
    auto report_bad = [&]() -> int {
        auto bad_of = [&](size_t i) {
            uint64_t bad;
            memcpy(&bad, mb->words + kMailboxBad + 2 * i, 8);
            return bad;
        };
        size_t at = 0;
        while (at < K && bad_of(at) == UINT64_MAX) ++at;
        if (at == K) return ZK_OK;
        uint64_t bad = bad_of(at);
        for (size_t i = 0; i < at; ++i) {
            Instance& I = inst[i];
            if (!I.unchecked) continue;
            uint8_t* const staged = mb->bulk + kBulkDigests;  // there was room for all instances' digests of m
            const CountJob job{&I.w, I.S, I.idx, I.T, I.D, I.N, staged, false, nullptr};
            const uint32_t seq = mb->next_seq();
            ZK_TRY(count_rows(&job, 1, false, seq, mb, stream));  // (its digests: their room is there whatever the call staged)
            ZK_TRY(mailbox_wait(mb, seq, stream));
            if (counted_bad(staged) == UINT64_MAX) continue;
            at = i;
            bad = counted_bad(staged);
            break;
        }
        if (c.aux) c.aux->bad_index = bad;
        if (c.baux) {
            c.baux->bad_instance = at;
            c.baux->bad_index = bad;
        }
        ZK_HIP_TRY(hipStreamSynchronize(stream));
        return ZK_E_NOT_IN_TABLE;
    };

    // The prover sends A and B before the sumcheck (Protocol 1, tlookup-Prove): their
    // digests, standing in for the commitments, enter the transcript before alpha
    // and u are drawn.
    {
        ProfileScope prof(kProfDigest, stream);
        const uint32_t seq = mb->next_seq();
        VecDigestJob jobs[2 * kMailboxMaxInstances];
        MakeAJobs<kMailboxMaxInstances> make{};
        size_t made = 0, longest = 0;
        if (from_ints) make.ints = ints_src;
        for (size_t i = 0; i < K; ++i) {
            Instance& I = inst[i];
            LeafGather from, table;
            if (I.gather) {
                from.rows = I.rows();
                from.T = I.w.rows;
                from.B = I.w.rows_b;
                from.N = (uint32_t)I.N;
                from.bad = (unsigned long long*)(I.w.flags + 2);
                if (I.deferred && !I.by_row) {
                    from.S = I.S.limbs;  // null with integers
                    from.ss = I.S.stride;
                }
                if (I.apart) {
                    const int check = !I.deferred ? kLeafRows : from_ints ? kLeafRowsInts : kLeafRowsCheck;
                    make.job[made++] = MakeAJob{I.w.A, I.D, I.D, from, check};
                    longest = std::max(longest, I.D);
                }
                if (I.apart || I.by_row) {
                    from.S = nullptr;
                    from.B = I.by_row ? I.rows_hash() : I.w.rows_b + 2;
                    from.hash_only = I.by_row ? 2 : 4;
                    table = from;  // B's canonical values are there for A's sake
                    table.rows = nullptr;
                }
            }
            jobs[2 * i] = VecDigestJob{I.w.A, I.D, I.D, I.w.dig_rows, from};
            jobs[2 * i + 1] = VecDigestJob{I.w.B, I.N, I.N, I.w.dig_rows_b, table};
        }
        if (made == 1) hipLaunchKernelGGL(k_make_a<1>, dim3(grid_for(longest)), dim3(kBlock), 0, stream, MakeAJobs<1>{{make.job[0]}, make.ints});
        else if (made) hipLaunchKernelGGL(k_make_a<kMailboxMaxInstances>, dim3(grid_for(longest), (unsigned)made), dim3(kBlock), 0, stream, make);
        BadWords bad{};
        bad.count = (int)K;
        bad.to = mb->words + kMailboxBad;
        for (size_t i = 0; i < K; ++i) bad.from[i] = (const unsigned long long*)(inst[i].w.flags + 2);
        ZK_TRY(vec_digest_launch(jobs, 2 * (int)K, who.leaves_to_host, dig_leaves, mb, seq, inst[0].w.flags + 1, stream,
                                 from_ints ? &ints_src : nullptr, bad));
        // the table side's sums, in the time the host takes: read with the first round's (shares, the host's to add up,
        // unless there are long tables)
        TableSumJobs sums;
        memset(&sums, 0, sizeof sums);
        size_t rows = 0;
        for (size_t i = 0; i < K; ++i) rows = std::max(rows, inst[i].N);
        const bool long_tables = rows > kLdsHistMaxRows;
        const unsigned shares = grid_for(rows, kBlock, long_tables ? kMaxPartialBlocks / 4 : kMailboxTableShares);
        for (size_t i = 0; i < K; ++i)
            sums.job[i] = TableSumJob{inst[i].w.B, inst[i].w.M, inst[i].N,
                                      long_tables ? inst[0].w.partT + i : mb->words + kMailboxTableSums + i * kMailboxTableShares * 8,
                                      long_tables ? inst[0].w.part_blocks * 6 : 0, (uint32_t)K};
        hipLaunchKernelGGL(k_table_sum, dim3(shares, (unsigned)K), dim3(kBlock), 0, stream, sums);
        if (long_tables)
            launch_final_sum(inst[0].w.partT, inst[0].w.part_blocks * 6, shares, (int)K, mb->words + kMailboxTableC, mb->words, 0,
                             inst[0].w.flags + 1, stream);
        table_shares = long_tables ? 0 : shares;
        ZK_HIP_TRY(hipGetLastError());
        ZK_TRY(mailbox_wait(mb, seq, stream));
        for (size_t i = 0; i < K; ++i) {
            vec_digest_finish(inst[i].dA, jobs[2 * i]);
            vec_digest_finish(inst[i].dB, jobs[2 * i + 1]);
            tr.absorb("A", inst[i].dA, 32);
            tr.absorb("B", inst[i].dB, 32);
        }
        ZK_TRY(report_bad());  // (after the leaves' bytes have been cleared)
    }

    F alpha = tr.challenge("alpha");
    F alpha2 = sqr(alpha);
    F u[32];
    for (int t = 0; t < n; ++t) u[t] = tr.challenge("u");
    F lambda = one();
    if (c.batch) lambda = tr.challenge("lambda");
    // an instance's weight in f: lambda^i, times 2^-skip when it is shorter than the longest
    {
        F lam_pow = one();
        for (size_t i = 0; i < K; ++i) {
            inst[i].lam = lam_pow;
            for (int t = 0; t < inst[i].skip; ++t) inst[i].lam = mul(inst[i].lam, inv2);
            lam_pow = mul(lam_pow, lambda);
        }
    }

    // The table side while none of its variables is bound: alpha^2 sum_j e'_j B_j (T_j + beta) - sum_j m_j B_j, the first
    // sum being one (k_table_sum).  Its shares are there once anything enqueued after them is.
    bool table_sums_read = false;
    auto read_table_sums = [&] {
        for (size_t i = 0; i < K && !table_sums_read; ++i) {
            const uint32_t* at = mb->words + kMailboxTableSums + i * kMailboxTableShares * 8;
            inst[i].sum_mB = table_shares ? zero() : from_dev(mb->words + kMailboxTableC + 8 * i);
            for (unsigned q = 0; q < table_shares; ++q) inst[i].sum_mB = add(inst[i].sum_mB, from_dev(at + 8 * q));
            inst[i].cB = sub(alpha2, inst[i].sum_mB);
        }
        table_sums_read = true;
    };

    // weight tables: instance i uses u_[skip_i:], so instances of one length share a pool
    EqPool pools[kMailboxMaxInstances];
    for (size_t i = 0; i < K; ++i) {
        for (size_t j = 0; j < i && !inst[i].ep; ++j)
            if (inst[j].D == inst[i].D) inst[i].ep = inst[j].ep;
        if (inst[i].ep) continue;
        ZK_TRY(eq_pool_build(pools[i], u + inst[i].skip, inst[i].n, cv, stream));
        inst[i].ep = &pools[i];
    }

    // -- header -----------------------------------------------------------------------------------------
    uint8_t* out = c.proof;
    if (c.multi) {
        memcpy(out, "ZKTM", 4);
        out[4] = 1; out[5] = out[6] = out[7] = 0;
        put_le64(out + 8, K);
        out += 16;
        for (size_t i = 0; i < K; ++i) {
            put_le64(out, inst[i].D);
            put_le64(out + 8, inst[i].N);
            out += 16;
        }
    } else {
        memcpy(out, c.batch ? "ZKTB" : "ZKTL", 4);
        out[4] = 2; out[5] = out[6] = out[7] = 0;
        put_le64(out + 8, inst[0].D);
        put_le64(out + 16, inst[0].N);
        out += 24;
        if (c.batch) {
            put_le64(out, K);
            out += 8;
        }
    }
    for (size_t i = 0; i < K; ++i) {
        memcpy(out, inst[i].md, 32);
        out += 32;
    }
    for (size_t i = 0; i < K; ++i) {
        memcpy(out, inst[i].dA, 32);
        memcpy(out + 32, inst[i].dB, 32);
        out += 64;
    }

    // -- rounds -----------------------------------------------------------------------------------------
    // Below, k counts the rounds of the whole proof and kk = k - skip those of one
    // instance ("local"): an instance's kernels, plan and arrays only ever see kk.
    F r_prev = zero(), r_prev2 = zero();  // the challenges of the last round and of the one before it
    // Rounds that fold the data arrays only and are large run on 29-bit limbs
    // (tlookup_round29.h).  Between two of them the arrays stay in 29-bit planes,
    // unreduced, for at most kMaxLazyRounds rounds in a row.
    const F29 beta29 = f29_unpack(to_dev(beta).l);
    const F inv32 = mul(inv2, mul(sqr(inv2), sqr(inv2)));
    // Where local round kk reads and writes the arrays that change place: S comes from
    // the caller's vector until it has been folded once, T likewise, and B alternates
    // between its two buffers on every fold (it has two readers).  b_cur: where B is
    // before the round; returns where it is afterwards.
    struct Moving {
        PairArray S, B, T;
    };
    auto moving_arrays = [&](int kk, const Instance& I, uint32_t*& b_cur, size_t& b_stride, bool s_unfolded) {
        const ProveWs& w = I.w;
        const size_t D = I.D, N = I.N;
        const int h = I.h;
        Moving m;
        if (s_unfolded) m.S = PairArray{I.S.limbs, I.S.stride, w.Sf, D / 2};
        else m.S = PairArray{w.Sf, D / 2, w.Sf, D / 2};
        if (kk > h) {
            uint32_t* other = b_cur == w.B ? w.Bf : w.B;
            size_t other_stride = b_cur == w.B ? N / 2 : N;
            m.B = PairArray{b_cur, b_stride, other, other_stride};
            b_cur = other;
            b_stride = other_stride;
        } else {
            m.B = PairArray{b_cur, b_stride, b_cur, b_stride};
        }
        if (kk <= h + 1) m.T = PairArray{I.T.limbs, I.T.stride, w.Tf, N / 2};
        else m.T = PairArray{w.Tf, N / 2, w.Tf, N / 2};
        return m;
    };
    // The last rounds: several from one pass, then the host's (grid_dev.h, HostTail).
    std::unique_ptr<HostTail[]> host_tails(new (std::nothrow) HostTail[K]);
    if (!host_tails) return ZK_E_BUFSZ;
    F r_last[3] = {zero(), zero(), zero()};  // the last three challenges, the last one in [2]
    // The arrays of instance I as a pass finds them: the pending variables bound as planned, 2^left elements (of the data
    // arrays; the table's if its variables are being bound).  Adds the folds; ship: into the mailbox.
    struct Bound {
        const uint32_t* p[5];
        size_t stride[5];
    };
    auto bind_pending = [&](GridPass& pass, const Instance& I, const RoundPlan& plan, int left, uint32_t* ship) {
        const ProveWs& w = I.w;
        const bool table_bound = left < I.l;
        const size_t n_data = (size_t)1 << left, n_table = table_bound ? (size_t)1 << left : I.N;
        Bound b;
        const uint32_t* src[5] = {w.A, plan.s_moved ? w.Sf : I.S.limbs, I.b_cur, w.M, plan.t_moved ? w.Tf : I.T.limbs};
        const size_t ss[5] = {I.D, plan.s_moved ? I.D / 2 : I.S.stride, I.b_cur_stride, I.N, plan.t_moved ? I.N / 2 : I.T.stride};
        uint32_t* const dst[5] = {w.A, w.Sf, I.b_cur, w.M, w.Tf};
        const size_t ds[5] = {I.D, I.D / 2, I.b_cur_stride, I.N, I.N / 2};
        for (int q = 0; q < 5; ++q) {
            const int vars = q < 2 ? plan.bind : plan.bind_t;
            const size_t count = q < 2 ? n_data : n_table;
            b.p[q] = vars ? dst[q] : src[q];
            b.stride[q] = vars ? ds[q] : ss[q];
            if (ship) {
                pass.add_fold(src[q], ss[q], ship, 0, count, vars, true);
                ship += 8 * count;
            } else if (vars) {
                pass.add_fold(src[q], ss[q], dst[q], ds[q], count, vars);
            }
        }
        return b;
    };
    // Hands the arrays of the instances whose host rounds start at round k to the host (k = n, instances of one element:
    // their claims are all that is left).
    RoundPlan plans[kMailboxMaxInstances] = {};
    auto ships = [&](size_t i, int k) {
        return k < n ? k >= inst[i].skip && plans[i].kind == kRoundHost && plans[i].starts : !inst[i].tail;
    };
    auto ship_to_host = [&](int k, uint32_t seq) -> int {
        GridPass pass;
        pass.challenges(r_last);
        for (size_t i = 0; i < K; ++i) {
            if (!ships(i, k)) continue;
            bind_pending(pass, inst[i], k < n ? plans[i] : RoundPlan{}, n - k, mb->words + kMailboxShip + i * kMailboxShipWords);
        }
        return pass.launch_folds(mb, seq, inst[0].w.flags + 1, stream);
    };
    auto read_shipped = [&](int k) {
        for (size_t i = 0; i < K; ++i) {
            if (!ships(i, k)) continue;
            Instance& I = inst[i];
            I.tail = &host_tails[i];
            const uint32_t* at = mb->words + kMailboxShip + i * kMailboxShipWords;
            const size_t n_data = (size_t)1 << (n - k), n_table = std::min(I.N, n_data);
            F* const arrays[5] = {I.tail->A, I.tail->S, I.tail->B, I.tail->M, I.tail->T};
            for (int q = 0; q < 5; ++q)
                for (size_t j = 0; j < (q < 2 ? n_data : n_table); ++j, at += 8) arrays[q][j] = from_dev(at);
            if (k < n) I.tail->weights(u + k + 1, n - k - 1);
        }
    };
    for (int k = 0; k < n; ++k) {
        // The 29-bit kernel sums one side of the round only (X = 0, or X = 1 with side1); the other side's two sums
        // follow from what the prover has already sent: sA0 + sA1 is the previous round's sum of A at its challenge,
        // g(0) + g(1) the running claim.  The second needs a division by alpha c e~(u_k, X) of the side that was not
        // summed, so the side is chosen by which of the two is not zero (alternating otherwise, both being equally
        // good); if alpha c itself is zero, q carries no weight in g and is not needed.
        const F e_side[2] = {sub(one(), u[k]), u[k]};
        bool side1 = (k & 1) != 0;
        if (is_zero(e_side[0])) side1 = false;  // u_k = 1: only g(1) can tell q1, so sum the X = 0 side
        if (is_zero(e_side[1])) side1 = true;
        // the last instance that has kernels in this round publishes it; a round in which no instance has any (every
        // active one is in the second round of a pass that served two) is answered by the host alone
        size_t last_launch = K;
        bool any_pass = false, any_ship = false;
        for (size_t i = 0; i < K; ++i) {
            Instance& I = inst[i];
            if (k < I.skip) continue;
            const RoundPlan& plan = plans[i] = plan_round(I.n, I.h, k - I.skip, K, from_ints, I.state);
            // cannot happen: small_source_shape_ok has walked these rounds
            if (plan.s_source == kSNowhere || (from_ints && plan.s_source == kSFromCaller)) return ZK_E_BADARG;
            if (plan.kind == kRoundHost) any_ship = any_ship || plan.starts;
            else if (plan.kind == kRoundGrid) any_pass = any_pass || plan.starts;
            else if (plan.kind != kRoundNoPass) last_launch = i;
        }
        const bool any_launch = last_launch < K || any_pass || any_ship;
        size_t pairs = 0;  // long passes over two variables: their values come out behind those of the short passes
        auto passes = [](const RoundPlan& pl) { return pl.kind == kRoundGrid || pl.kind == kRoundPair; };

        const uint32_t seq = any_launch ? mb->next_seq() : 0;
        for (size_t i = 0; i < K; ++i) {
            Instance& I = inst[i];
            if (k < I.skip || plans[i].kind == kRoundNoPass || plans[i].kind == kRoundGrid || plans[i].kind == kRoundHost) continue;
            ProveWs& w = I.w;
            const size_t D = I.D, N = I.N;
            const int h = I.h, kk = k - I.skip;
            const RoundPlan& plan = plans[i];
            const size_t half = (size_t)1 << (I.n - kk - 1);
            const EqSplit eq = I.ep->round(kk);
            const EqPool& ep = *I.ep;
            const bool table_round = plan.table_round;
            const bool in32 = plan.in32, out32 = plan.out32;
            // pairs per workgroup: a workgroup's pairs must share the high factor of
            // their weights (at most 2^kLoBits pairs, 16 per thread).  As many as that
            // allows, since a thread's closing reduction costs about as much as two
            // pairs, but at least 512 workgroups while the round is large enough;
            // small rounds get one pair per thread
            size_t span = half / 512;
            if (span < (size_t)kBlock) span = (size_t)kBlock;
            if (span > ((size_t)1 << kLoBits)) span = (size_t)1 << kLoBits;
            if (span > half) span = half;
            const unsigned blocks = (unsigned)(half / span);
            if (blocks > w.part_blocks) return ZK_E_BUFSZ;  // cannot happen: see round_blocks_max
            const uint32_t my_seq = i == last_launch && !any_pass && !any_ship ? seq : 0;  // the last launch publishes the round
            uint32_t* b_next = I.b_cur;
            size_t b_next_stride = I.b_cur_stride;
            const Moving mv = moving_arrays(kk, I, b_next, b_next_stride, kk <= 1 || plan.fold2);
            DataRoundArgs d;
            d.A = PairArray{w.A, D, w.A, D};
            d.S = mv.S;
            d.half = half;
            d.block_span = span;
            d.r_prev = to_dev(r_prev);
            d.beta = to_dev(beta);
            d.eq = eq;
            d.partials = w.partD;
            d.pstride = w.part_blocks * 5;
            memset(&d.ints, 0, sizeof d.ints);
            if (plan.s_source == kSFromInts && plan.kind == kRoundFirst) d.ints = ints_src;
            // every kernel below reads S through d.S.src unless the plan says otherwise: no launch with nothing behind it
            if ((plan.s_source == kSFromCaller || plan.s_source == kSFromWords) && !d.S.src) return ZK_E_BADARG;
            if (plan.s_source == kSFromInts && !ints_src.x) return ZK_E_BADARG;
            if (!d.A.src || !d.partials) return ZK_E_BADARG;
            TableRoundArgs t;
            t.B = mv.B;
            t.T = mv.T;
            t.M = PairArray{w.M, N, w.M, N};
            t.half = half;
            t.block_span = span;
            t.r_prev = d.r_prev;
            t.beta = d.beta;
            t.eq = eq;
            t.partials = w.partT;
            t.pstride = w.part_blocks * 6;

            if (plan.kind == kRoundFirstTwo) {
                // one pass for this round and the next: nothing is folded, the weights are the next round's
                const size_t quarter = half / 2;
                const EqSplit eq1 = ep.round(kk + 1);
                size_t span01 = quarter / 512;
                if (span01 < (size_t)kBlock) span01 = (size_t)kBlock;
                if (span01 > (size_t)kBlock * kRound01MaxQuads) span01 = (size_t)kBlock * kRound01MaxQuads;
                if (span01 > quarter) span01 = quarter;
                const unsigned blocks01 = (unsigned)(quarter / span01);
                if (blocks01 > w.part_blocks || span01 > ((size_t)1 << eq1.lbits) || (!I.S.limbs && !I.by_row)) return ZK_E_BADARG;  // cannot happen
                DataRound01Args d01;
                d01.A = w.A;
                d01.as = D;
                d01.S = I.S.limbs;
                d01.ss = I.S.stride;
                d01.quarter = quarter;
                d01.block_span = span01;
                d01.weights = Planes29{ep.pool29, ep.count29};
                d01.lo_off = ep.suffix29_off[eq1.lbits];
                d01.lbits = eq1.lbits;
                d01.has_hi = eq1.has_hi;
                d01.hi_pool = ep.pool;
                d01.hi_stride = ep.stride;
                d01.hi_off = eq1.hi_off;
                d01.partD = w.partD;
                d01.pstrideD = w.part_blocks * 5;
                d01.partT = w.partT;
                d01.pstrideT = w.part_blocks * 6;
                d01.beta = to_dev(beta);
                {
                    ProfileScope prof(kProfRoundData, stream);
                    if (I.by_row) {
                        FirstTwoRowsArgs rows;
                        rows.sums = d01;
                        rows.rows = I.rows();
                        rows.table = I.rows_first();
                        rows.N = (uint32_t)N;
                        rows.bad = (unsigned long long*)(w.flags + 2);
                        rows.ints = ints_src;
                        if (!I.deferred) hipLaunchKernelGGL(k_first_two_rows<kRowsTrusted>, dim3(blocks01), dim3(kBlock), 0, stream, rows);
                        else if (from_ints) hipLaunchKernelGGL(k_first_two_rows<kRowsCheckInts>, dim3(blocks01), dim3(kBlock), 0, stream, rows);
                        else hipLaunchKernelGGL(k_first_two_rows<kRowsCheckWords>, dim3(blocks01), dim3(kBlock), 0, stream, rows);
                        I.unchecked = false;
                    } else {
                        hipLaunchKernelGGL(k_round_first_two, dim3(blocks01), dim3(kBlock), 0, stream, d01);
                    }
                }
                const bool checked = I.by_row && I.deferred;
                launch_final_sum2(w.partD, d01.pstrideD, 5, w.partT, d01.pstrideT, 6, blocks01, I.words, mb->words, my_seq,
                                  w.flags + 1, stream, checked ? w.flags + 2 : nullptr, mb->words + kMailboxBad + 2 * i);
            } else if (plan.kind == kRoundPair) {
                // binds the last two challenges, sums what this round and the next need
                PairArgs pr;
                memset(&pr, 0, sizeof pr);
                const EqSplit eq1 = ep.round(kk + 1);
                pr.rows = I.rows();
                pr.table = I.rows_pair();
                pr.N = (uint32_t)N;
                pr.a = I.planes(w.A29);
                pr.s = I.planes(w.S29);
                pr.aw = w.A;
                pr.aws = D;
                pr.sw = w.Sf;
                pr.sws = D / 2;
                pr.P = half / 2;
                pr.span = pair_span(pr.P);
                const unsigned pair_blocks = (unsigned)(pr.P / pr.span);
                pr.pstride = (size_t)pair_blocks * kPairValues;
                // cannot happen
                if (plan.bind != 2 || pr.span > ((size_t)1 << eq1.lbits) || pr.pstride > w.part_blocks * 5) return ZK_E_BADARG;
                F e[4];
                long_constants(e, r_last, 2, one());
                for (int q = 0; q < 4; ++q) pr.e[q] = to_dev(e[q]);
                pr.bias = long_bias(zero(), 32, 4);
                pr.weights = Planes29{ep.pool29, ep.count29};
                pr.lo_off = ep.suffix29_off[eq1.lbits];
                pr.lbits = eq1.lbits;
                pr.has_hi = eq1.has_hi;
                pr.hi_pool = ep.pool;
                pr.hi_stride = ep.stride;
                pr.hi_off = eq1.hi_off;
                pr.beta = to_dev(beta);
                pr.partials = w.partD;
                {
                    ProfileScope prof(kProfRound29, stream);
                    const bool from_rows = plan.s_source == kSFromRows;
                    if (from_rows && out32) hipLaunchKernelGGL((k_round_pair<true, true>), dim3(pair_blocks), dim3(kPairThreads), 0, stream, pr);
                    else if (from_rows) hipLaunchKernelGGL((k_round_pair<true, false>), dim3(pair_blocks), dim3(kPairThreads), 0, stream, pr);
                    else if (out32) hipLaunchKernelGGL((k_round_pair<false, true>), dim3(pair_blocks), dim3(kPairThreads), 0, stream, pr);
                    else hipLaunchKernelGGL((k_round_pair<false, false>), dim3(pair_blocks), dim3(kPairThreads), 0, stream, pr);
                }
                uint32_t* const pair_words = mb->words + kMailboxGrid + 8 * 89 * (kMailboxMaxInstances - ++pairs);
                I.grid_words = pair_words;
                hipLaunchKernelGGL(k_long_total, dim3(kPairValues), dim3(kBlock), 0, stream, w.partD, pr.pstride, pair_blocks, pair_words,
                                   mb->words, my_seq, w.flags + 1);
            } else if (plan.kind == kRoundBoth) {
                {
                    ProfileScope prof(kProfRoundSmall, stream);
                    if (kk > h) hipLaunchKernelGGL(k_round_both<true>, dim3(blocks, 3), dim3(kBlock), 0, stream, d, t);
                    else hipLaunchKernelGGL(k_round_both<false>, dim3(blocks, 3), dim3(kBlock), 0, stream, d, t);
                }
                launch_final_sum2(w.partD, d.pstride, 5, w.partT, t.pstride, 6, blocks, I.words, mb->words, my_seq,
                                  w.flags + 1, stream);
            } else if (plan.kind == kRound29) {
                // as many pairs per workgroup as its weights' shared factor allows, but at least 512 workgroups while the
                // round is large enough (measured: 1024 workgroups do the same, 2048 and workgroups of three or two
                // wavefronts are slower)
                const unsigned threads29 = (unsigned)kBlock;
                const size_t span29 = span;
                const unsigned blocks29 = blocks;
                if (span29 > (size_t)threads29 * kRound29MaxPairs) return ZK_E_BUFSZ;  // cannot happen
                DataRound29Args d29;
                // 32-bit words: A in place (stride D), S from the caller's vector or Sf; 29-bit limbs: A29, S29
                d29.A = Array29{w.A, D, Planes29{w.A29, D / 2}, w.A, D};
                d29.S = Array29{d.S.src, d.S.ss, Planes29{w.S29, D / 2}, w.Sf, D / 2};
                d29.half = half;
                d29.block_span = span29;
                d29.off0 = side1 ? half : 0;
                d29.off1 = side1 ? 0 : half;
                d29.r_prev = f29_unpack(to_dev(mul(r_prev, from_u64(32))).l);
                d29.r_first = f29_unpack(to_dev(mul(r_prev2, from_u64(32))).l);
                d29.r_both = f29_unpack(to_dev(mul(mul(r_prev2, r_prev), from_u64(32))).l);
                d29.beta = beta29;
                d29.weights = Planes29{ep.pool29, ep.count29};
                d29.lo_off = ep.suffix29_off[eq.lbits];
                d29.lbits = eq.lbits;
                d29.has_hi = eq.has_hi;
                d29.hi_pool = ep.pool;
                d29.hi_stride = ep.stride;
                d29.hi_off = eq.hi_off;
                d29.partials = d.partials;
                d29.pstride = d.pstride;
                d29.sx = nullptr;
                d29.sy = nullptr;
                d29.sf = w.fold4;
                const bool ints_round = plan.s_source == kSFromInts;
                if (ints_round) {
                    // constants of x0 + r (x1 - x0) + rho y0 + rho r (y1 - y0), r the first challenge
                    d29.sx = c.ints_x;
                    d29.sy = c.ints_y;
                    SmallFold4 f4;
                    const F cr = mul(r_prev, two64), crho = mul(ints_rho, two64), crr = mul(crho, r_prev);
                    to_device_limbs(f4.plus_one, two64);
                    to_device_limbs(f4.minus_one, neg(two64));
                    to_device_limbs(f4.plus_c, cr);
                    to_device_limbs(f4.minus_c, neg(cr));
                    to_device_limbs(f4.plus_rho, crho);
                    to_device_limbs(f4.minus_rho, neg(crho));
                    to_device_limbs(f4.plus_rho_c, crr);
                    to_device_limbs(f4.minus_rho_c, neg(crr));
                    hipLaunchKernelGGL(k_store_fold4, dim3(1), dim3(64), 0, stream, f4, w.fold4);
                }
                {
                    ProfileScope prof(kProfRound29, stream);
                    // cannot happen, see plan_round (integers are folded with 17 or fewer variables left: passes follow)
                    if ((plan.fold2 && (ints_round || !in32)) || (ints_round && !out32)) return ZK_E_BADARG;
                    if (plan.fold2 && out32) hipLaunchKernelGGL((k_round_data29<true, true, false, true>), dim3(blocks29), dim3(threads29), 0, stream, d29);
                    else if (plan.fold2) hipLaunchKernelGGL((k_round_data29<true, false, false, true>), dim3(blocks29), dim3(threads29), 0, stream, d29);
                    else if (ints_round) hipLaunchKernelGGL((k_round_data29<true, true, true>), dim3(blocks29), dim3(threads29), 0, stream, d29);
                    else if (in32 && out32) hipLaunchKernelGGL((k_round_data29<true, true>), dim3(blocks29), dim3(threads29), 0, stream, d29);
                    else if (in32) hipLaunchKernelGGL((k_round_data29<true, false>), dim3(blocks29), dim3(threads29), 0, stream, d29);
                    else if (out32) hipLaunchKernelGGL((k_round_data29<false, true>), dim3(blocks29), dim3(threads29), 0, stream, d29);
                    else hipLaunchKernelGGL((k_round_data29<false, false>), dim3(blocks29), dim3(threads29), 0, stream, d29);
                }
                launch_final_sum2(w.partD, d.pstride, 5, w.partT, t.pstride, 0, blocks29, I.words, mb->words, my_seq,
                                  w.flags + 1, stream);
            } else {
                {  // the first round (every later one is small, binds a table variable, or runs on 29-bit limbs)
                    ProfileScope prof(kProfRoundData, stream);
                    hipLaunchKernelGGL(k_round_data0, dim3(blocks), dim3(kBlock), 0, stream, d);
                }
                if (table_round) {  // only with kk == 0, i.e. D == N
                    ProfileScope prof(kProfRoundTable, stream);
                    hipLaunchKernelGGL(k_round_table<false>, dim3(blocks), dim3(kBlock), 0, stream, t);
                }
                launch_final_sum2(w.partD, d.pstride, 5, w.partT, t.pstride, table_round ? 6 : 0, blocks, I.words,
                                  mb->words, my_seq, w.flags + 1, stream);
            }
            ZK_HIP_TRY(hipGetLastError());
            I.b_cur = b_next;
            I.b_cur_stride = b_next_stride;
        }
        auto starts_pass = [&](size_t i) { return k >= inst[i].skip && plans[i].kind == kRoundGrid && plans[i].starts; };
        if (any_pass) {
            ProfileScope prof(kProfRoundSmall, stream);
            GridPass pass(K <= 2 ? kGridChunks : K <= 4 ? kGridChunks / 2 : kGridChunks / 4);  // 89 values an instance in 6 * 4096 places
            pass.challenges(r_last);
            for (size_t i = 0; i < K; ++i) {
                const RoundPlan& plan = plans[i];
                if (!starts_pass(i)) continue;
                Instance& I = inst[i];
                const int left = n - k, vars = plan.vars, tvars = plan.tvars;
                const Bound b = bind_pending(pass, I, plan, left, nullptr);
                const size_t P = (size_t)1 << (left - vars);
                const EqSplit eq = I.ep->round(k - I.skip + vars - 1);
                I.grid_words = mb->words + kMailboxGrid + 8 * pass.values;
                pass.add(b.p[0], b.stride[0], b.p[1], b.stride[1], vars, kGridWeighted, P, eq);
                if (tvars) {
                    pass.add(b.p[2], b.stride[2], b.p[4], b.stride[4], tvars, kGridTable, P, eq);
                    pass.add(b.p[2], b.stride[2], b.p[3], b.stride[3], tvars, kGridPlain, P, eq);
                }
            }
            ZK_TRY(pass.launch(mb, beta, inst[0].w.partT, mb->words + kMailboxGrid, any_ship ? 0 : seq, inst[0].w.flags + 1, stream));
        }
        if (any_ship) ZK_TRY(ship_to_host(k, seq));
        // while the device works: each instance's running claim, and the inverse the 29-bit round's other side needs
        // (instances of one length share it)
        for (size_t i = 0; i < K; ++i) {
            Instance& I = inst[i];
            if (k < I.skip) continue;
            I.claim = k == I.skip ? add(alpha, alpha2) : interpolate_at(I.fX, 4, r_prev);
            I.inv_den = zero();
            const F wD = mul(alpha, I.cD);
            if (plans[i].kind != kRound29 || is_zero(wD)) continue;
            bool shared = false;
            for (size_t j = 0; j < i && !shared; ++j)
                if (k >= inst[j].skip && inst[j].skip == I.skip && plans[j].kind == kRound29) {
                    I.inv_den = inst[j].inv_den;  // same bound variables, same product of weights
                    shared = true;
                }
            if (!shared) I.inv_den = inv(mul(wD, e_side[side1 ? 0 : 1]));
        }
        if (any_launch) ZK_TRY(mailbox_wait(mb, seq, stream));
        for (size_t i = 0; i < K; ++i) {
            if (!starts_pass(i)) continue;
            Instance& I = inst[i];
            const int vars = plans[i].vars, tvars = plans[i].tvars;
            const uint32_t* at = I.grid_words;
            I.gq.read(at, vars);
            at += 8 * grid_points(vars);
            for (int x = 0; x < 1 << vars; ++x, at += 8) I.gs[x] = from_dev(at);
            if (!tvars) continue;
            I.gt.read(at, tvars);
            I.gm.read(at + 8 * grid_points(tvars), tvars);
        }
        for (size_t i = 0; i < K; ++i) {
            if (k < inst[i].skip || plans[i].kind != kRoundPair) continue;
            Instance& I = inst[i];
            I.gq.read(I.grid_words, 2);
            for (int q = 0; q < 9; ++q) I.gq.g[q] = mul(I.gq.g[q], inv32);
            long_classes_to_grid(I.gq);
            for (int x = 0; x < 4; ++x) I.gs[x] = from_dev(I.grid_words + 8 * (9 + x));
            if (plans[i].vars == 2) continue;
            // this round alone: the next variable is the table's too
            F h3[3];
            for (int X = 0; X < 3; ++X)
                h3[X] = add(I.gq.g[3 * X], mul(u[k + 1], sub(I.gq.g[3 * X + 1], I.gq.g[3 * X])));
            for (int X = 0; X < 3; ++X) I.gq.g[X] = h3[X];
            I.gq.vars = 1;
            for (int x = 0; x < 2; ++x) I.gs[x] = add(I.gs[2 * x], I.gs[2 * x + 1]);
        }
        if (any_ship) read_shipped(k);
        if (any_launch) read_table_sums();
        for (size_t i = 0; i < K; ++i)
            if (k == inst[i].skip && inst[i].by_row) ZK_TRY(report_bad());

        F e[4], g[4];
        line_values(e, e_side[0], e_side[1]);
        for (int X = 0; X < 4; ++X) g[X] = zero();
        for (size_t i = 0; i < K; ++i) {
            Instance& I = inst[i];
            if (k < I.skip) {
                // not one of this instance's variables: its summand is the same at every X, and over the rest of the
                // cube it sums to 2^(skip - k - 1) times its whole sum alpha + alpha^2 (before its weight 2^-skip)
                F f = add(alpha, alpha2);
                for (int t = 0; t < I.skip - k - 1; ++t) f = add(f, f);
                for (int X = 0; X < 4; ++X) g[X] = add(g[X], mul(I.lam, f));
                continue;
            }
            const int kk = k - I.skip;
            const RoundPlan& plan = plans[i];
            const bool table_round = plan.table_round;
            const F wD = mul(alpha, I.cD);
            const F wT = table_round ? mul(alpha2, I.cT) : zero();
            I.half_pow = mul(I.half_pow, inv2);
            const uint32_t* sums = I.words;
            F q0, q1, qi, sA0, sA1;
            F hs[11];  // kRoundHost, kRoundGrid: the round's sums, formed here
            if (passes(plan)) {
                I.gq.sums(hs, u + k + 1);
                hs[3] = hs[4] = zero();
                const int later = 1 << (plan.left - 1);
                for (int x = 0; x < later; ++x) {
                    hs[3] = add(hs[3], I.gs[x]);
                    hs[4] = add(hs[4], I.gs[later + x]);
                }
                if (table_round) {
                    I.gt.sums(hs + 5, u + k + 1);
                    I.gm.sums(hs + 8, nullptr);
                }
                q0 = hs[0];
                q1 = hs[1];
                qi = hs[2];
                sA0 = hs[3];
                sA1 = hs[4];
            } else if (plan.kind == kRoundHost) {
                I.tail->sums((size_t)1 << (I.n - kk - 1), table_round, beta, hs);
                q0 = hs[0];
                q1 = hs[1];
                qi = hs[2];
                sA0 = hs[3];
                sA1 = hs[4];
            } else if (plan.kind == kRoundFirstTwo) {
                // the pass has summed, with the NEXT round's weights, what this round and the next are made of
                // (k_round_first_two): this round's leading coefficient splits by the next variable
                for (int q = 0; q < 9; ++q) I.pass01[q] = from_dev(sums + 8 * q);
                for (int q = 0; q < 5; ++q) I.pass01[q] = add(mul(I.pass01[q], inv32), from_u64(q < 4 ? 2 : 4));
                q0 = q1 = one();
                qi = add(mul(sub(one(), u[k + 1]), I.pass01[0]), mul(u[k + 1], I.pass01[1]));
                sA0 = add(I.pass01[5], I.pass01[6]);
                sA1 = add(I.pass01[7], I.pass01[8]);
            } else if (plan.kind == kRoundNoPass) {
                // every sum of this round is a polynomial of degree two in the challenge r before it
                const F& r = r_prev;
                const F t = mul(r, sub(one(), r));
                const F* P = I.pass01;
                q0 = sub(one(), mul(t, P[0]));
                q1 = sub(one(), mul(t, P[1]));
                qi = add(P[2], mul(r, add(sub(sub(P[3], P[2]), P[4]), mul(r, P[4]))));  // qd + r (T - qd - qe) + r^2 qe
                sA0 = add(P[5], mul(r, sub(P[7], P[5])));
                sA1 = add(P[6], mul(r, sub(P[8], P[6])));
            } else {
                q0 = from_dev(sums);
                q1 = from_dev(sums + 8);
                qi = from_dev(sums + 16);
                if (kk == 0) q0 = q1 = one();  // A (S + beta) = 1 everywhere and the weights sum to 1
                sA0 = from_dev(sums + 24);
                sA1 = from_dev(sums + 32);
            }
            const F table_const = mul(I.cB, I.half_pow);
            if (plan.kind == kRound29) {
                // the kernel has summed one side: (q0, sA0) hold that side's q and sum of A; the other side from
                // sA(0) + sA(1) = sA_prev(r_prev) and g(0) + g(1) = claim (never a table round: the table side is a constant)
                const int a = side1 ? 1 : 0;
                const F sA_b = sub(add(I.sA_prev[0], mul(r_prev, sub(I.sA_prev[1], I.sA_prev[0]))), sA0);
                const F g_a = add(add(mul(mul(wD, e_side[a]), q0), sA0), table_const);
                const F q_b = mul(sub(sub(sub(I.claim, g_a), sA_b), table_const), I.inv_den);
                const F q_a = q0, sA_a = sA0;
                q0 = a == 0 ? q_a : q_b;
                q1 = a == 0 ? q_b : q_a;
                sA0 = a == 0 ? sA_a : sA_b;
                sA1 = a == 0 ? sA_b : sA_a;
            }
            I.sA_prev[0] = sA0;
            I.sA_prev[1] = sA1;
            if (kk == 0) I.sum_A = add(sA0, sA1);
            F q[4], sa[4], tq[4], tm[4];
            quad_values(q, q0, q1, qi);
            line_values(sa, sA0, sA1);
            if (table_round && (plan.kind == kRoundHost || passes(plan))) {
                quad_values(tq, hs[5], hs[6], hs[7]);
                quad_values(tm, hs[8], hs[9], hs[10]);
            } else if (table_round) {
                quad_values(tq, from_dev(sums + 40), from_dev(sums + 48), from_dev(sums + 56));
                quad_values(tm, from_dev(sums + 64), from_dev(sums + 72), from_dev(sums + 80));
            }
            for (int X = 0; X < 4; ++X) {
                F data = add(mul(mul(wD, e[X]), q[X]), sa[X]);
                F table = table_round ? mul(I.scale, sub(mul(mul(wT, e[X]), tq[X]), tm[X])) : table_const;
                F f = add(data, table);
                I.fX[X] = f;
                g[X] = add(g[X], !c.batch ? f : mul(I.lam, f));
            }
        }
        for (int X = 0; X < 4; ++X) to_bytes(out + 32 * X, g[X]);
        tr.absorb("g", out, 128);
        out += 128;
        F r = tr.challenge("r");
        F er = add(mul(sub(one(), u[k]), sub(one(), r)), mul(u[k], r));
        for (size_t i = 0; i < K; ++i) {
            Instance& I = inst[i];
            if (k < I.skip) continue;
            I.cD = mul(I.cD, er);
            if (plans[i].table_round) I.cT = mul(I.cT, er);
        }
        r_prev2 = r_prev;
        r_prev = r;
        r_last[0] = r_last[1];
        r_last[1] = r_last[2];
        r_last[2] = r;
        for (size_t i = 0; i < K; ++i) {
            Instance& I = inst[i];
            if (k < I.skip) continue;
            if (plans[i].kind == kRoundHost) {
                I.tail->fold((size_t)1 << (n - k - 1), plans[i].table_round, r);
            } else if (passes(plans[i])) {
                I.gq.bind(r);
                const int half = 1 << (plans[i].left - 1);
                for (int x = 0; x < half; ++x) I.gs[x] = add(I.gs[x], mul(r, sub(I.gs[half + x], I.gs[x])));
                if (plans[i].table_round) {
                    I.gt.bind(r);
                    I.gm.bind(r);
                }
            }
        }
    }

    // -- final claims -------------------------------------------------------------------------------------
    {
        // the host has bound the last variables itself: each array's first element is its claim (an instance of one
        // element has had no rounds: its arrays are fetched now)
        bool missing = false;
        for (size_t i = 0; i < K; ++i) missing = missing || !inst[i].tail;
        if (missing) {
            const uint32_t seq = mb->next_seq();
            ZK_TRY(ship_to_host(n, seq));
            ZK_TRY(mailbox_wait(mb, seq, stream));
            read_shipped(n);
        }
        ZK_HIP_TRY(hipStreamSynchronize(stream));  // everything of this call has left the device
        read_table_sums();
        uint8_t* first = out;
        for (size_t i = 0; i < K; ++i) {
            const HostTail& t = *inst[i].tail;
            const F claims[5] = {t.A[0], t.S[0], t.B[0], t.M[0], t.T[0]};
            for (int q = 0; q < 5; ++q) {
                const F& v = claims[q];
                if (q == 0 && inst[i].n == 0) inst[i].sum_A = v;
                to_bytes(out, v);
                out += 32;
            }
        }
        tr.absorb("final", first, 160 * K);
    }
    if (c.aux) {
        c.aux->beta = to_canonical(beta);
        c.aux->alpha = to_canonical(alpha);
        c.aux->sum_A = to_canonical(inst[0].sum_A);
        c.aux->sum_mB = to_canonical(inst[0].sum_mB);
        c.aux->bad_index = 0;
    }
    if (c.baux) {
        memset(c.baux, 0, sizeof *c.baux);
        c.baux->beta = to_canonical(beta);
        c.baux->alpha = to_canonical(alpha);
        c.baux->lambda = to_canonical(lambda);
        for (size_t i = 0; i < K; ++i) {
            c.baux->sum_A[i] = to_canonical(inst[i].sum_A);
            c.baux->sum_mB[i] = to_canonical(inst[i].sum_mB);
        }
    }
    return ZK_OK;
}

// ---- verifier ----------------------------------------------------------------------------------

static size_t verify_ws_bytes(size_t D, size_t N) {
    Carver cv(nullptr, 0);
    cv.limbs(N);                                   // m as field elements
    cv.take((vec_digest_leaves(D) + vec_digest_leaves(N)) * 32);  // hash trees over the witness vectors A and B
    cv.take(vec_digest_row_digests(D) * 32);
    cv.take(vec_digest_row_digests(N) * 32);
    cv.take(256);                                  // their ticket
    const int n = log2_floor(D), l = log2_floor(N);
    const int nvars[kMleMaxJobs] = {n, n, l, l, l};
    cv.take(mle_scratch_bytes_many(nvars, kMleMaxJobs));
    return cv.used();
}

struct VerifyCall {
    const uint8_t* seed = nullptr;
    const uint8_t* proof = nullptr;
    size_t len = 0;
    size_t K = 1;
    const fr_vec* T = nullptr;
    size_t D = 0;
    bool batch = false;
    bool multi = false;            // shapes may differ: lengths of the tensors in Ds, of the tables in T[i].n
    const size_t* Ds = nullptr;
    const tlookup_witness* wit = nullptr;  // K entries, or null
    tlookup_claims* claims = nullptr;      // single proof
    tlookup_batch_claims* bclaims = nullptr;
    void* ws = nullptr;
    size_t ws_bytes = 0;
    void* stream = nullptr;
};

static int verify_core(const VerifyCall& c) {
    using namespace host;
    const size_t K = c.K;
    if (!c.seed || !c.proof || !c.T || K == 0 || K > kMailboxMaxInstances || (!c.batch && (K != 1 || c.multi))) return ZK_E_BADARG;
    if (c.multi && !c.Ds) return ZK_E_BADARG;
    // shapes: n variables in all; instance i has n_i of them, the last ones (skip_i = n - n_i)
    size_t Ds[kMailboxMaxInstances], Ns[kMailboxMaxInstances];
    int ns[kMailboxMaxInstances], ls[kMailboxMaxInstances], hs[kMailboxMaxInstances], skips[kMailboxMaxInstances];
    int n = 0;
    size_t D_max = 1, N_max = 1;
    for (size_t i = 0; i < K; ++i) {
        Ds[i] = c.multi ? c.Ds[i] : c.D;
        Ns[i] = c.T[c.multi ? i : 0].n;
        if (!is_pow2(Ds[i]) || !is_pow2(Ns[i]) || Ns[i] > Ds[i] || Ds[i] > ((size_t)1 << 31)) return ZK_E_BADARG;
        if (c.T[i].n != Ns[i] || !vec_ok(c.T[i], Ns[i])) return ZK_E_BADARG;
        ns[i] = log2_floor(Ds[i]);
        ls[i] = log2_floor(Ns[i]);
        hs[i] = ns[i] - ls[i];
        if (ns[i] > n) n = ns[i];
        if (Ds[i] > D_max) D_max = Ds[i];
        if (Ns[i] > N_max) N_max = Ns[i];
    }
    for (size_t i = 0; i < K; ++i) skips[i] = n - ns[i];
    if (!c.ws || c.ws_bytes < verify_ws_bytes(D_max, N_max)) return ZK_E_BUFSZ;
    const uint8_t* proof = c.proof;
    const uint8_t* digests;
    if (c.multi) {
        if (c.len != multi_proof_bytes(n, K)) return ZK_E_REJECT;
        if (memcmp(proof, "ZKTM\x01\0\0\0", 8) != 0) return ZK_E_REJECT;
        if (get_le64(proof + 8) != K) return ZK_E_REJECT;
        for (size_t i = 0; i < K; ++i)
            if (get_le64(proof + 16 + 16 * i) != Ds[i] || get_le64(proof + 24 + 16 * i) != Ns[i]) return ZK_E_REJECT;
        digests = proof + 16 + 16 * K;
    } else if (c.batch) {
        if (c.len != batch_proof_bytes(Ds[0], K)) return ZK_E_REJECT;
        if (memcmp(proof, "ZKTB\x02\0\0\0", 8) != 0) return ZK_E_REJECT;
        if (get_le64(proof + 8) != Ds[0] || get_le64(proof + 16) != Ns[0] || get_le64(proof + 24) != K) return ZK_E_REJECT;
        digests = proof + 32;
    } else {
        if (c.len != tlookup_proof_bytes(Ds[0])) return ZK_E_REJECT;
        if (memcmp(proof, "ZKTL\x02\0\0\0", 8) != 0) return ZK_E_REJECT;
        if (get_le64(proof + 8) != Ds[0] || get_le64(proof + 16) != Ns[0]) return ZK_E_REJECT;
        digests = proof + 24;
    }
    const uint8_t* ab_digests = digests + 32 * K;  // per instance: digest(A), digest(B)
    const uint8_t* body = ab_digests + 64 * K;
    F el[4 * 32 + 5 * kMailboxMaxInstances];
    const int nel = 4 * n + 5 * (int)K;
    for (int i = 0; i < nel; ++i)
        if (!from_bytes(&el[i], body + 32 * i)) return ZK_E_REJECT;

    uint64_t dims[1 + 2 * kMailboxMaxInstances];
    int ndims;
    if (c.multi) {
        dims[0] = K;
        for (size_t i = 0; i < K; ++i) {
            dims[1 + 2 * i] = Ds[i];
            dims[2 + 2 * i] = Ns[i];
        }
        ndims = 1 + 2 * (int)K;
    } else {
        dims[0] = Ds[0];
        dims[1] = Ns[0];
        dims[2] = K;
        ndims = c.batch ? 3 : 2;
    }
    Transcript tr(c.multi ? "zkmi/tlookup-multi/v1" : c.batch ? "zkmi/tlookup-batch/v2" : "zkmi/tlookup/v2", c.seed, dims, ndims);
    for (size_t i = 0; i < K; ++i) tr.absorb("m", digests + 32 * i, 32);
    F beta = tr.challenge("beta");
    for (size_t i = 0; i < K; ++i) {
        tr.absorb("A", ab_digests + 64 * i, 32);
        tr.absorb("B", ab_digests + 64 * i + 32, 32);
    }
    F alpha = tr.challenge("alpha");
    F alpha2 = sqr(alpha);
    F u[32], v[32];
    for (int t = 0; t < n; ++t) u[t] = tr.challenge("u");
    F lambda = one();
    if (c.batch) lambda = tr.challenge("lambda");
    F lam[kMailboxMaxInstances], lam_sum = zero();
    for (size_t i = 0; i < K; ++i) {
        lam[i] = i == 0 ? one() : mul(lam[i - 1], lambda);
        lam_sum = add(lam_sum, lam[i]);
    }
    F claim = mul(lam_sum, add(alpha, alpha2));
    for (int k = 0; k < n; ++k) {
        const F* g = &el[4 * k];
        if (!equal(add(g[0], g[1]), claim)) return ZK_E_REJECT;
        tr.absorb("g", body + 128 * k, 128);
        v[k] = tr.challenge("r");
        claim = interpolate_at(g, 4, v[k]);
    }
    const F* fin = &el[4 * n];
    tr.absorb("final", body + 128 * n, 160 * K);
    const F inv2 = inv(from_u64(2));
    F total = zero();
    for (size_t i = 0; i < K; ++i) {
        const F* f = fin + 5 * i;
        const int skip = skips[i], h = hs[i];
        F scale = one(), weight = lam[i];  // 2^-h; lambda^i 2^-skip
        for (int t = 0; t < h; ++t) scale = mul(scale, inv2);
        for (int t = 0; t < skip; ++t) weight = mul(weight, inv2);
        const F e_full = eq_point(u + skip, v + skip, ns[i]), e_tab = eq_point(u + skip + h, v + skip + h, ls[i]);
        F lhs = mul(f[0], add(mul(mul(alpha, e_full), add(f[1], beta)), one()));
        F rhs = mul(scale, mul(f[2], sub(mul(mul(alpha2, e_tab), add(f[4], beta)), f[3])));
        total = add(total, mul(weight, add(lhs, rhs)));
    }
    if (!equal(total, claim)) return ZK_E_REJECT;

    // claims against tensors
    hipStream_t stream = as_stream(c.stream);
    Mailbox* mb;
    ZK_TRY(mailbox_get(&mb));
    Carver cv(c.ws, c.ws_bytes);
    uint32_t* Mfr = cv.limbs(N_max);
    uint32_t* dig_leaves = (uint32_t*)cv.take((vec_digest_leaves(D_max) + vec_digest_leaves(N_max)) * 32);
    uint32_t* dig_rows = (uint32_t*)cv.take(vec_digest_row_digests(D_max) * 32);
    uint32_t* dig_rows_b = (uint32_t*)cv.take(vec_digest_row_digests(N_max) * 32);
    uint32_t* dig_ticket = (uint32_t*)cv.take(256);
    for (size_t i = 0; i < K; ++i) {
        const F* f = fin + 5 * i;
        const size_t D = Ds[i], N = Ns[i];
        const int ni = ns[i], l = ls[i];
        const F* vd = v + skips[i];          // the instance's point
        const F* vt = vd + hs[i];            // its table's
        const uint32_t nleaves = (uint32_t)div_up(N, kLeafCounts);
        const tlookup_witness* wit = c.wit ? c.wit + i : nullptr;
        const bool have_s = wit && wit->S.limbs && vec_ok(wit->S, D), have_a = wit && wit->A.limbs && vec_ok(wit->A, D),
                   have_b = wit && wit->B.limbs && vec_ok(wit->B, N), have_m = wit && wit->m;
        // Everything of the instance is enqueued before anything is waited for: the hash trees of A and B in the same
        // launches, the values of all tensors in the same launches.
        launch_fill_u32(dig_ticket, 1, 0u, stream);
        ZK_TRY(mailbox_bulk(mb, (size_t)nleaves * 32));  // before anything is on its way there
        VecDigestJob trees[2];
        int ntrees = 0;
        if (have_a) trees[ntrees++] = VecDigestJob{wit->A.limbs, wit->A.stride, D, dig_rows, LeafGather()};
        if (have_b) trees[ntrees++] = VecDigestJob{wit->B.limbs, wit->B.stride, N, dig_rows_b, LeafGather()};
        MleJob jobs[kMleMaxJobs];
        int njobs = 0;
        auto add_job = [&](const uint32_t* a, size_t stride, int nv, const F* pt) {
            jobs[njobs] = MleJob{a, stride, nv, pt, mb->words + 8 * njobs};
            return njobs++;
        };
        const int job_t = add_job(c.T[i].limbs, c.T[i].stride, l, vt);
        const int job_s = have_s ? add_job(wit->S.limbs, wit->S.stride, ni, vd) : -1;
        const int job_a = have_a ? add_job(wit->A.limbs, wit->A.stride, ni, vd) : -1;
        const int job_b = have_b ? add_job(wit->B.limbs, wit->B.stride, l, vt) : -1;
        int job_m = -1;
        if (have_m) {
            TableJobs<1> tables{};
            tables.job[0].N = (uint32_t)N;
            tables.job[0].m = const_cast<uint32_t*>(wit->m);  // only read
            tables.job[0].M = Mfr;
            hipLaunchKernelGGL(k_counts_to_fr<1>, dim3(grid_for(N)), dim3(kBlock), 0, stream, tables);
            job_m = add_job(Mfr, N, l, vt);
        }
        {
            Carver scratch = cv;
            const uint32_t seq = mb->next_seq();
            MlePlan plan;
            ZK_TRY(mle_eval_begin(plan, jobs, njobs, scratch, mb, seq, stream));
            LeafDigestArgs<1> lf{};
            if (have_m) lf.job[0] = LeafDigestJob{(uint32_t*)(mb->bulk + kBulkDigests), wit->m, (uint32_t)N, nleaves, nullptr, nullptr};
            LeavesBeside beside{lf.job[0], &plan.step[0], plan.blocks[0], false};
            const size_t leaves = (have_a ? vec_digest_leaves(D) : 0) + (have_b ? vec_digest_leaves(N) : 0);
            if (ntrees)
                ZK_TRY(vec_digest_launch(trees, ntrees, host_leaves(leaves, Sha256::has_instructions()), dig_leaves, mb, 0, dig_ticket,
                                         stream, nullptr, BadWords{}, plan.steps > 1 ? &beside : nullptr));
            if (have_m && !beside.launched)
                hipLaunchKernelGGL(k_leaf_digests<1>, dim3((unsigned)div_up(nleaves, 64)), dim3(128), 0, stream, lf);
            ZK_TRY(mle_eval_rest(plan, beside.launched ? 1 : 0, mb, stream));
            ZK_TRY(mailbox_wait(mb, seq, stream));
            ZK_HIP_TRY(hipStreamSynchronize(stream));
        }
        auto value_is = [&](int job, const F& want) { return equal(from_dev(mb->words + 8 * job), want); };
        uint8_t tree_digests[2][32];  // of all trees, also where a value is rejected first: finishing clears the leaves' bytes
        for (int q = 0; q < ntrees; ++q) vec_digest_finish(tree_digests[q], trees[q]);
        auto digest_is = [&](int tree, const uint8_t* want) { return memcmp(tree_digests[tree], want, 32) == 0; };
        if (!value_is(job_t, f[4])) return ZK_E_REJECT;
        if (!wit) continue;
        if (wit->S.limbs && !have_s) return ZK_E_BADARG;
        if (have_s && !value_is(job_s, f[1])) return ZK_E_REJECT;
        if (wit->A.limbs && !have_a) return ZK_E_BADARG;
        // a witness vector must also be the one whose digest the proof carries
        if (have_a && (!value_is(job_a, f[0]) || !digest_is(0, ab_digests + 64 * i))) return ZK_E_REJECT;
        if (wit->B.limbs && !have_b) return ZK_E_BADARG;
        if (have_b && (!value_is(job_b, f[2]) || !digest_is(ntrees - 1, ab_digests + 64 * i + 32)))
            return ZK_E_REJECT;
        if (have_m) {
            if (!value_is(job_m, f[3])) return ZK_E_REJECT;
            uint8_t md[32];
            digest_of_leaves(md, mb->bulk + kBulkDigests, nleaves);
            if (memcmp(md, digests + 32 * i, 32) != 0) return ZK_E_REJECT;
        }
    }
    if (c.claims) {
        memset(c.claims, 0, sizeof *c.claims);
        c.claims->A_v = to_canonical(fin[0]);
        c.claims->S_v = to_canonical(fin[1]);
        c.claims->B_vp = to_canonical(fin[2]);
        c.claims->m_vp = to_canonical(fin[3]);
        c.claims->T_vp = to_canonical(fin[4]);
        c.claims->nvars = n;
        for (int t = 0; t < n; ++t) c.claims->v[t] = to_canonical(v[t]);
    }
    if (c.bclaims) {
        memset(c.bclaims, 0, sizeof *c.bclaims);
        c.bclaims->nvars = n;
        c.bclaims->count = (int)K;
        c.bclaims->lambda = to_canonical(lambda);
        for (int t = 0; t < n; ++t) c.bclaims->v[t] = to_canonical(v[t]);
        for (size_t i = 0; i < K; ++i)
            for (int q = 0; q < 5; ++q) c.bclaims->value[i][q] = to_canonical(fin[5 * i + q]);
    }
    return ZK_OK;
}

}  // namespace zkmi

using namespace zkmi;

extern "C" {

size_t tlookup_proof_bytes(size_t D) { return 120 + (size_t)log2_floor(D ? D : 1) * 128 + 160; }

size_t tlookup_workspace_bytes(size_t D, size_t N) {
    if (!is_pow2(D) || !is_pow2(N) || N > D) return 0;
    return prove_ws_bytes(D, N);
}

int tlookup_multiplicities(uint32_t* m, fr_vec S, const uint32_t* idx, fr_vec T, void* ws, size_t ws_bytes,
                           uint64_t* bad_index, void* stream) {
    const size_t D = S.n, N = T.n;
    if (!m || D == 0 || N == 0 || N > ((size_t)1 << 31) || !vec_ok(S, D) || !vec_ok(T, N)) return ZK_E_BADARG;
    if (!is_pow2(D) || !is_pow2(N) || N > D) return ZK_E_BADARG;
    if (!ws || ws_bytes < prove_ws_bytes(D, N)) return ZK_E_BUFSZ;
    Mailbox* mb;
    ZK_TRY(mailbox_get(&mb));
    Carver cv(ws, ws_bytes);
    ProveWs w;
    carve_prove(w, cv, D, N);
    const bool to_host = host_counts(&N, 1, host::Sha256::has_instructions());
    ZK_TRY(mailbox_bulk(mb, counted_bytes(w, N, to_host)));
    const uint8_t* const staged = mb->bulk + kBulkDigests;
    const uint32_t seq = mb->next_seq();
    const CountJob job{&w, S, idx, T, D, N, mb->bulk + kBulkDigests, false, nullptr};
    ZK_TRY(count_rows(&job, 1, to_host, seq, mb, as_stream(stream)));
    ZK_TRY(mailbox_wait(mb, seq, as_stream(stream)));
    forget_counts(&job, 1, to_host);
    const uint64_t bad = counted_bad(staged);
    if (bad != UINT64_MAX) {
        if (bad_index) *bad_index = bad;
        ZK_HIP_TRY(hipStreamSynchronize(as_stream(stream)));
        return ZK_E_NOT_IN_TABLE;
    }
    ZK_HIP_TRY(hipMemcpyAsync(m, w.m, N * 4, hipMemcpyDeviceToDevice, as_stream(stream)));
    ZK_HIP_TRY(hipStreamSynchronize(as_stream(stream)));
    return ZK_OK;
}

static int prove_single(const uint8_t seed[32], fr_vec S, const uint32_t* idx, fr_vec T, const fr_t* forced_beta,
                        bool by_rows, uint8_t* proof, size_t cap, size_t* len, tlookup_aux* aux, void* ws,
                        size_t ws_bytes, void* stream, bool check_upfront = false) {
    ProveCall c;
    c.check_upfront = check_upfront;
    c.seed = seed;
    c.K = 1;
    c.S = &S;
    c.idx = &idx;
    c.T = &T;
    c.forced_beta = forced_beta;
    c.by_rows = by_rows;
    c.proof = proof;
    c.cap = cap;
    c.len = len;
    c.aux = aux;
    c.ws = ws;
    c.ws_bytes = ws_bytes;
    c.stream = stream;
    return prove_core(c);
}

int tlookup_prove(const uint8_t seed[32], fr_vec S, const uint32_t* idx, fr_vec T, uint8_t* proof, size_t cap,
                  size_t* len, tlookup_aux* aux, void* ws, size_t ws_bytes, void* stream) {
    return prove_single(seed, S, idx, T, nullptr, false, proof, cap, len, aux, ws, ws_bytes, stream);
}

static __global__ void __launch_bounds__(kBlock) k_small_materialize(uint32_t* __restrict__ dst, size_t ds, size_t n,
                                                                     SmallSource ints) {
    for (size_t i = blockIdx.x * (size_t)kBlock + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlock) {
        Fr v;
        small_source_load(v.l, ints, i);
        fr_store(dst, ds, i, v);
    }
}

size_t tlookup_small_workspace_bytes(size_t D, size_t N) {
    if (!is_pow2(D) || !is_pow2(N) || N > D) return 0;
    size_t base = align_up(prove_ws_bytes(D, N), 256);
    return small_source_shape_ok(D, N) ? base : base + D * 32;  // other shapes: S is written out as field elements first
}

int tlookup_prove_small(const uint8_t seed[32], const int32_t* X, const int32_t* Y, const fr_t* rho, size_t D,
                        const uint32_t* idx, fr_vec T, uint8_t* proof, size_t cap, size_t* len, tlookup_aux* aux, void* ws,
                        size_t ws_bytes, void* stream) {
    using namespace host;
    const size_t N = T.n;
    if (!seed || !X || !idx || (Y != nullptr) != (rho != nullptr)) return ZK_E_BADARG;
    if (!is_pow2(D) || !is_pow2(N) || N > D || D > ((size_t)1 << 31) || !vec_ok(T, N)) return ZK_E_BADARG;
    if (rho && !canonical_in_range(*rho)) return ZK_E_BADARG;
    if (len) *len = tlookup_proof_bytes(D);
    if (!ws || ws_bytes < tlookup_small_workspace_bytes(D, N)) return ZK_E_BUFSZ;
    if (small_source_shape_ok(D, N)) {
        ProveCall c;
        c.seed = seed;
        c.K = 1;
        c.idx = &idx;
        c.T = &T;
        c.ints_x = X;
        c.ints_y = Y;
        c.ints_rho = rho;
        c.ints_D = D;
        c.proof = proof;
        c.cap = cap;
        c.len = len;
        c.aux = aux;
        c.ws = ws;
        c.ws_bytes = ws_bytes;
        c.stream = stream;
        return prove_core(c);
    }
    // a shape whose first fold is not a kernel of its own: the tensor as field elements, then the usual path
    const size_t base = align_up(prove_ws_bytes(D, N), 256);
    SmallSource src;
    memset(&src, 0, sizeof src);
    const F two64 = mul(from_u64((uint64_t)1 << 32), from_u64((uint64_t)1 << 32));
    const F r = rho ? from_canonical(*rho) : zero();
    src.x = X;
    src.y = Y;
    to_device_limbs(src.plus_one, two64);
    to_device_limbs(src.minus_one, neg(two64));
    to_device_limbs(src.plus_rho, mul(r, two64));
    to_device_limbs(src.minus_rho, neg(mul(r, two64)));
    fr_vec S = {(uint32_t*)((uint8_t*)ws + base), D, D};
    hipLaunchKernelGGL(k_small_materialize, dim3(grid_for(D, kBlock, 16384)), dim3(kBlock), 0, as_stream(stream), S.limbs,
                       S.stride, D, src);
    ZK_HIP_TRY(hipGetLastError());
    return prove_single(seed, S, idx, T, nullptr, false, proof, cap, len, aux, ws, base, stream);
}

// The rounds of a proof of this shape, walked on the host (no GPU is touched): four
// integers per round, see zkmi.h.
static int selftest_plan(size_t D, size_t N, size_t K, bool from_ints, int32_t* out, size_t cap_rounds) {
    const int n = log2_floor(D), h = n - log2_floor(N);
    if ((size_t)n > cap_rounds) return ZK_E_BUFSZ;
    RoundState st;
    for (int k = 0; k < n; ++k) {
        const RoundPlan pl = plan_round(n, h, k, K, from_ints, st);
        const bool several = pl.kind == kRoundGrid || pl.kind == kRoundHost, pair = pl.kind == kRoundPair;
        out[4 * k] = pl.kind;
        out[4 * k + 1] = pl.s_source;
        out[4 * k + 2] = pair ? pl.vars : several ? pl.vars + 8 * pl.tvars : pl.in32 ? 1 : 0;
        out[4 * k + 3] = pair ? pl.bind + (pl.out32 ? 8 : 0) : several ? pl.bind + 8 * pl.bind_t : pl.out32 ? 1 : 0;
    }
    return n;
}
static bool selftest_shape_ok(size_t D, size_t N, size_t K, const int32_t* out) {
    return out && is_pow2(D) && is_pow2(N) && N <= D && D <= ((size_t)1 << 31) && K != 0 && K <= kMailboxMaxInstances;
}

int zkmi_selftest_tlookup_plan(size_t D, size_t N, size_t K, int from_ints, int32_t* out, size_t cap_rounds) {
    if (!selftest_shape_ok(D, N, K, out)) return ZK_E_BADARG;
    if (from_ints && (K != 1 || !small_source_shape_ok(D, N))) return ZK_E_BADARG;
    return selftest_plan(D, N, K, from_ints != 0, out, cap_rounds);
}

int zkmi_selftest_tlookup_rows_plan(size_t D, size_t N, size_t K, int32_t* out, size_t cap_rounds) {
    if (!selftest_shape_ok(D, N, K, out) || !rounds_by_row(log2_floor(D), log2_floor(D) - log2_floor(N))) return ZK_E_BADARG;
    return selftest_plan(D, N, K, false, out, cap_rounds);
}

// Who makes, compares and hashes what (hash_plan), see zkmi.h.
int zkmi_selftest_tlookup_hashes(const size_t* D, const size_t* N, const int32_t* hints, size_t K, int how, int sha_instructions,
                                 int32_t* out) {
    if (!D || !N || !hints || !out || K == 0 || K > kMailboxMaxInstances || how < 0 || how > 2) return ZK_E_BADARG;
    bool given[kMailboxMaxInstances];
    for (size_t i = 0; i < K; ++i) {
        if (!selftest_shape_ok(D[i], N[i], K, out) || (how == 2 && !hints[i])) return ZK_E_BADARG;
        given[i] = hints[i] != 0;
    }
    const HashPlan p = hash_plan(D, N, given, K, how == 1, how == 2, sha_instructions != 0);
    out[0] = p.leaves_to_host;
    out[1] = p.counts_to_host;
    for (size_t i = 0; i < K; ++i) {
        out[2 + 2 * i] = p.of[i].maker;
        out[3 + 2 * i] = p.of[i].deferred;
    }
    return ZK_OK;
}

// The host's rounds (HostTail) on arrays and challenges of the caller's choosing: no GPU is touched.
int zkmi_selftest_host_rounds(const fr_t* A, const fr_t* S, const fr_t* B, const fr_t* M, const fr_t* T, size_t n_data,
                              size_t n_table, const fr_t* u_rest, const fr_t* beta, const fr_t* challenges, fr_t* sums,
                              fr_t* finals) {
    using namespace host;
    if (!A || !S || !B || !M || !T || !beta || !sums || !finals) return ZK_E_BADARG;
    if (!is_pow2(n_data) || !is_pow2(n_table) || n_data < 2 || n_data > kMailboxShipEntries || n_table > n_data) return ZK_E_BADARG;
    const int d = log2_floor(n_data);
    if (d > 1 && !u_rest) return ZK_E_BADARG;
    if (!challenges) return ZK_E_BADARG;
    for (int t = 0; t < d - 1; ++t)
        if (!canonical_in_range(u_rest[t])) return ZK_E_BADARG;
    for (int t = 0; t < d; ++t)
        if (!canonical_in_range(challenges[t])) return ZK_E_BADARG;
    if (!canonical_in_range(*beta)) return ZK_E_BADARG;
    HostTail ht;
    const fr_t* const src[5] = {A, S, B, M, T};
    F* const dst[5] = {ht.A, ht.S, ht.B, ht.M, ht.T};
    for (int q = 0; q < 5; ++q)
        for (size_t j = 0; j < (q < 2 ? n_data : n_table); ++j) {
            if (!canonical_in_range(src[q][j])) return ZK_E_BADARG;
            dst[q][j] = from_canonical(src[q][j]);
        }
    F us[8];
    for (int t = 0; t < d - 1; ++t) us[t] = from_canonical(u_rest[t]);
    ht.weights(us, d - 1);
    const F b = from_canonical(*beta);
    int round = 0;
    for (size_t half = n_data / 2; half >= 1; half >>= 1, ++round) {
        const bool table_round = 2 * half <= n_table;
        F out[11];
        ht.sums(half, table_round, b, out);
        for (int q = 0; q < 11; ++q) sums[11 * round + q] = to_canonical(out[q]);
        ht.fold(half, table_round, from_canonical(challenges[round]));
    }
    for (int q = 0; q < 5; ++q) finals[q] = to_canonical(dst[q][0]);
    return d;
}

int tlookup_prove_checked(const uint8_t seed[32], fr_vec S, const uint32_t* idx, fr_vec T, uint8_t* proof, size_t cap,
                          size_t* len, tlookup_aux* aux, void* ws, size_t ws_bytes, void* stream) {
    return prove_single(seed, S, idx, T, nullptr, false, proof, cap, len, aux, ws, ws_bytes, stream, true);
}

int tlookup_prove_by_rows(const uint8_t seed[32], fr_vec S, const uint32_t* idx, fr_vec T, uint8_t* proof, size_t cap,
                          size_t* len, tlookup_aux* aux, void* ws, size_t ws_bytes, void* stream) {
    if (!idx) return ZK_E_BADARG;
    return prove_single(seed, S, idx, T, nullptr, true, proof, cap, len, aux, ws, ws_bytes, stream);
}

int tlookup_prove_with_beta(const uint8_t seed[32], fr_vec S, const uint32_t* idx, fr_vec T, const fr_t* forced_beta,
                            uint8_t* proof, size_t cap, size_t* len, tlookup_aux* aux, void* ws, size_t ws_bytes,
                            void* stream) {
    if (!forced_beta) return ZK_E_BADARG;
    return prove_single(seed, S, idx, T, forced_beta, false, proof, cap, len, aux, ws, ws_bytes, stream);
}

size_t tlookup_verify_workspace_bytes(size_t D, size_t N) {
    if (!is_pow2(D) || !is_pow2(N) || N > D) return 0;
    return verify_ws_bytes(D, N);
}

int tlookup_verify(const uint8_t seed[32], const uint8_t* proof, size_t len, fr_vec T, size_t D,
                   const tlookup_witness* witness, tlookup_claims* claims, void* ws, size_t ws_bytes, void* stream) {
    VerifyCall c;
    c.seed = seed;
    c.proof = proof;
    c.len = len;
    c.K = 1;
    c.T = &T;
    c.D = D;
    c.wit = witness;
    c.claims = claims;
    c.ws = ws;
    c.ws_bytes = ws_bytes;
    c.stream = stream;
    return verify_core(c);
}

size_t tlookup_batch_proof_bytes(size_t D, size_t K) { return batch_proof_bytes(D, K); }

size_t tlookup_batch_workspace_bytes(size_t D, size_t N, size_t K) {
    if (!is_pow2(D) || !is_pow2(N) || N > D || K == 0 || K > TLOOKUP_BATCH_MAX) return 0;
    return prove_ws_bytes(D, N, K);
}

int tlookup_prove_batch(const uint8_t seed[32], const fr_vec* S, const uint32_t* const* idx, const fr_vec* T, size_t K,
                        uint8_t* proof, size_t cap, size_t* len, tlookup_batch_aux* aux, void* ws, size_t ws_bytes,
                        void* stream) {
    ProveCall c;
    c.seed = seed;
    c.K = K;
    c.S = S;
    c.idx = idx;
    c.T = T;
    c.batch = true;
    c.proof = proof;
    c.cap = cap;
    c.len = len;
    c.baux = aux;
    c.ws = ws;
    c.ws_bytes = ws_bytes;
    c.stream = stream;
    return prove_core(c);
}

int tlookup_verify_batch(const uint8_t seed[32], const uint8_t* proof, size_t len, const fr_vec* T, size_t K, size_t D,
                         const tlookup_witness* witness, tlookup_batch_claims* claims, void* ws, size_t ws_bytes,
                         void* stream) {
    VerifyCall c;
    c.seed = seed;
    c.proof = proof;
    c.len = len;
    c.K = K;
    c.T = T;
    c.D = D;
    c.batch = true;
    c.wit = witness;
    c.bclaims = claims;
    c.ws = ws;
    c.ws_bytes = ws_bytes;
    c.stream = stream;
    return verify_core(c);
}

static bool multi_shapes_ok(const size_t* D, const size_t* N, size_t K) {
    if (!D || !N || K == 0 || K > TLOOKUP_BATCH_MAX) return false;
    for (size_t i = 0; i < K; ++i)
        if (!is_pow2(D[i]) || !is_pow2(N[i]) || N[i] > D[i] || D[i] > ((size_t)1 << 31)) return false;
    return true;
}

size_t tlookup_multi_proof_bytes(const size_t* D, size_t K) {
    if (!D || K == 0 || K > TLOOKUP_BATCH_MAX) return 0;
    int n = 0;
    for (size_t i = 0; i < K; ++i) {
        if (!is_pow2(D[i])) return 0;
        if (log2_floor(D[i]) > n) n = log2_floor(D[i]);
    }
    return multi_proof_bytes(n, K);
}

size_t tlookup_multi_workspace_bytes(const size_t* D, const size_t* N, size_t K) {
    if (!multi_shapes_ok(D, N, K)) return 0;
    return prove_ws_bytes_shapes(D, N, K);
}

int tlookup_prove_multi(const uint8_t seed[32], const fr_vec* S, const uint32_t* const* idx, const fr_vec* T, size_t K,
                        uint8_t* proof, size_t cap, size_t* len, tlookup_batch_aux* aux, void* ws, size_t ws_bytes,
                        void* stream) {
    ProveCall c;
    c.seed = seed;
    c.K = K;
    c.S = S;
    c.idx = idx;
    c.T = T;
    c.batch = true;
    c.multi = true;
    c.proof = proof;
    c.cap = cap;
    c.len = len;
    c.baux = aux;
    c.ws = ws;
    c.ws_bytes = ws_bytes;
    c.stream = stream;
    return prove_core(c);
}

size_t tlookup_multi_verify_workspace_bytes(const size_t* D, const size_t* N, size_t K) {
    if (!multi_shapes_ok(D, N, K)) return 0;
    size_t D_max = 1, N_max = 1;
    for (size_t i = 0; i < K; ++i) {
        if (D[i] > D_max) D_max = D[i];
        if (N[i] > N_max) N_max = N[i];
    }
    return verify_ws_bytes(D_max, N_max);
}

int tlookup_verify_multi(const uint8_t seed[32], const uint8_t* proof, size_t len, const fr_vec* T, const size_t* D,
                         size_t K, const tlookup_witness* witness, tlookup_batch_claims* claims, void* ws,
                         size_t ws_bytes, void* stream) {
    VerifyCall c;
    c.seed = seed;
    c.proof = proof;
    c.len = len;
    c.K = K;
    c.T = T;
    c.Ds = D;
    c.batch = true;
    c.multi = true;
    c.wit = witness;
    c.bclaims = claims;
    c.ws = ws;
    c.ws_bytes = ws_bytes;
    c.stream = stream;
    return verify_core(c);
}

}  // extern "C"

// Sums of products of field elements on the matrix cores.
//
// sum_p x_p y_p needs no reduction until its end, and in base 256 it is
//   sum_(i,j) 2^(8 (i + j)) C_ij,   C_ij = sum_p (digit i of x_p) (digit j of y_p):
// the 32 x 32 matrix C is a product of a 32 x P matrix of bytes with a P x 32 one,
// and v_mfma_i32_32x32x32_i8 adds 32 positions p to it in 32 cycles.  64 products of
// 256-bit integers so cost two matrix instructions, 64 cycles, beside which the vector
// ALU is free; on the vector ALU they are 81 multiply-adds and the carries, 500 cycles.
// What the vector ALU still does is a digit conversion per operand: sixteen
// instructions, then two 16-byte stores to LDS and four transposing loads.
//
// Digits are balanced (-128..127), so that nothing has to be corrected afterwards:
// the bytes of v + C0 with the top bit of each flipped, C0 = 128 (1 + 256 + ...).
// Needs v + C0 < 2^256, i.e. v < 1.099 r: reduced elements, and products as f29_mul
// leaves them (below r + r^2 / 2^261 < 1.015 r).
//
// Operands come one element per lane (lane = position).  A transposing LDS load gives
// sixteen lanes that read eight rows of sixteen bytes one column each, so the digits
// are staged as two planes (digits 0..15 and 16..31) of sixteen bytes per position:
// stores and loads both run over consecutive addresses.  The staging area is a
// wavefront's own; LDS instructions of one wavefront execute in order, so there are no
// barriers in the loop.
#pragma once
#include "mfma_dev.h"
#include "reduce_dev.h"

namespace zkmi {

typedef int v2i __attribute__((ext_vector_type(2)));

static const int kOuterBatch = 64;         // positions a wavefront takes at a time
static const int kOuterStage = 2048;       // bytes of LDS a wavefront stages one operand in

// One operand of 64 positions for two matrix instructions: lane l holds digit l % 32
// of positions 32 s + 16 (l / 32) .. + 15 in half s.
struct OuterOperand {
    v4i half[2];
};

__device__ __forceinline__ void balanced_digits(uint32_t (&d)[8], const uint32_t (&v)[8]) {
    uint32_t carry = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        uint32_t co;
        d[j] = __builtin_addc(v[j], kFlip, carry, &co) ^ kFlip;
        carry = co;
    }
}

// The words of element first + lane (first the same in all lanes, its plane addresses in
// scalar registers, stepped from one to the next).  Global, not flat, accesses: a flat load
// also counts as an LDS instruction, so that every wait for staged digits would wait for it.
__device__ __forceinline__ void outer_load(uint32_t (&v)[8], const uint32_t* p, size_t stride, size_t first) {
    typedef const __attribute__((address_space(1))) uint32_t* global_words;
    global_words q = (global_words)p + first;
    const uint32_t lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        asm("" : "+s"(q));
        v[k] = q[lane];
        q += stride;
    }
}

// The same of the first `count` lanes' elements; the lanes after them read the last of those.
__device__ __forceinline__ void outer_load_part(uint32_t (&v)[8], const uint32_t* p, size_t stride, size_t first, uint32_t count) {
    typedef const __attribute__((address_space(1))) uint32_t* global_words;
    global_words q = (global_words)p + first;
    uint32_t lane = threadIdx.x & 63;
    if (lane >= count) lane = count - 1;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        asm("" : "+s"(q));
        v[k] = q[lane];
        q += stride;
    }
}

// digits: 32 bytes of this lane's position.  A fence of the wavefront's own accesses and
// no instruction: it keeps the compiler from mixing the lanes' stores with the loads.
__device__ __forceinline__ void outer_put(const uint32_t (&digits)[8], uint8_t* stage) {
    const int lane = threadIdx.x & 63;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    *reinterpret_cast<uint4*>(stage + 16 * lane) = make_uint4(digits[0], digits[1], digits[2], digits[3]);
    *reinterpret_cast<uint4*>(stage + 1024 + 16 * lane) = make_uint4(digits[4], digits[5], digits[6], digits[7]);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
}

__device__ __forceinline__ OuterOperand outer_get(const uint8_t* stage) {
    const int lane = threadIdx.x & 63;
    const uint8_t* at = stage + ((lane >> 4) & 1) * 1024 + (lane >> 5) * 256 + (lane & 15) * 8;
    OuterOperand o;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        typedef __attribute__((address_space(3))) v2i lds_v2i;
        const v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i*)(at + 512 * s));
        const v2i hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i*)(at + 512 * s + 128));
        o.half[s] = v4i{lo.x, lo.y, hi.x, hi.y};
    }
    return o;
}

// Sixteen bytes from `from` (each lane its own) to LDS, lane l's at lds + 16 l, without a trip
// through registers; not waited for (vector_loads_done).  Inline, as the compiler would wait
// for it at the next LDS access of whatever address; its own waits count too few loads in
// flight and so are never too short.
__device__ __forceinline__ void load_to_lds(const void* from, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(from), "s"(lds) : "memory", "m0");
}
// The same from a place all lanes share and an offset of each.
__device__ __forceinline__ void load_to_lds(const void* from, uint32_t offset, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(offset), "s"(from), "s"(lds) : "memory", "m0");
}
// Where in LDS p lies, as those take it: uniform.
__device__ __forceinline__ uint32_t lds_place(const uint8_t* p) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint8_t*)p);
}
// Waits until at most LATER of this wavefront's vector memory accesses are on their way: they
// complete in order, so all but the last LATER are done.
template <int LATER = 0>
__device__ __forceinline__ void vector_loads_done() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LATER) : "memory"); }
// This wavefront's LDS reads so far have come back: what they read may be overwritten.
__device__ __forceinline__ void lds_reads_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

__device__ __forceinline__ OuterOperand outer_stage(const uint32_t (&digits)[8], uint8_t* stage) {
    outer_put(digits, stage);
    return outer_get(stage);
}

__device__ __forceinline__ OuterOperand outer_operand(const uint32_t (&v)[8], uint8_t* stage) {
    uint32_t d[8];
    balanced_digits(d, v);
    return outer_stage(d, stage);
}

// Operands made beforehand: those of positions 64 b .. 64 b + 63 at table[128 b ..).
__device__ __forceinline__ void outer_save(uint4* table, size_t b, const OuterOperand& o) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int s = 0; s < 2; ++s) table[(2 * b + s) * 64 + lane] = make_uint4(o.half[s].x, o.half[s].y, o.half[s].z, o.half[s].w);
}
__device__ __forceinline__ OuterOperand outer_saved(const uint4* table, size_t b) {
    typedef const __attribute__((address_space(1))) v4i* global_v4i;
    const global_v4i at = (global_v4i)table + 128 * b + (threadIdx.x & 63);
    return OuterOperand{{at[0], at[64]}};
}

__device__ __forceinline__ void outer_mac(v16i& acc, const OuterOperand& a, const OuterOperand& b) {
    acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a.half[0], b.half[0], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a.half[1], b.half[1], acc, 0, 0, 0);
}

__device__ __forceinline__ void outer_clear(v16i& acc) {
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0;
}

// An operand whose column n is one at every position and whose other columns are zero:
// outer_mac(acc, x, outer_column(n)) adds up x's digits in column n.
__device__ __forceinline__ OuterOperand outer_column(int n) {
    const int v = (int)(threadIdx.x & 31) == n ? 0x01010101 : 0;
    return OuterOperand{{v4i{v, v, v, v}, v4i{v, v, v, v}}};
}

// The sums of a workgroup of four wavefronts.  `sums`: N * 1024 words of LDS (may
// overlap the staging areas; they are still being read when the first wavefronts return,
// so that a caller who stages or closes again waits at a barrier first).  Columns are taken in groups of GROUP lanes, each the
// digits of one value: 32 (field elements), 8 or 4 (64- or 32-bit integers, four or
// eight to an operand).  Calls out(q, group, x) in one lane for every sum of accumulator q,
//   x = sum_(i,j) 2^(8 (i + j)) C_ij / 2^256 mod r, reduced.
// An accumulator may hold kOuterMaxProducts products per column (limbs_dev.h): callers
// assert their positions per workgroup times products per position.
// SUMS: the last accumulator's columns are values by themselves (outer_column): out(N - 1,
// column, sum_i 2^(8 i) C_ij mod r) for every column.
template <int N, int GROUP, bool SUMS, class Out>
__device__ __forceinline__ void outer_values(const int* sums, Out&& out);

template <int N, int GROUP, bool SUMS = false, class Out>
__device__ __forceinline__ void outer_close(const v16i (&acc)[N], int* sums, Out&& out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int q = 0; q < N; ++q)
#pragma unroll
            for (int r = 0; r < 16; ++r) sums[(q * 16 + r) * 64 + lane] = acc[q][r];
    }
    __syncthreads();
    if (wave != 0) {
#pragma unroll
        for (int q = 0; q < N; ++q)
#pragma unroll
            for (int r = 0; r < 16; ++r) atomicAdd(&sums[(q * 16 + r) * 64 + lane], acc[q][r]);
    }
    __syncthreads();
    outer_values<N, GROUP, SUMS>(sums, out);
}

// The second half of it: from the workgroup's sums in LDS (accumulator q's at 1024 q), for
// workgroups of any number of wavefronts.  outer_sums_clear (all threads, between barriers) and
// outer_sums_add make such sums of accumulators that the wavefronts hold different ones of.
template <int N>
__device__ __forceinline__ void outer_sums_clear(int* sums) {
    for (unsigned k = threadIdx.x; k < N * 1024; k += blockDim.x) sums[k] = 0;
}
__device__ __forceinline__ void outer_sums_add(int* sums, int q, const v16i& acc) {
#pragma unroll
    for (int r = 0; r < 16; ++r) atomicAdd(&sums[(q * 16 + r) * 64 + (threadIdx.x & 63)], acc[r]);
}
template <int N, int GROUP, bool SUMS, class Out>
__device__ __forceinline__ void outer_values(const int* sums, Out&& out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const ToepBias bias = outer_bias();
    // two accumulators at a time: lanes 0..31 take the columns of the first, the others those of the second
#pragma unroll 1
    for (int q = 2 * wave; q < N; q += blockDim.x / 32) {
        const int q1 = q + 1 < N ? q + 1 : q;
        v16i a, b;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            a[r] = sums[(q * 16 + r) * 64 + lane];
            b[r] = sums[(q1 * 16 + r) * 64 + lane];
        }
        Fr v = toeplitz_finish(a, b, bias);
        Fr pw;
        const int at = lane & (GROUP - 1);
#pragma unroll
        for (int j = 0; j < 8; ++j) pw.l[j] = (at >> 2) == j ? 1u << (8 * (at & 3)) : 0u;
        const int which = lane < 32 ? q : q + 1;
        if constexpr (SUMS) {
            const Fr column = v;
            if (which == N - 1) out(which, lane & 31, column);
        }
        v = fr_mul(v, pw);
        v = dpp_add_step<0x111, 0xf>(v);
        v = dpp_add_step<0x112, 0xf>(v);
        if constexpr (GROUP >= 8) v = dpp_add_step<0x114, 0xf>(v);
        if constexpr (GROUP == 32) {
            v = dpp_add_step<0x118, 0xf>(v);
            v = dpp_add_step<0x142, 0xa>(v);
        }
        if (which < (SUMS ? N - 1 : N) && at == GROUP - 1) out(which, (lane & 31) / GROUP, v);
    }
}

}  // namespace zkmi

// Field arithmetic on the matrix cores: multiplication of many elements by a few
// constants.
//
// x * e mod r for a fixed e is linear in the base-256 digits of x:
//   x e = sum_k d_k (2^(8k) e mod r),   d_k the digits of x, k = 0..31,
// and the digits of (2^(8k) e mod r) form a 32 x 32 matrix E of bytes that depends
// on e alone.  So a sum  sum_c e_c x_c  over C constants is, for 32 elements p at
// once, a product of a 32 x 32C matrix with a 32C x 32 one: C instructions
// v_mfma_i32_32x32x32_i8, whose second operand is the elements' own 32-bit words
// as they lie in memory (lane i holds sixteen consecutive digits of element i).
// What comes out are 32 column sums per element; one pass of carries and one
// multiple of r taken off give the reduced result.  Nothing here cares whether x
// is in Montgomery form: the map is linear, x * 2^256 goes to x e * 2^256.
//
// Signs.  The instruction multiplies signed bytes.  The constants' digits are
// balanced (-128..127: the bytes of v + C0 with the top bit of each flipped, C0 =
// 128 * (1 + 256 + 256^2 + ...)).  The elements' bytes are used as d - 128 (top
// bit flipped): what is accumulated is the sum for x - C0 instead of x, which is
// put right by one addition of C0 sum_c e_c mod r per output (toeplitz_bias).
//
// Cost per 64 outputs: 2C matrix instructions of 32 cycles and about 130 + 8C
// vector instructions per lane, against about 300 C for multiplications on the
// vector ALU.
#pragma once
#include "fr_dev.h"
#include "limbs_dev.h"

namespace zkmi {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

static const uint32_t kFlip = 0x80808080u;  // top bit of every byte: unsigned digit d <-> signed digit d - 128
static const int kToepBytes = 1024;         // one constant's matrix: 64 lanes x 16 bytes

// Column k of the matrix of a constant: the balanced digits of 2^(8k) e mod r, for
// e in Montgomery form, as eight words of signed bytes.
__device__ __forceinline__ void toeplitz_column(uint32_t (&digits)[8], const Fr& e_mont, int k) {
    Fr pw;
#pragma unroll
    for (int j = 0; j < 8; ++j) pw.l[j] = (k >> 2) == j ? 1u << (8 * (k & 3)) : 0u;
    const Fr v = fr_mul(e_mont, pw);  // e 2^(8k), no longer in Montgomery form
    uint32_t carry = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        uint32_t co;
        digits[j] = __builtin_addc(v.l[j], kFlip, carry, &co) ^ kFlip;
        carry = co;  // v + C0 < 2^256: no carry out of the top word
    }
}

// Where the byte (row m, column k) of a matrix lies: lane (k/16) * 32 + m of the
// first operand holds row m, columns 16 (k/16) .. + 15.
__device__ __forceinline__ int toeplitz_byte(int m, int k) { return (((k >> 4) * 32 + m) << 4) + (k & 15); }

__device__ __forceinline__ void toeplitz_store(uint8_t* matrix, const uint32_t (&digits)[8], int k) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int b = 0; b < 4; ++b) matrix[toeplitz_byte(4 * j + b, k)] = (uint8_t)(digits[j] >> (8 * b));
}

// acc of a tile of 32 elements (lane l: element l % 32, rows 8 g + 4 (l / 32) + t for
// g, t = 0..3, i.e. digits 0..3 of limbs g' = 2 g + l / 32) -> four limbs, 64 bits signed.
// As multiply-adds by powers the compiler cannot see through: four instructions a limb,
// where shifts, sign extensions and 64-bit additions are twelve.
__device__ __forceinline__ void digits_to_limbs(int64_t (&limb)[4], const v16i& acc) {
    int unit = 1, d1 = 1 << 8, d2 = 1 << 16, d3 = 1 << 24;
    asm("" : "+s"(unit), "+s"(d1), "+s"(d2), "+s"(d3));
#pragma unroll
    for (int g = 0; g < 4; ++g)
        limb[g] = ((((int64_t)acc[4 * g] * unit + (int64_t)acc[4 * g + 1] * d1) + (int64_t)acc[4 * g + 2] * d2) + (int64_t)acc[4 * g + 3] * d3);
}

// Two tiles' half limbs -> all eight limbs of one element per lane: lanes 0..31 get
// the element of the first tile, lanes 32..63 that of the second.
__device__ __forceinline__ void limbs_of_pair(int64_t (&out)[8], const int64_t (&a)[4], const int64_t (&b)[4]) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)a[g], (uint32_t)b[g], false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)((uint64_t)a[g] >> 32), (uint32_t)((uint64_t)b[g] >> 32), false, false);
        out[2 * g] = (int64_t)(((uint64_t)hi[0] << 32) | lo[0]);
        out[2 * g + 1] = (int64_t)(((uint64_t)hi[1] << 32) | lo[1]);
    }
}

// The bias of a sum over C constants e_c: what it is short of when the elements' digits go
// in as d - 128, C0 sum_c e_c mod r, plus the multiple of r that keeps the result from
// being negative (a column sum is at least -C * 32 * 128 * 128, so 4096 C r do).
__device__ __forceinline__ Fr limbs_reduce(const int64_t (&limb)[8], const ToepBias& bias) {
    uint32_t w[8];
    limbs_reduce_words(w, limb, bias);
    return fr_reduce_once(w);
}

// ---- folding several variables at once --------------------------------------------
//
// dst_p = sum_c e_c src_(c P + p), p < P: the top log2 C variables of a vector of
// C P elements bound to a point, e_c = e~(point, c).  A wavefront makes 128 outputs
// (four tiles of 32): per constant it reads 128 elements, four words per load.
struct ToepSource {
    const uint32_t* p;
    size_t stride;
    int vec;  // 16-byte loads allowed: base and stride multiples of four words, P a multiple of four
};

// Adds constants [c0, c1) into acc.  `table`: the constants' matrices, one after the
// other.  Tile j's element in lane i = lane % 32 is base + 4 i + j (vec) or base +
// 32 j + i; places beyond P read the last element(s) instead.
template <bool VEC>
__device__ __forceinline__ void toeplitz_accumulate(v16i (&acc)[4], const ToepSource& src, size_t P, size_t base,
                                                    const uint4* __restrict__ table, unsigned c0, unsigned c1) {
    const int lane = threadIdx.x & 63, i = lane & 31, h = lane >> 5;
    const uint32_t* at[VEC ? 1 : 4];
    if constexpr (VEC) {
        size_t e = base + 4 * (size_t)i;
        if (e + 4 > P) e = P - 4;
        at[0] = src.p + 4 * (size_t)h * src.stride + e;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            size_t e = base + 32 * (size_t)j + i;
            if (e >= P) e = P - 1;
            at[j] = src.p + 4 * (size_t)h * src.stride + e;
        }
    }
#pragma unroll 2
    for (unsigned c = c0; c < c1; ++c) {
        const uint4 raw = table[(size_t)c * 64 + lane];
        const v4i m = {(int)raw.x, (int)raw.y, (int)raw.z, (int)raw.w};
        uint32_t x[4][4];  // [limb][tile]
        if constexpr (VEC) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint4 v = *reinterpret_cast<const uint4*>(at[0] + (size_t)c * P + q * src.stride);
                x[q][0] = v.x; x[q][1] = v.y; x[q][2] = v.z; x[q][3] = v.w;
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int j = 0; j < 4; ++j) x[q][j] = at[j][(size_t)c * P + q * src.stride];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const v4i b = {(int)(x[0][j] ^ kFlip), (int)(x[1][j] ^ kFlip), (int)(x[2][j] ^ kFlip), (int)(x[3][j] ^ kFlip)};
            acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(m, b, acc[j], 0, 0, 0);
        }
    }
}

// The reduced results of a pair of tiles, one element per lane.
__device__ __forceinline__ Fr toeplitz_finish(const v16i& first, const v16i& second, const ToepBias& bias) {
    int64_t a[4], b[4], limb[8];
    digits_to_limbs(a, first);
    digits_to_limbs(b, second);
    limbs_of_pair(limb, a, b);
    return limbs_reduce(limb, bias);
}

}  // namespace zkmi

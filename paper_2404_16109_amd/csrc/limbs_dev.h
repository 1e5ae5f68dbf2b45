// The way from sums of byte products (matrix cores) to a field element, as plain functions:
// no device-only construct, checked on the host against big integers at its bounds.
#pragma once
#include <stddef.h>

#include "fr29_dev.h"

namespace zkmi {

// Added to a sum of limbs that may be negative: a multiple of r, and with it (toeplitz_finish's
// callers) what the digits' form is short of.
struct ToepBias {
    uint32_t w[9];
};

// V = sum_q limb_q 2^(32 q) + bias, known to lie in [0, 2^23 r), less a multiple of r: a value
// below 2 r congruent to V.
ZK_HD void limbs_reduce_words(uint32_t (&w)[8], const int64_t (&limb)[8], const ToepBias& bias) {
    int64_t c = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        c += limb[q] + (int64_t)(uint64_t)bias.w[q];
        w[q] = (uint32_t)c;
        c >>= 32;
    }
    c += bias.w[8];
    // quotient by t = floor(V / 2^248) < 2^29.9 and floor(2^280 / r) / 2^32: the two truncations cost less than
    // 2^248 / r + V / 2^280 < 1/115 + 2^29.9 / 2^32 < 1/4, so that it is at most one too small and V - q r < 2 r;
    // subtracted as q (2^256 - r) modulo 2^256
    const uint32_t t = ((uint32_t)c << 8) | (w[7] >> 24);
    const uint32_t q = (uint32_t)(((uint64_t)t * 0x02355094u) >> 32);
    constexpr uint32_t nr[8] = {0xffffffffu, 0x00000000u, 0x0001a401u, 0xac425bfdu, 0xf65e27fau, 0xccc627f7u, 0xd66282b7u, 0x8c1258acu};
    uint64_t acc = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        acc += (uint64_t)q * nr[j] + w[j];
        w[j] = (uint32_t)acc;
        acc >>= 32;
    }
}

// Sums of products (outer_dev.h).  A column sum_p x_p d_p over the products p of an
// accumulator, x_p below 1.015 r and the digits d_p -128..127, is below 1.015 * 2^21 r in
// magnitude for kOuterMaxProducts of them, and reaches it where all d_p are alike: the bias
// of 2^22 r leaves a value in [2^20 r, 2^23 r).
static const size_t kOuterMaxSpan = 4096;          // positions per workgroup
static const size_t kOuterMaxProducts = 4 * 4096;  // products per workgroup and accumulator

ZK_HD ToepBias outer_bias() {
    constexpr uint32_t r32[8] = {0x00000001u, 0xffffffffu, 0xfffe5bfeu, 0x53bda402u, 0x09a1d805u, 0x3339d808u, 0x299d7d48u, 0x73eda753u};
    ToepBias bias;
#pragma unroll
    for (int k = 0; k < 9; ++k) bias.w[k] = (k < 8 ? r32[k] << 22 : 0u) | (k > 0 ? r32[k - 1] >> 10 : 0u);
    return bias;
}

}  // namespace zkmi

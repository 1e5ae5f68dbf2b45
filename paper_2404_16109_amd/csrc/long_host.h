// Host side of the passes whose folds and sums run on the matrix cores (link_long.h, tlookup_rows.h).
#pragma once
#include "grid_dev.h"
#include "limbs_dev.h"

namespace zkmi {

// C0 s mod r (C0: 0x80 in each of the low `bytes` bytes) plus 4096 m r.
static inline ToepBias long_bias(const host::F& s, int bytes, uint32_t m) {
    using namespace host;
    fr_t c0;
    memset(&c0, 0, sizeof c0);
    memset(&c0, 0x80, (size_t)bytes);
    if (bytes == 32) {  // C0 - r
        static const uint32_t w[8] = {0x8080807fu, 0x80808081u, 0x80822481u, 0x2cc2dc7du, 0x76dea87bu, 0x4d46a878u, 0x56e30338u, 0x0c92d92du};
        memcpy(&c0, w, sizeof w);
    }
    const fr_t v = to_canonical(mul(from_canonical(c0), s));
    uint32_t c[8];
    memcpy(c, &v, sizeof c);
    static const uint32_t r32[8] = {ZK_R0, ZK_R1, ZK_R2, ZK_R3, ZK_R4, ZK_R5, ZK_R6, ZK_R7};
    ToepBias b;
    uint64_t acc = 0;
    for (int k = 0; k < 8; ++k) {
        acc += (uint64_t)r32[k] * (4096u * m) + c[k];
        b.w[k] = (uint32_t)acc;
        acc >>= 32;
    }
    b.w[8] = (uint32_t)acc;
    return b;
}

// e~(r, c) over the last `vars` challenges, the last one in r[2], times s.
static inline void long_constants(host::F* e, const host::F r[3], int vars, const host::F& s) {
    using namespace host;
    e[0] = s;
    for (int v = 0; v < vars; ++v)
        for (int c = (1 << v) - 1; c >= 0; --c) {
            const F hi = mul(e[c], r[3 - vars + v]);
            e[2 * c] = sub(e[c], hi);
            e[2 * c + 1] = hi;
        }
}

// Class sums (per variable: 0, 1, mixed) to values on {0, 1, inf}: inf = 0 + 1 - mixed.
static inline void long_classes_to_grid(HostGrid& g) {
    using namespace host;
    const int count = (int)grid_points(g.vars);
    for (int step = 1; step < count; step *= 3)
        for (int i = 0; i < count; ++i)
            if (i / step % 3 == 2) g.g[i] = sub(add(g.g[i - 2 * step], g.g[i - step]), g.g[i]);
}

}  // namespace zkmi

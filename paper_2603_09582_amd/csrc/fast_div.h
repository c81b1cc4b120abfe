// Division of non-negative ints by a divisor that the host knows, with one high product (Granlund and Montgomery, "Division by
// invariant integers using multiplication", 1994, figure 4.1): plain C++, the same on the device and in a host program.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define BINATTN_HD_DIV __host__ __device__ __attribute__((always_inline)) inline
#else
#define BINATTN_HD_DIV inline
#endif

namespace binattn {

struct FastDiv {
    uint32_t m;
    int s;
};

// 1 <= d < 2^31
inline FastDiv make_fast_div(int d) {
    FastDiv f;
    f.s = 0;
    while (((int64_t)1 << f.s) < d) ++f.s;
    f.m = (uint32_t)(((((uint64_t)1 << f.s) - (uint64_t)d) << 32) / (uint64_t)d + 1);
    return f;
}

// n / d for 0 <= n < 2^31, m and s those of make_fast_div(d)
BINATTN_HD_DIV int fast_div(int n, uint32_t m, int s) {
    const uint32_t t = (uint32_t)(((uint64_t)m * (uint32_t)n) >> 32);
    return (int)((t + (uint32_t)n) >> s);
}

}  // namespace binattn

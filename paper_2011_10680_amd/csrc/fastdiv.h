// Division of the kernels' indices by launch constants: a multiplication and a shift.
#pragma once
#include "common.h"

namespace hawq {

// n / d for 0 <= n < 2^31: umulhi(n, mul) >> sh, mul = ceil(2^(31 + s) / d), s = ceil(log2 d), sh = s - 1; d = 1: mul = 0
struct FastDiv { uint32_t mul, sh; };

inline FastDiv fast_div(uint32_t d) {
    if (d <= 1) return {0, 0};
    uint32_t s = 0;
    while ((1ull << s) < d) ++s;
    return {(uint32_t)(((1ull << (31 + s)) + d - 1) / d), s - 1};
}
__device__ __forceinline__ uint32_t fdiv(uint32_t n, FastDiv f) { return f.mul ? __umulhi(n, f.mul) >> f.sh : n; }

}  // namespace hawq

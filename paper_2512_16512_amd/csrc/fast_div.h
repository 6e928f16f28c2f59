// Integer division by a launch constant without the divide sequence.
#pragma once

#include <hip/hip_runtime.h>

namespace xtc {

// Division of n < 2^31 by a launch constant d, by multiplication (Granlund and
// Montgomery, "Division by invariant integers using multiplication", PLDI
// 1994): (n * mul) >> (32 + shift) with
// mul = ceil(2^(31 + l) / d), l = ceil(log2 d): the rounding of mul adds less
// than n / 2^(31 + l) < 1 / d.
struct FastDiv {
    unsigned mul;
    int shift;       // l - 1; -1: d is 1
    int d;
};
inline FastDiv fast_div(int d) {
    int l = 0;
    while ((1ll << l) < d) ++l;
    return FastDiv{(unsigned)(((1ull << (31 + l)) + d - 1) / d), l - 1, d};
}
__device__ __forceinline__ int div_by(int n, const FastDiv &f) {
    return f.shift < 0 ? n : (int)(__umulhi((unsigned)n, f.mul) >> f.shift);
}

}  // namespace xtc

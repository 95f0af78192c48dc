// Division by a kernel argument.
#pragma once

#include <hip/hip_runtime.h>

namespace fs {

// n / d for 0 <= n < 2^31 by a multiplication (d = 1 .. 2^31 - 1 fixed on the
// host): mul = floor(2^(31 + l) / d) + 1 with l = ceil(log2 d), so that n * mul
// exceeds n * 2^(31 + l) / d by at most n < 2^(31 + l) / d.  A division by a
// kernel argument costs some 25 dependent instructions ahead of the first load.
struct Div {
    unsigned mul;
    int shift;
    __device__ __forceinline__ unsigned operator()(unsigned n) const {
        return (unsigned)(((unsigned long long)n * mul) >> shift);
    }
};
inline Div make_div(int d) {
    int l = 0;
    while (l < 31 && (1ll << l) < d) ++l;
    return Div{(unsigned)((1ull << (31 + l)) / (unsigned)d + 1), 31 + l};
}

}  // namespace fs

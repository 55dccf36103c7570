// Division by a divisor that the host knows: a multiplication and a shift (T. Granlund and P. Montgomery, "Division by Invariant Integers
// using Multiplication", 1994), where the kernel would spend some forty dependent instructions.
#pragma once
#include <stdint.h>

namespace cp {

// n / d for 0 <= n < 2^31, 1 <= d < 2^31
struct FastDiv {
    uint32_t mul, shift;
    FastDiv() : mul(1), shift(0) {}
    explicit FastDiv(uint32_t d) : shift(0) {
        while ((1ull << shift) < d) ++shift;
        mul = (uint32_t)(((((1ull << shift) - d) << 32) / d) + 1);
    }
    __host__ __device__ __forceinline__ uint32_t div(uint32_t n) const { return ((uint32_t)(((unsigned long long)mul * n) >> 32) + n) >> shift; }
};

}  // namespace cp

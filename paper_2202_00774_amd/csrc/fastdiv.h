// Division of an index by a number that is fixed for a launch, as one multiplication.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sdgp {

struct FastDiv {
    uint32_t mul, shift;
};

// n / d for 0 <= n < 2^31, 1 <= d < 2^31: mul = ceil(2^(31 + shift) / d) with 2^shift >= d fits 32 bits, and its rounding error
// of less than one part in 2^31 cannot carry a quotient over.
inline FastDiv fast_div(uint32_t d) {
    FastDiv f{0, 0};
    while (((uint64_t)1 << f.shift) < d) ++f.shift;
    f.mul = (uint32_t)((((uint64_t)1 << (31 + f.shift)) + d - 1) / d);
    return f;
}
__host__ __device__ __forceinline__ uint32_t divide(uint32_t n, FastDiv f) { return (uint32_t)(((uint64_t)n * f.mul) >> (31 + f.shift)); }

}  // namespace sdgp

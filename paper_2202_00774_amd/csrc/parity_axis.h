// Parity classes of the input pixels of a strided filter, along one axis.
#pragma once

#include <hip/hip_runtime.h>

namespace sdgp {

// Pixel i*stride + a of class a meets filter positions r0, r0 + stride, ... (count of them) at gradient positions i + shift,
// i + shift - 1, ...; n pixels of the axis are of the class.  Int holds a pixel's index.
template <typename Int>
struct ParityAxis {
    int r0, count, shift;
    Int n;
};

template <typename Int>
__device__ __forceinline__ ParityAxis<Int> parity_axis(Int size, int filter, int stride, int pad, int a) {
    ParityAxis<Int> x;
    x.r0 = (a + pad) % stride;
    x.count = x.r0 < filter ? (filter - x.r0 + stride - 1) / stride : 0;
    x.shift = (a + pad - x.r0) / stride;
    x.n = size > a ? (size - a + stride - 1) / stride : 0;
    return x;
}

}  // namespace sdgp

// Launch helpers for the small-problem backward-data kernel; included by the files that instantiate it.
#pragma once

#include "bwd_small.h"

namespace sdgp {

template <int M, int RK, bool NLE2>
int launch_small_one(const SmallParams& p, hipStream_t stream) {
    constexpr int lds = kSmallWaves * 4 * 16 * 64 * (int)sizeof(float);
    auto kern = bwd_small<M, RK, NLE2>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return SDGP_ERR_HIP;
    const unsigned x = ((unsigned)p.col_tiles * (unsigned)p.row_tiles + 7u) / 8u * 8u;
    hipLaunchKernelGGL(kern, dim3(x, (unsigned)(p.stride * p.stride)), dim3(64 * kSmallWaves), lds, stream, p);
    return launch_status();
}

template <int M, int RK>
int launch_small_n(const SmallParams& p, hipStream_t stream) {
    return p.n <= 2 ? launch_small_one<M, RK, true>(p, stream) : launch_small_one<M, RK, false>(p, stream);
}

template <int M>
int launch_small_rk(const SmallParams& p, int rk, hipStream_t stream) {
    switch (rk) {
        case kRandom: return launch_small_n<M, kRandom>(p, stream);
        case kGreedy: return launch_small_n<M, kGreedy>(p, stream);
        default: return launch_small_n<M, kAdjusted>(p, stream);
    }
}

}  // namespace sdgp

// Launch helpers of the stride-2 kernel; included by the files that instantiate it.
#pragma once

#include "bwd_stride2.h"

namespace sdgp {

template <int BN, int TM, int M, int RK, bool TAIL>
int launch_stride2_as(const Stride2Params& p, hipStream_t stream) {
    auto kern = bwd_stride2<BN, TM, M, RK, TAIL>;
    static const hipError_t attr =
        hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess) return SDGP_ERR_HIP;
    hipLaunchKernelGGL(kern, dim3(p.nblocks), dim3(kStride2Threads), (Stride2Layout<BN, TM>::total(p.npos, p.parts)), stream, p);
    return launch_status();
}

template <int BN, int TM, int M, int RK>
int launch_stride2_one(const Stride2Params& p, hipStream_t stream) {
    return p.C_out % kStride2KC != 0 ? launch_stride2_as<BN, TM, M, RK, true>(p, stream) : launch_stride2_as<BN, TM, M, RK, false>(p, stream);
}

template <int M>
int launch_stride2_rk(const Stride2Params& p, int shape, int rk, hipStream_t stream) {
    switch (rk) {
        case kRandom:
            return shape == 0 ? launch_stride2_one<128, 4, M, kRandom>(p, stream) : shape == 1 ? launch_stride2_one<128, 2, M, kRandom>(p, stream) : launch_stride2_one<64, 2, M, kRandom>(p, stream);
        case kGreedy:
            return shape == 0 ? launch_stride2_one<128, 4, M, kGreedy>(p, stream) : shape == 1 ? launch_stride2_one<128, 2, M, kGreedy>(p, stream) : launch_stride2_one<64, 2, M, kGreedy>(p, stream);
        default:
            return shape == 0 ? launch_stride2_one<128, 4, M, kAdjusted>(p, stream) : shape == 1 ? launch_stride2_one<128, 2, M, kAdjusted>(p, stream) : launch_stride2_one<64, 2, M, kAdjusted>(p, stream);
    }
}

}  // namespace sdgp

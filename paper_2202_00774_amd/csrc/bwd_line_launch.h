// Launch helpers of the line kernel; included by the files that instantiate it.
#pragma once

#include "bwd_line.h"

namespace sdgp {

template <int BN, int MODE, int M, int RK, bool TAIL, bool TWO>
int launch_line_as(const LineParams& p, hipStream_t stream) {
    if constexpr (MODE == 2 && BN == 128 && !line_has_128(M, RK, !TWO, TAIL)) {
        return 1;   // not built, and not asked for
    } else {
        auto kern = bwd_line<BN, MODE, M, RK, TAIL, TWO>;
        static const hipError_t attr =
            hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (attr != hipSuccess) return SDGP_ERR_HIP;
        hipLaunchKernelGGL(kern, dim3(p.nblocks), dim3(kLineThreads), (LineLayout<BN, MODE>::total(p.npos)), stream, p);
        return launch_status();
    }
}

// (one of m is rarer than two: one instantiation for all channel counts)
template <int BN, int M, int RK>
int launch_line_one(const LineParams& p, hipStream_t stream) {
    if (p.n == 1) return launch_line_as<BN, 2, M, RK, true, false>(p, stream);
    return p.C_out % kLineKC != 0 ? launch_line_as<BN, 2, M, RK, true, true>(p, stream) : launch_line_as<BN, 2, M, RK, false, true>(p, stream);
}

template <int M>
int launch_line_rk(const LineParams& p, int bn, int rk, hipStream_t stream) {
    switch (rk) {
        case kRandom: return bn == 128 ? launch_line_one<128, M, kRandom>(p, stream) : launch_line_one<64, M, kRandom>(p, stream);
        case kGreedy: return bn == 128 ? launch_line_one<128, M, kGreedy>(p, stream) : launch_line_one<64, M, kGreedy>(p, stream);
        default: return bn == 128 ? launch_line_one<128, M, kAdjusted>(p, stream) : launch_line_one<64, M, kAdjusted>(p, stream);
    }
}

// any n of m, with zeros (groups of 32 are never cut), on 64 columns: two workgroups a CU
template <int M, int RK>
int launch_line_masked_one(const LineParams& p, hipStream_t stream) {
    if constexpr (M < 32) {
        if (p.C_out % kLineKC != 0) return launch_line_as<64, 1, M, RK, true, false>(p, stream);
    }
    return launch_line_as<64, 1, M, RK, false, false>(p, stream);
}

template <int M>
int launch_line_masked_rk(const LineParams& p, int rk, hipStream_t stream) {
    switch (rk) {
        case kRandom: return launch_line_masked_one<M, kRandom>(p, stream);
        case kGreedy: return launch_line_masked_one<M, kGreedy>(p, stream);
        default: return launch_line_masked_one<M, kAdjusted>(p, stream);
    }
}

}  // namespace sdgp

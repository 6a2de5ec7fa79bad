// Launch helpers for the fp32 backward-data kernel; included by the files that instantiate it.
#pragma once

#include "bwd_f32.h"

namespace sdgp {

// tile shape (see launch_f32_shape) and number of workgroups along rows, columns and parity classes
struct F32Grid {
    int shape;
    unsigned x, y, z;
};

template <int M, int RK, bool NLE2, int CN, int WV, int WK>
int launch_f32_one(const F32Params& p, const F32Grid& g, hipStream_t stream) {
    hipLaunchKernelGGL((bwd_f32<M, RK, NLE2, CN, WV, WK>), dim3(g.x, g.y, g.z), dim3(64 * WV), 0, stream, p);
    return launch_status();
}

template <int M, int RK, bool NLE2>
int launch_f32_shape(const F32Params& p, const F32Grid& g, hipStream_t stream) {
    switch (g.shape) {
        case 0: return launch_f32_one<M, RK, NLE2, 4, 4, 1>(p, g, stream);
        case 1: return launch_f32_one<M, RK, NLE2, 2, 4, 1>(p, g, stream);
        default: return launch_f32_one<M, RK, NLE2, 2, 8, 8>(p, g, stream);
    }
}

template <int M, int RK>
int launch_f32_n(const F32Params& p, const F32Grid& g, hipStream_t stream) {
    if constexpr (M >= 16) {   // (the ranker of smaller fp32 groups is the same for every n)
        if (p.n <= 2) return launch_f32_shape<M, RK, true>(p, g, stream);
    }
    return launch_f32_shape<M, RK, false>(p, g, stream);
}

template <int M>
int launch_f32_rk(const F32Params& p, const F32Grid& g, int rk, hipStream_t stream) {
    switch (rk) {
        case kRandom: return launch_f32_n<M, kRandom>(p, g, stream);
        case kGreedy: return launch_f32_n<M, kGreedy>(p, g, stream);
        default: return launch_f32_n<M, kAdjusted>(p, g, stream);
    }
}

}  // namespace sdgp

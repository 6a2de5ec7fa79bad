// Instantiates the fp32 backward-data kernel for groups of 4 channels and for the dense product.
#include "bwd_f32_launch.h"
namespace sdgp {
int launch_f32_dense(const F32Params& p, const F32Grid& g, hipStream_t stream) {
    return launch_f32_shape<4, kDenseRanker, true>(p, g, stream);
}
int launch_f32_m4(const F32Params& p, const F32Grid& g, int rk, hipStream_t stream) {
    return launch_f32_rk<4>(p, g, rk, stream);
}
}  // namespace sdgp

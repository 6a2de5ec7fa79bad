// Instantiates the fp32 backward-data kernel for groups of 32 channels.
#include "bwd_f32_launch.h"
namespace sdgp {
int launch_f32_m32(const F32Params& p, const F32Grid& g, int rk, hipStream_t stream) {
    return launch_f32_rk<32>(p, g, rk, stream);
}
}  // namespace sdgp

// Instantiates the stride-2 kernel for n <= 2 of m = 16.
#include "bwd_stride2_launch.h"
namespace sdgp {
int launch_stride2_m16(const Stride2Params& p, int shape, int rk, hipStream_t stream) { return launch_stride2_rk<16>(p, shape, rk, stream); }
}  // namespace sdgp

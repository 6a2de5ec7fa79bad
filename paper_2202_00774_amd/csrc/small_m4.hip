// Instantiates the small-problem backward-data kernel for groups of 4 channels and for the dense product.
#include "bwd_small_launch.h"
namespace sdgp {
int launch_small_dense(const SmallParams& p, hipStream_t stream) { return launch_small_one<4, kSmallDense, true>(p, stream); }
int launch_small_m4(const SmallParams& p, int rk, hipStream_t stream) { return launch_small_rk<4>(p, rk, stream); }
}  // namespace sdgp

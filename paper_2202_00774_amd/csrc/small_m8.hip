// Instantiates the small-problem backward-data kernel for groups of 8 channels.
#include "bwd_small_launch.h"
namespace sdgp {
int launch_small_m8(const SmallParams& p, int rk, hipStream_t stream) { return launch_small_rk<8>(p, rk, stream); }
}  // namespace sdgp

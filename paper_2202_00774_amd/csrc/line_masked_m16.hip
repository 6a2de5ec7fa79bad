// Instantiates the line kernel for any n of m = 16, the pruned gradient stored with zeros.
#include "bwd_line_launch.h"
namespace sdgp {
int launch_line_masked_m16(const LineParams& p, int rk, hipStream_t stream) { return launch_line_masked_rk<16>(p, rk, stream); }
}  // namespace sdgp

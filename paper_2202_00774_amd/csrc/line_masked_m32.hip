// Instantiates the line kernel for any n of m = 32, the pruned gradient stored with zeros.
#include "bwd_line_launch.h"
namespace sdgp {
int launch_line_masked_m32(const LineParams& p, int rk, hipStream_t stream) { return launch_line_masked_rk<32>(p, rk, stream); }
}  // namespace sdgp

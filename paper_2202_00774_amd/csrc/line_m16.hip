// Instantiates the line kernel for n <= 2 of m = 16.
#include "bwd_line_launch.h"
namespace sdgp {
int launch_line_m16(const LineParams& p, int bn, int rk, hipStream_t stream) { return launch_line_rk<16>(p, bn, rk, stream); }
}  // namespace sdgp

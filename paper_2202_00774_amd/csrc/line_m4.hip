// Instantiates the line kernel for n <= 2 of m = 4.
#include "bwd_line_launch.h"
namespace sdgp {
int launch_line_m4(const LineParams& p, int bn, int rk, hipStream_t stream) { return launch_line_rk<4>(p, bn, rk, stream); }
}  // namespace sdgp

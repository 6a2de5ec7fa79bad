// Instantiates the line kernel for n <= 2 of m = 8.
#include "bwd_line_launch.h"
namespace sdgp {
int launch_line_m8(const LineParams& p, int bn, int rk, hipStream_t stream) { return launch_line_rk<8>(p, bn, rk, stream); }
}  // namespace sdgp

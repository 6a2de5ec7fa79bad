// Instantiates the line kernel without pruning (n == m).
#include "bwd_line_launch.h"
namespace sdgp {
int launch_line_dense(const LineParams& p, hipStream_t stream) {
    return p.C_out % kLineKC != 0 ? launch_line_as<64, 0, 4, kGreedy, true, false>(p, stream) : launch_line_as<64, 0, 4, kGreedy, false, false>(p, stream);
}
}  // namespace sdgp

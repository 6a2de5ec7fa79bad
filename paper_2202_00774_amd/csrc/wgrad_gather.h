// Weight gradient on the matrix cores for any filter and stride: plan and launch (wgrad_gather.hip).
#pragma once

#include "common.h"

namespace sdgp {

struct WgradGatherPlan {
    bool ok;
    int shape;
    int64_t kblocks, cblocks, nsplit, per;
};

WgradGatherPlan wgrad_gather_plan(int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out, int R, int S, int stride,
                                  int pad, int dt);

// out: dW when the plan has one split, room for nsplit partial filters otherwise.  D and dO 16-byte aligned.
int wgrad_gather_launch(const WgradGatherPlan& pl, const void* D, const void* dO, float* out, int64_t B, int64_t H, int64_t Wd,
                        int64_t C_in, int64_t C_out, int R, int S, int stride, int pad, hipStream_t stream);

}  // namespace sdgp

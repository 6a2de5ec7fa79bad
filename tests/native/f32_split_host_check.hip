// Host build of what the planner of the fp32 products on the bf16 matrix instructions and its first pass share
// (csrc/bwd_f32_split.h, csrc/bwd_f32_split_tiles.h).
//   * class_slots, slot_tap: every slot of every filter up to 11 x 11 at strides 1 to 4 is the tap that the product, walking a
//     class's taps row by row from the class's first slot on, takes it for (Fig. 3: dD's pixels of one parity class meet the
//     taps r0, r0 + stride, ... of each axis), every tap has one slot, and no slot lies outside the filter.
//   * grid_side: never below one, and no position fewer than the taps reach.
//   * the planner declines launches of 2^32 threads and more.
// Prints one line per check and returns the number of mismatches.  Test infrastructure, not product code.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstring>

#include "bwd_f32_split_tiles.h"

using namespace sdgp;

static int check_slots() {
    int bad = 0;
    for (int R = 1; R <= 11; ++R)
        for (int S = 1; S <= 11; ++S)
            for (int stride = 1; stride <= 4; ++stride) {
                int slot0[16] = {}, seen[121] = {}, slots = 0;
                class_slots(R, S, stride, slot0);
                for (int r0 = 0; r0 < stride; ++r0)
                    for (int s0 = 0; s0 < stride; ++s0) {
                        int slot = slot0[r0 * stride + s0];
                        for (int r = r0; r < R; r += stride)
                            for (int s = s0; s < S; s += stride, ++slot, ++slots) {
                                int gr = -1, gs = -1;
                                slot_tap(slot0, R, S, stride, slot, gr, gs);
                                if (slot < 0 || slot >= R * S || gr != r || gs != s) ++bad;
                                else ++seen[slot];
                            }
                    }
                if (slots != R * S) ++bad;
                for (int i = 0; i < R * S; ++i) bad += seen[i] != 1;
            }
    printf("slots: mismatches %d\n", bad);
    return bad;
}

static int check_sides() {
    int bad = 0;
    for (int side = 1; side <= 256; ++side)
        for (int count = 0; count <= 11; ++count) bad += grid_side(side, count) < 1 || grid_side(side, count) < side + count - 1;
    printf("sides: mismatches %d\n", bad);
    return bad;
}

static int check_limits() {
    SplitPlan s;
    int bad = 0;
    for (int64_t B = (1 << 22) - 2; B <= 1 << 22; ++B) {   // one tile of 256 rows an image, 1024 threads each
        const bool takes = split_plan(s, B, 16, 16, 33, 16, 1, 1, 1, 0, 4, 4);
        bad += takes != (B < 1 << 22) || (takes && (s.rows != 256 || s.p.nblocks != B));
    }
    printf("limits: mismatches %d\n", bad);
    return bad;
}

int main() {
    const int total = check_slots() + check_sides() + check_limits();
    printf("total mismatches %d\n", total);
    return total != 0;
}

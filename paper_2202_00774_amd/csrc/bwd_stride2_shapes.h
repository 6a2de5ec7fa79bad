// Tile shapes of the stride-2 kernel: what one costs, and which one a layer gets.  Host code only.
#pragma once

#include "bwd_stride2.h"

namespace sdgp {

struct Stride2Shape {
    int bn, rows, npos, lds;
    int64_t blocks;
    double time;
};

constexpr int kStride2Lds = 160 * 1024;

template <int BN, int TM>
Stride2Shape stride2_shape(int64_t pixels, int P, int Q, int64_t C_in, int parts) {
    using L = Stride2Layout<BN, TM>;
    Stride2Shape s;
    s.bn = BN, s.rows = L::kRows, s.npos = L::positions(P, Q), s.lds = L::total(s.npos, parts);
    s.blocks = (pixels + s.rows - 1) / s.rows * ((C_in + BN - 1) / BN);
    // Time in units of a workgroup of 256 positions and 128 columns beside another one; one of half the size takes 0.7 of that, one
    // alone on its CU loses a third of the CU, a third one gains 15 percent.  (131 layers: 1.03 times the best shape's time; always
    // the first shape 1.27, the second 1.07, the third 1.10.)
    const int most = (int)(kStride2Lds / s.lds), per_cu = most < (TM == 4 ? 2 : 3) ? most : (TM == 4 ? 2 : 3);
    constexpr double kBeside[4] = {0.0, 1.5, 1.0, 0.85};
    if (per_cu < 1) {   // does not fit a CU at all
        s.time = 1e300;
        return s;
    }
    const int64_t round = 256 * per_cu, rest = s.blocks % round;
    const int left = (int)((rest + 255) / 256);
    s.time = (TM == 4 ? 1.0 : 0.7) * ((double)(s.blocks / round) * per_cu * kBeside[per_cu] + left * kBeside[left]);
    return s;
}

// The fastest of the three shapes whose LDS stays within `lds` bytes: its number, or -1, and the shape.
inline int stride2_choose(int64_t pixels, int P, int Q, int64_t C_in, int parts, int lds, Stride2Shape& chosen) {
    const Stride2Shape shapes[3] = {stride2_shape<128, 4>(pixels, P, Q, C_in, parts), stride2_shape<128, 2>(pixels, P, Q, C_in, parts),
                                    stride2_shape<64, 2>(pixels, P, Q, C_in, parts)};
    int best = -1;
    for (int i = 0; i < 3; ++i)
        if (shapes[i].lds <= lds && (best < 0 || shapes[i].time < shapes[best].time)) best = i;
    if (best >= 0) chosen = shapes[best];
    return best;
}

// Whether the parity-class kernel is the faster one for a layer that it would take, ranking the gradient ahead (`ahead`, in a pass of its
// own) or once per tap.
//   * Less than a workgroup for every CU here (its classes are four workgroups: 32 <- 64 at 10x10, batch 452, 10.3 us against 12.9).
//   * 192 channels and more, ranked ahead there, on little more than a workgroup a CU (256 <- 192 at 17x17, batch 233, 28 against 31) or
//     with half of the columns empty (64 <- 192 at 25x25, batch 484, 45 against 50).  More than 224 never fit two workgroups on a CU.
//   * Small images of odd sides: all four classes are computed for every position, and at 3x3 nine of the sixteen pixels exist, 0.44 of
//     the products; the classes have what exists.  128 channels and more, ranked ahead there, and less than 5/8 of the products needed
//     (3x3, 3x5, 3x7, 5x5): 0.87 of this kernel's time over 186 layers (448 <- 128 at 3x3, batch 11004, 44 against 66).  With 64
//     channels, or from 5x7 on, this one is faster: 0.89 over 319 layers, 0.94 over 48.
inline bool stride2_classes_faster(bool ahead, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out, int64_t blocks) {
    if (C_out > 224 || (C_out >= 192 && C_in <= 64) || blocks < (C_out >= 192 ? 320 : 256)) return true;
    const int64_t P = (H + 1) / 2, Q = (Wd + 1) / 2;
    const int64_t needed = (2 * (H / 2) + P) * (2 * (Wd / 2) + Q), computed = 9 * P * Q;   // taps times pixels of an image
    return ahead && C_out >= 128 && 8 * needed < 5 * computed;
}

}  // namespace sdgp

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

}  // namespace sdgp

// Which tile of the line kernel a layer gets.  Host code only.
#pragma once

#include "bwd_line.h"

namespace sdgp {

constexpr int kLineLdsPair = 80 * 1024;   // more than this leaves one workgroup on a CU

// LDS bytes of a workgroup; mode and columns as in bwd_line.
inline int line_lds(int mode, int bn, int H, int Wd) {
    const int npos = line_positions(H, Wd);
    if (mode != 2) return LineLayout<64, 0>::total(npos);
    return bn == 128 ? LineLayout<128, 2>::total(npos) : LineLayout<64, 2>::total(npos);
}

// Columns of a tile for n <= 2.  What decides is how many workgroups the fullest CU gets: one of 128 columns takes about 1.7 times as long as
// one of 64, which ranks the same pixels (94 layers of more than 64 input channels: 1.2 percent above the better of the two, at most
// 15; always 64 columns 4.8 and 33 percent, always 128 10 and 59).  3x3 224 <- 192 at 34x34, batch 82, 2:8 Rescaled 64 us on 128
// columns and 86 on 64; 128 <- 96 at 9x9, batch 301, 2:4 Rescaled 14.6 and 11.9.
//   * 1.9 times where the LDS leaves one workgroup of 128 columns on a CU but two of 64 -- images 61 to 63 pixels wide, and of few lines:
//     1124 layers 0.3 percent above the better of the two, at most 15 (by 1.7 times 1.1 and 29: 432 <- 240 at 62x62, batch 15, 2:8 Random
//     145 us on 128 columns, 118 on 64; 2.0 times 1.9 and 25).
//   * Always 64 where the magnitude rankers that sort keys would have no registers left: line_has_128
//     (448 <- 128 at 27x27, batch 60, 1:4 Magnitude 56 us, 41 on 64 columns; 368 <- 272 at 22x22, batch 62, 2:16 79 and 54).
//   * The random ranker spills there too (5 to 16 registers), but where this rule picks 128 columns they are still the faster ones: 0.91
//     of the time of 64 over 78 layers, 0.95 over 33 whose last chunk is cut.
inline int tile_columns(int64_t row_tiles, int H, int Wd, int64_t C_in, int64_t C_out, int n, int m, int rk) {
    if (C_in <= 64 || !line_has_128(m, rk, n == 1, C_out % kLineKC != 0)) return 64;
    const bool alone = line_lds(2, 128, H, Wd) > kLineLdsPair && line_lds(2, 64, H, Wd) <= kLineLdsPair;
    const int64_t per_cu_64 = (row_tiles * ((C_in + 63) / 64) + 255) / 256, per_cu_128 = (row_tiles * ((C_in + 127) / 128) + 255) / 256;
    return per_cu_128 * (alone ? 19 : 17) < per_cu_64 * 10 ? 128 : 64;
}

// The whole gradient of an image of few lines (zeros between the lines and images: 1x1 to 3x3, one or two lines, one column) leaves one
// workgroup of the line kernel on a CU; so do images 58 to 63 pixels wide.
inline bool line_alone(int H, int Wd) { return line_lds(0, 64, H, Wd) > kLineLdsPair; }

// A round of 256 workgroups of rows x bn of the row kernel, in rounds of a line kernel that has the CUs to itself (mode 0 or 1).
inline double row_round(int mode, int m, int rows, int bn) {
    if (mode == 0) return rows == 256 ? (bn == 64 ? 1.1 : 1.8) : (bn == 64 ? 1.85 : 3.0);
    if (rows == 256) return bn == 64 ? 1.2 : 1.75;
    return bn == 64 && m != 32 ? 1.75 : 2.1;
}

// Whether the row kernel, planned with `blocks` tiles of rows x bn, is faster than a line kernel alone on its CUs with `line_blocks`
// workgroups.  With row_worth_planning, over images of few lines: 600 unpruned layers 1.4 percent above the better of the two (line kernel
// only 3.8; 512 <- 64 at 1x1, batch 95360, 85 us, 57 on the row kernel), 600 of general n:m 0.4 (0.6; 56 <- 152 at 2x2, batch 63185, 4:8, 80
// and 66).  On wide images it gained nothing over the line kernel, which is 0.4 and 0.5 percent above the better one there (643 layers).
inline bool row_faster_than_lone_line(int mode, int m, int64_t blocks, int rows, int bn, int64_t line_blocks) {
    return (double)((blocks + 255) / 256) * row_round(mode, m, rows, bn) < (double)((line_blocks + 255) / 256);
}

// Whether a layer is worth planning for the row kernel to find that out: an image of few lines, no fewer tiles than without any waste
// faster, and a search (7 us for 1x56, 25 for 600x1, 2 for 3x3) that the call hides: a round is 7 us and more.
inline bool row_worth_planning(int mode, int m, int64_t pixels, int64_t H, int64_t Wd, int64_t C_in, int64_t line_blocks) {
    if (mode == 2 || H < 1 || Wd < 1 || Wd > 56 || !line_alone((int)H, (int)Wd)) return false;
    if (H * Wd > 16 && line_blocks <= 5 * 256) return false;
    for (int rows = 256; rows <= 512; rows *= 2)
        for (int bn = 64; bn <= 128; bn *= 2)
            if (row_faster_than_lone_line(mode, m, (pixels + rows - 1) / rows * ((C_in + bn - 1) / bn), rows, bn, line_blocks)) return true;
    return false;
}

}  // namespace sdgp

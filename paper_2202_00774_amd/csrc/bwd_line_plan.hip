// Host side of the line kernel: 3x3 stride-1 layers with one pixel of padding, pruned by n of m in {4, 8, 16, 32} or not at all, on
// images up to 63 pixels wide.
#include <climits>

#include "bwd_line_choice.h"

namespace sdgp {

int launch_line_m4(const LineParams& p, int bn, int rk, hipStream_t stream);
int launch_line_m8(const LineParams& p, int bn, int rk, hipStream_t stream);
int launch_line_m16(const LineParams& p, int bn, int rk, hipStream_t stream);
int launch_line_masked_m4(const LineParams& p, int rk, hipStream_t stream);
int launch_line_masked_m8(const LineParams& p, int rk, hipStream_t stream);
int launch_line_masked_m16(const LineParams& p, int rk, hipStream_t stream);
int launch_line_masked_m32(const LineParams& p, int rk, hipStream_t stream);
int launch_line_dense(const LineParams& p, hipStream_t stream);

// SDGP_OK after launching, a positive value when the problem does not fit, or a negative sdgp_status.
int bwd_line_launch(const void* dO, const void* W, void* dD, int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out, int R, int S,
                    int stride, int pad, int n, int m, int rk, uint64_t seed, hipStream_t stream) {
    if (R != 3 || S != 3 || stride != 1 || pad != 1) return 1;
    const int mode = n == m ? 0 : n <= 2 && (m == 4 || m == 8 || m == 16) ? 2 : 1;
    if (mode != 0 && m != 4 && m != 8 && m != 16 && m != 32) return 1;
    if (C_out < 8 || (C_out % 8) != 0 || (mode != 0 && (C_out % m) != 0) || (C_in % 8) != 0) return 1;
    if (!is_aligned16(dO) || !is_aligned16(W) || !is_aligned16(dD)) return 1;
    if (Wd > kLineMaxWidth) return 1;   // wider: the three items a lane has do not cover a tile's window (bwd_row takes them)
    const int64_t pixels = B * H * Wd;
    // (the random ranker's sixteen channels of a short chunk must not straddle a carry into the index's high word)
    if (rk == kRandom && mode != 0 && C_out % 16 != 0 && pixels > (int64_t)0xFFFFFFFFu / C_out) return 1;
    // a position of the padded line is below four times the pixel's number; offsets into W are counted in 32 bits
    if (pixels >= (1 << 28) || 9 * C_in >= (1 << 24) || C_out * 9 * C_in >= (1 << 30) || C_out > (1 << 20)) return 1;
    LineParams p{};
    p.dO = static_cast<const uint16_t*>(dO);
    p.W = static_cast<const uint16_t*>(W);
    p.dD = static_cast<uint16_t*>(dD);
    p.pixels = (int)pixels, p.H = (int)H, p.Wd = (int)Wd, p.C_out = (int)C_out, p.C_in = (int)C_in;
    p.by_line = fast_div((uint32_t)Wd), p.by_image = fast_div((uint32_t)H);
    p.w_row = 9 * (int)C_in;
    p.n = n;
    p.mix = seed_mix(seed);
    const int64_t row_tiles = (pixels + kLineRows - 1) / kLineRows;
    // (the whole gradient takes twice the LDS of the compressed one: 128 columns leave one workgroup on a CU, 1.3 times the time over 60
    // unpruned layers)
    const int bn = mode == 2 ? tile_columns(row_tiles, (int)H, (int)Wd, C_in, C_out, n, m, rk) : 64;
    p.npos = line_positions((int)H, (int)Wd);
    p.ntiles_n = (int)((C_in + bn - 1) / bn);
    const int64_t blocks = row_tiles * p.ntiles_n;
    if (blocks >= INT_MAX / kLineThreads) return 1;
    p.nblocks = (int)blocks;
    if (mode == 0) return launch_line_dense(p, stream);
    if (mode == 1) {
        if (m == 4) return launch_line_masked_m4(p, rk, stream);
        if (m == 8) return launch_line_masked_m8(p, rk, stream);
        if (m == 16) return launch_line_masked_m16(p, rk, stream);
        return launch_line_masked_m32(p, rk, stream);
    }
    if (m == 4) return launch_line_m4(p, bn, rk, stream);
    if (m == 8) return launch_line_m8(p, bn, rk, stream);
    return launch_line_m16(p, bn, rk, stream);
}

}  // namespace sdgp

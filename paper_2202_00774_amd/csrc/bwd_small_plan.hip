// Planner of the small-problem backward-data kernel.
#include "bwd_small.h"

namespace sdgp {

int launch_small_dense(const SmallParams& p, hipStream_t stream);
int launch_small_m4(const SmallParams& p, int rk, hipStream_t stream);
int launch_small_m8(const SmallParams& p, int rk, hipStream_t stream);
int launch_small_m16(const SmallParams& p, int rk, hipStream_t stream);
int launch_small_m32(const SmallParams& p, int rk, hipStream_t stream);

// A positive value: the problem does not fit, or is one for the other kernels.
int bwd_small_launch(const void* dO, const void* W, void* dD, int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out,
                     int R, int S, int stride, int pad, int n, int m, int rk, uint64_t seed, hipStream_t stream) {
    const bool dense = n == m;
    if (!dense && m != 4 && m != 8 && m != 16 && m != 32) return 1;
    if (C_out < 8 || C_out % 8 != 0 || C_in < 8 || C_in % 8 != 0 || C_out > (1 << 20) || C_in > (1 << 20)) return 1;
    if (!is_aligned16(dO) || !is_aligned16(W) || !is_aligned16(dD)) return 1;
    if (B < 1 || H < 1 || Wd < 1 || B > (1 << 24) || H > (1 << 24) || Wd > (1 << 24)) return 1;
    const int64_t P = (H + 2 * pad - R) / stride + 1, Q = (Wd + 2 * pad - S) / stride + 1;
    const int64_t rows = B * ((H + stride - 1) / stride) * ((Wd + stride - 1) / stride);   // of the largest parity class
    const int64_t row_tiles = (rows + kSmallRows - 1) / kSmallRows, col_tiles = (C_in + kSmallCols - 1) / kSmallCols;
    // pixel indices and offsets within the filter in 32 bits, channels of the step past the last one included
    if (B * (P + 16) * (Q + 16) > (1 << 30) || B * H * Wd > (1 << 30) || (int64_t)R * S * C_in > (1 << 28)) return 1;
    // Up to 256 tiles, one per compute unit, nothing else fills the chip (us, other kernel / this one: linear 256 x 1000 ->
    // 2048 64 / 11.6, 1024 x 1024 -> 1024 58 / 12; 3x3 128 -> 128 at 16x16, batch 32 33 / 14).  Beyond that it is a question of who
    // else takes the problem:
    //   strided filters: the parity classes of the pointwise kernel want 1024 of these tiles; until then bwd_tiled (3x3 512
    //     -> 256 at 7x7, batch 100 39 / 29; 784 tiles of 128 -> 128 at 28x28, batch 32 25.3 / 24.6);
    //   1x1: the pointwise kernel from 257 tiles on, which a long reduction on that few workgroups makes the slower one
    //     (2048 x 2048 -> 1024 50 / 36, 2048 x 512 -> 1024 11 / 14); where C_out is no multiple of its chunk bwd_tiled (2048 x
    //     1000 -> 2048 84 / 43; 4096 rows 85 / 81);
    //   other filters: the row kernel from 512 tiles on (256 -> 256 at 16x16, batch 32 29 / 36), bwd_conv3 and bwd_tiled
    //     before it (512 -> 512 at 7x7, batch 64 69 / 59).
    const int64_t tiles = row_tiles * col_tiles * stride * stride;
    const bool whole_chunks = C_out % 32 == 0;
    const int64_t most = stride > 1 ? 1023 : R == 1 && S == 1 ? (!whole_chunks ? 1024 : C_out >= 1024 ? 512 : 256) : 511;
    if (tiles > most) return 1;
    SmallParams p;
    p.dO = static_cast<const uint16_t*>(dO), p.W = static_cast<const uint16_t*>(W), p.dD = static_cast<uint16_t*>(dD);
    p.B = B, p.H = (int)H, p.Wd = (int)Wd, p.P = (int)P, p.Q = (int)Q, p.C_in = (int)C_in, p.C_out = (int)C_out;
    p.R = R, p.S = S, p.stride = stride, p.pad = pad, p.n = n, p.mix = seed_mix(seed);
    p.col_tiles = (int)col_tiles, p.row_tiles = (int)row_tiles;
    if (dense) return launch_small_dense(p, stream);
    switch (m) {
        case 4: return launch_small_m4(p, rk, stream);
        case 8: return launch_small_m8(p, rk, stream);
        case 16: return launch_small_m16(p, rk, stream);
        default: return launch_small_m32(p, rk, stream);
    }
}

}  // namespace sdgp

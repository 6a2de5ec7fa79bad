// Host side of the stride-2 kernel: 3x3 layers of stride 2 with one pixel of padding and n <= 2 of m in {4, 8, 16} whose ranked
// gradient fits into LDS.
#include <climits>

#include "bwd_stride2_shapes.h"

namespace sdgp {

int launch_stride2_m4(const Stride2Params& p, int shape, int rk, hipStream_t stream);
int launch_stride2_m8(const Stride2Params& p, int shape, int rk, hipStream_t stream);
int launch_stride2_m16(const Stride2Params& p, int shape, int rk, hipStream_t stream);

// SDGP_OK after launching, a positive value when the problem does not fit, or a negative sdgp_status.
// classes: 1 if the parity-class kernel would take the problem, ranking per tap, 2 if it would with the gradient ranked ahead, 0 if not.
// That kernel is also the faster one where the ranked gradient leaves one workgroup on a CU here (384 <- 256 at 40x40, batch 61, 61 us
// against 85).  Above these lines 150 layers took 0.78 of its time, the slowest 1.04.  Against what takes the others (bwd_tiled) one
// workgroup on a CU is still the faster way: 0.53 to 0.96.
int bwd_stride2_launch(int classes, const void* dO, const void* W, void* dD, int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out,
                       int R, int S, int stride, int pad, int n, int m, int rk, uint64_t seed, hipStream_t stream) {
    if (R != 3 || S != 3 || stride != 2 || pad != 1 || n == m || n > 2 || (m != 4 && m != 8 && m != 16)) return 1;
    if (C_out < 8 || (C_out % 8) != 0 || (C_out % m) != 0 || (C_in % 8) != 0) return 1;
    if (!is_aligned16(dO) || !is_aligned16(W) || !is_aligned16(dD)) return 1;
    // (a pixel's number shares a word with three flags; offsets into W and into a tile's gradient are counted in 32 bits)
    if (H >= (1 << 20) || Wd >= (1 << 10) || C_out > (1 << 10) || C_in > (1 << 16) || B * H * Wd >= (1 << 28)) return 1;
    const int64_t P = (H + 1) / 2, Q = (Wd + 1) / 2, pixels = B * P * Q;
    // (the random ranker's sixteen channels of a short chunk must not straddle a carry into the index's high word)
    if (rk == kRandom && C_out % 16 != 0 && pixels > (int64_t)0xFFFFFFFFu / C_out) return 1;
    Stride2Params p{};
    p.parts = 2 * (int)((C_out + 31) / 32);
    Stride2Shape shape;
    const int best = stride2_choose(pixels, (int)P, (int)Q, C_in, p.parts, (classes != 0 ? 80 : 132) * 1024, shape);
    if (best < 0) return 1;
    if (classes != 0 && stride2_classes_faster(classes == 2, H, Wd, C_in, C_out, shape.blocks)) return 1;
    p.dO = static_cast<const uint16_t*>(dO);
    p.W = static_cast<const uint16_t*>(W);
    p.dD = static_cast<uint16_t*>(dD);
    p.pixels = (int)pixels, p.P = (int)P, p.Q = (int)Q, p.H = (int)H, p.Wd = (int)Wd, p.C_out = (int)C_out, p.C_in = (int)C_in;
    p.by_line = fast_div((uint32_t)Q), p.by_image = fast_div((uint32_t)P), p.by_parts = fast_div((uint32_t)p.parts);
    p.w_row = 9 * (int)C_in;
    p.n = n;
    p.mix = seed_mix(seed);
    p.npos = shape.npos;
    p.ntiles_n = (int)((C_in + shape.bn - 1) / shape.bn);
    if (shape.blocks >= INT_MAX / kStride2Threads) return 1;
    p.nblocks = (int)shape.blocks;
    if (m == 4) return launch_stride2_m4(p, best, rk, stream);
    if (m == 8) return launch_stride2_m8(p, best, rk, stream);
    return launch_stride2_m16(p, best, rk, stream);
}

}  // namespace sdgp

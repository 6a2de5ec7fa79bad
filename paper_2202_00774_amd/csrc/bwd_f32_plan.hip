// Planner of the fp32 backward-data kernel: which problems it takes and with which tile shape.
#include "bwd_f32_launch.h"

namespace sdgp {

int launch_f32_dense(const F32Params& p, const F32Grid& g, hipStream_t stream);
int launch_f32_m4(const F32Params& p, const F32Grid& g, int rk, hipStream_t stream);
int launch_f32_m8(const F32Params& p, const F32Grid& g, int rk, hipStream_t stream);
int launch_f32_m16(const F32Params& p, const F32Grid& g, int rk, hipStream_t stream);
int launch_f32_m32(const F32Params& p, const F32Grid& g, int rk, hipStream_t stream);

// A positive value: the problem does not fit (other group sizes, channel counts or pointers that 16-byte gradient loads
// and 8-byte weight loads do not suit, grids beyond the launch limits).
int bwd_f32_launch(const void* dO, const void* W, void* dD, int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out,
                   int R, int S, int stride, int pad, int n, int m, int rk, uint64_t seed, hipStream_t stream) {
    const bool dense = n == m;
    if (!dense && m != 4 && m != 8 && m != 16 && m != 32) return 1;
    if (C_out == 0 || C_out % 4 != 0 || C_out > (1 << 24) || C_in == 0 || C_in % 2 != 0 || C_in > (1 << 24)) return 1;
    // A 1x1 product of a handful of channels is all edge on tiles of 64 columns and steps of 16 channels; one thread an element
    // reads its few weights from the cache: this kernel's time over the plain one's, dense 4 -> 2 channels 1.24-2.40, 8 -> 2
    // 1.02-2.00, 4 -> 4 0.95-2.19, 4 -> 6 0.67-1.44, 8 -> 4 0.74-1.79; pruned 4 -> 2 1.02-1.99, 8 -> 2 0.72-1.45, 4 -> 4 0.66-1.79, 4 -> 6
    // 0.47-1.17, 16 -> 2 0.42-1.56.
    if (R == 1 && S == 1 && stride == 1 && C_in * C_out <= (dense ? 24 : 16)) return 1;
    // one image of the gradient and the filter are indexed with 32 bits, the zero half of an odd last step included
    const int64_t P = (H + 2 * pad - R) / stride + 1, Q = (Wd + 2 * pad - S) / stride + 1;
    const int64_t reach = (int64_t)1 << 30;
    if (H > (1 << 24) || Wd > (1 << 24) || P * Q > reach / (C_out + 64) || (int64_t)R * S * C_in > reach / (C_out + 64)) return 1;
    if (!is_aligned16(dO) || !is_aligned16(W) || !is_aligned16(dD)) return 1;
    const int64_t rows = B * ((H + stride - 1) / stride) * ((Wd + stride - 1) / stride);   // of the largest parity class
    const int64_t tiles = (rows + 31) / 32;
    if (B == 0 || tiles > (1 << 25)) return 1;   // (a launch holds fewer than 2^32 threads)
    // One wavefront per SIMD (1024 of them) is the least that fills the matrix units.  Tiles of 128 columns read a
    // gradient row half as often as tiles of 64; with too few of either the eight wavefronts of a workgroup share a tile
    // and split the reduction.  Measured (us, 128 columns / 64 columns / shared): 3x3 128 -> 128 at 16x16, batch 128
    // 99 / 112 / 120; 64 -> 128 channels at 32x32, batch 64 179 / 112 / 120; batch 32 of the first 96 / 65 / 35.
    const int64_t classes = (int64_t)stride * stride;
    const int64_t wide = tiles * ((C_in + 127) / 128) * classes, slim = tiles * ((C_in + 63) / 64) * classes;
    F32Grid g;
    g.shape = C_in > 64 && C_in % 4 == 0 && wide >= 1024 ? 0 : slim >= 1024 ? 1 : 2;
    const int64_t gx = g.shape == 2 ? tiles : (tiles + 3) / 4, gy = g.shape == 0 ? (C_in + 127) / 128 : (C_in + 63) / 64;
    if (gy > 65535) return 1;
    g.x = (unsigned)gx, g.y = (unsigned)gy, g.z = (unsigned)classes;
    F32Params p;
    p.dO = static_cast<const float*>(dO), p.W = static_cast<const float*>(W), p.dD = static_cast<float*>(dD);
    p.B = B, p.H = H, p.Wd = Wd, p.C_in = C_in, p.C_out = C_out;
    p.P = P, p.Q = Q;
    p.R = R, p.S = S, p.stride = stride, p.pad = pad, p.n = n, p.mix = seed_mix(seed);
    if (dense) return launch_f32_dense(p, g, stream);
    switch (m) {
        case 4: return launch_f32_m4(p, g, rk, stream);
        case 8: return launch_f32_m8(p, g, rk, stream);
        case 16: return launch_f32_m16(p, g, rk, stream);
        default: return launch_f32_m32(p, g, rk, stream);
    }
}

}  // namespace sdgp

// Planner of the fp32 backward-data products on the bf16 matrix instructions: which problems, which tiles, what the
// workspace holds.  (Host code, apart from the launcher so that it can be checked without a GPU.)
#pragma once

#include <algorithm>

#include "bwd_f32_split.h"

namespace sdgp {

struct SplitPlan {
    SplitParams p;
    bool sparse;
    int rows, np;   // of the product's tile; np: grid positions the kernel variant holds
    size_t bytes;   // workspace
    size_t off_idx, off_wimg, off_wnotes, off_gnotes;
};

inline size_t split_align(size_t x) { return (x + 255u) & ~(size_t)255u; }

// Tile sides worth a look on an axis of n pixels, longest first: the shortest for every number of tiles.  Beside a short other
// axis all of them: a longer side makes another count of images to halve, there sometimes a better one.
struct SplitSides {
    int count;
    int side[256], tiles[256];
};
inline void split_sides(SplitSides& s, int64_t n, int64_t other) {
    s.count = 0;
    for (int side = (int)std::min<int64_t>(n, 256); side >= 1; --side) {
        const int tiles = (int)((n + side - 1) / side);
        if (other > 8) side = (int)((n + tiles - 1) / tiles);
        s.side[s.count] = side, s.tiles[s.count++] = tiles;
    }
}

// The tiles of `rows` rows on grids of at most `np` positions that take the fewest steps: rows times taps and grid positions,
// of all tiles.  Their number, 0 when nothing fits.  (On the host, in every call: trying every side took 10 to 40 us.)
inline int64_t split_tiles(SplitPlan& s, int rows, int np, int64_t B, const SplitSides& hs, const SplitSides& ws, int ny, int nx) {
    SplitParams& p = s.p;
    double best = 1e300;
    int64_t tiles = 0;
    for (int j = 0; j < ws.count; ++j)
        for (int i = 0; i < hs.count; ++i) {
            const int area = hs.side[i] * ws.side[j], grid = (hs.side[i] + ny - 1) * (ws.side[j] + nx - 1);
            if (area > rows || grid > np) continue;
            const double each = (double)hs.tiles[i] * ws.tiles[j];
            if ((double)B * each * (area * (double)(ny * nx) + grid) >= best) continue;   // with full tiles
            int TB = (int)std::min<int64_t>(B, rows / area);
            while (TB * grid > np) TB /= 2;
            const int64_t tb = (B + TB - 1) / TB;
            const double cost = (double)tb * each * (rows * (double)(ny * nx) + (double)(TB * grid));
            if (cost < best) {
                best = cost, tiles = tb * hs.tiles[i] * ws.tiles[j];
                p.TB = TB, p.TH = hs.side[i], p.TW = ws.side[j], p.tiles_h = hs.tiles[i], p.tiles_w = ws.tiles[j];
                s.rows = rows, s.np = np;
            }
        }
    return tiles;
}

// Estimates (us) of this path and of the fp32 matrix instruction's (bwd_f32), which share what decides: rounds of workgroups
// or wavefronts over the chip times the steps of one.  Fitted to both paths' times on 330 convolutions of 16 to 512 channels,
// images of 4 to 32 pixels, batches of 10 to 128, filters 1x1 and 3x3, strides 1 and 2, every pattern: 14 and 20 percent
// rms.  Taking this path where it is estimated a tenth faster loses 1 percent on average against the faster of both on
// those, 11 percent once; 3x3 384 -> 224 channels at 18x18, batch 17, 1:4 182 -> 65 us, 416 -> 96 at 15x15, batch 19, 4:32 248 -> 58,
// and what stays: 64 -> 384 at 14x14, batch 20, dense 42 (81 here), 1x1 160 -> 480 at 4x4, batch 59 9.8 (22).
struct SplitEstimates {
    double split, plain;
};
inline SplitEstimates split_estimate(const SplitPlan& s, int64_t tiles, int m) {
    const SplitParams& p = s.p;
    const int64_t classes = (int64_t)p.stride * p.stride, h = (p.H + p.stride - 1) / p.stride, w = (p.Wd + p.stride - 1) / p.stride;
    const int64_t rows = p.B * h * w, row_tiles = (rows + 31) / 32;
    const int group = s.sparse ? (s.np > 384 ? 1 : 2) : 3;
    const int64_t wide = row_tiles * ((p.C_in + 127) / 128) * classes, slim = row_tiles * ((p.C_in + 63) / 64) * classes;
    const int shape = p.C_in > 64 && p.C_in % 4 == 0 && wide >= 1024 ? 0 : slim >= 1024 ? 1 : 2;   // as bwd_f32 chooses
    const bool dense = p.n == m;
    const int64_t ch = !dense && m > 8 ? m : 8, pairs = (p.C_out + 2 * ch - 1) / (2 * ch);
    double taps = 0, stages = 0, steps = 0;   // a workgroup's, a wavefront's, summed over the classes
    for (int i = 0; i < classes; ++i) {
        const int r0 = i / p.stride, s0 = i % p.stride;
        const int64_t t = (int64_t)(r0 < p.R ? (p.R - r0 + p.stride - 1) / p.stride : 0) * (s0 < p.S ? (p.S - s0 + p.stride - 1) / p.stride : 0);
        taps += (double)(t * p.nchunks);
        stages += (double)((t + group - 1) / group * p.nchunks);
        steps += (double)(shape == 2 ? (t * pairs + 7) / 8 : t * pairs);
    }
    const double here = (double)((tiles * p.ntiles_n * classes + 255) / 256) / (double)classes;
    SplitEstimates e;
    e.split = 6.8 + here * ((s.rows == 256 ? 0.44 : 0.02) * taps + 1.02 * stages + 3.1 * (double)classes) + 1.76e-6 * (double)p.npix * p.C_out;
    const double rounds = shape == 0 ? (double)((wide + 1023) / 1024) : shape == 1 ? (double)((slim + 1023) / 1024) : (double)((slim + 255) / 256);
    const double ranking = dense || m < 16 ? 1.0 : m == 16 ? 1.47 : 2.34;
    e.plain = 4.0 + rounds * (steps / (double)classes * (double)ch * (shape == 1 ? 0.099 : 0.196) * ranking + 1.25) + 0.227e-6 * (double)rows * p.C_in;
    // odd widths would go to one thread an element: 20 ms for 4.8e9 products
    if (p.C_in % 2 != 0) e.plain = 4.0 + 4.2e-6 * (double)p.B * p.H * p.Wd * p.C_in * p.R * p.S * p.C_out / (double)classes;
    return e;
}

inline bool split_plan(SplitPlan& s, int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out, int R, int S, int stride, int pad, int n, int m) {
    const bool dense = n == m;
    if (!dense && m != 4 && m != 8 && m != 16 && m != 32) return false;
    if (B < 1 || C_out < 16 || C_out % 4 != 0 || C_in < 32 || H < 1 || Wd < 1) return false;
    const int64_t P = (H + 2 * pad - R) / stride + 1, Q = (Wd + 2 * pad - S) / stride + 1;
    const int64_t limit = (int64_t)1 << 30;
    if (P < 1 || Q < 1 || H > limit || Wd > limit || C_in > (1 << 20) || C_out > (1 << 20)) return false;
    if (B > limit / H || B * H > limit / Wd || B * P > limit / Q) return false;
    SplitParams& p = s.p;
    p = SplitParams{};
    s.sparse = !dense && n <= 2 && m <= 16;
    p.npix = B * P * Q;
    p.B = (int)B, p.H = (int)H, p.Wd = (int)Wd, p.P = (int)P, p.Q = (int)Q, p.C_in = (int)C_in, p.C_out = (int)C_out;
    p.R = R, p.S = S, p.stride = stride, p.pad = pad, p.n = n;
    p.nchunks = (int)((C_out + (s.sparse ? 31 : 15)) / (s.sparse ? 32 : 16));
    p.nc32 = (int)((C_out + 31) / 32), p.ntiles_n = (int)((C_in + 63) / 64);
    const int ny = (R + stride - 1) / stride, nx = (S + stride - 1) / stride;
    const int64_t h = (H + stride - 1) / stride, w = (Wd + stride - 1) / stride;
    const int64_t classes = (int64_t)stride * stride;
    // most small problems go by without the search for tiles: the estimate is lowest with whole tiles of 256 rows, the cheaper step
    // of 128 and the larger group of taps
    const int64_t whole = (B * h * w + 255) / 256;
    s.rows = 128, s.np = 384;
    const SplitEstimates least = split_estimate(s, whole, m);
    if (least.split > 0.9 * least.plain) return false;
    SplitSides hs, ws;
    split_sides(hs, h, w), split_sides(ws, w, h);
    // 384 positions leave room for two taps of compressed planes per stage, 512 for one
    int64_t tiles = split_tiles(s, 256, 384, B, hs, ws, ny, nx);
    if (tiles == 0 || tiles > whole) {
        SplitPlan other = s;
        const int64_t t = split_tiles(other, 256, 512, B, hs, ws, ny, nx);
        if (t > 0 && (tiles == 0 || t < tiles)) s = other, tiles = t;
    }
    if (tiles * p.ntiles_n * classes < 192) {
        SplitPlan other = s;
        const int64_t t = split_tiles(other, 128, 256, B, hs, ws, ny, nx);
        if (t > 0) s = other, tiles = t;
    }
    const int64_t blocks = tiles * p.ntiles_n;
    if (tiles == 0 || blocks >= (1 << 22)) return false;   // (a launch holds fewer than 2^32 threads)
    const SplitEstimates e = split_estimate(s, tiles, m);
    if (e.split > 0.9 * e.plain) return false;
    class_slots(R, S, stride, p.slot0);
    s.p.nblocks = (int)blocks;
    const int64_t units = (int64_t)R * S * p.nc32 * p.ntiles_n * 4;
    if (units > (1 << 22)) return false;
    s.p.wblocks = (int)((units + 3) / 4);
    const int ic = m > 16 && !dense ? 32 : 16, px = 256 / (64 / ic);
    s.p.gblocks = (int)std::min<int64_t>(2048, (p.npix + px - 1) / px * ((C_out + 63) / 64));
    s.off_idx = split_align((size_t)p.nchunks * 96 * (size_t)p.npix);
    s.off_wimg = s.off_idx + (s.sparse ? split_align((size_t)p.nchunks * 4 * (size_t)p.npix) : 0);
    s.off_wnotes = s.off_wimg + (size_t)units * 3 * 1024;
    s.off_gnotes = s.off_wnotes + split_align((size_t)units * 8);
    s.bytes = s.off_gnotes + split_align((size_t)s.p.gblocks * 4);
    return true;
}

}  // namespace sdgp

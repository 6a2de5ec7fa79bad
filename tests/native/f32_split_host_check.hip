// Host build of what the planner of the fp32 products on the bf16 matrix instructions and its first pass share
// (csrc/bwd_f32_split.h, csrc/bwd_f32_split_tiles.h).
//   * class_slots, slot_tap: every slot of every filter up to 11 x 11 at strides 1 to 4 is the tap that the product, walking a
//     class's taps row by row from the class's first slot on, takes it for (Fig. 3: dD's pixels of one parity class meet the
//     taps r0, r0 + stride, ... of each axis), every tap has one slot, and no slot lies outside the filter.
//   * grid_side: never below one, and no position fewer than the taps reach.
//   * split3, split_join: three bf16 parts that add up to 2^24 x exactly, the second at most 2^-8 of it and the third 2^-17, no
//     subnormal among them, so that the products left out are at most 2^-24 (1 + 2^-9) of the whole; and back to x's own bits.
//   * split_tiles against every tile side, and how many it looks at.
//   * the planner declines launches of 2^32 threads and more.
// Prints one line per check and returns the number of mismatches; with the eleven numbers of a layer and a pattern as arguments
// prints the tile (rows, grid positions of the kernel, images, height, width) the planner gives it, or "none".  Test
// infrastructure, not product code.
#include <hip/hip_runtime.h>

#include <chrono>
#include <cstdio>
#include <cstdlib>

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

static bool bf16_part(uint32_t u) { return (u & 0xFFFFu) == 0u && ((u & 0x7F800000u) != 0u || (u & 0x7FFFFFFFu) == 0u); }

static int check_split() {
    int bad = 0;
    uint64_t state = 88172645463325252ull;
    double most = 0.0, other = 0.0;
    for (int64_t i = 0; i < 20000000; ++i) {
        state ^= state << 13, state ^= state >> 7, state ^= state << 17;
        uint32_t x = (uint32_t)state, kind = (uint32_t)(state >> 40) & 7u;
        if (kind == 0) x = (x & 0x80000000u) | (0x3F800000u + (x & 0xFFFFu) * 0x81u);       // runs of ones
        if (kind == 1) x &= 0x807FFFFFu;                                                     // subnormal
        if (kind == 2) x = (x & 0x80FFFFFFu) | 0x73000000u;                                  // about 2^104
        if (kind == 3) x |= 0x7F800000u;                                                     // infinite, NaN
        if (kind == 4) x |= 0xFFFFu << (x >> 27 & 7u);
        if (i < 4) x = (i & 1 ? 0x80000000u : 0u) | (i & 2 ? 0x7F800000u : 0u);
        const Split3 s = split3(x);
        const float back = split_join(s.h >> 16, s.m >> 16, s.l >> 16);
        if (float_to_bits(back) != x && !(back == 0.0f && (x << 1) == 0u)) ++bad;
        if (s.h == 0x7FC00000u) {
            if ((x & 0x7FFFFFFFu) < 0x737F8000u) ++bad;   // (rounds to 2^104 and beyond)
            continue;
        }
        const double v = (double)bits_to_float(x) * 0x1p24, m = bits_to_float(s.m), l = bits_to_float(s.l);
        if (!bf16_part(s.h) || !bf16_part(s.m) || !bf16_part(s.l) || (double)bits_to_float(s.h) + m + l != v) ++bad;
        if (v < 0 ? m < v * 0x1p-8 || m > -v * 0x1p-8 || l < v * 0x1p-17 || l > -v * 0x1p-17 : m > v * 0x1p-8 || m < -v * 0x1p-8 || l > v * 0x1p-17 || l < -v * 0x1p-17) ++bad;
        if (v != 0) {   // the products left out, of this value and the one before
            static double pm = 0, pl = 0;
            const double dm = m / v, dl = l / v, out = dm * pl + dl * pm + dl * pl;
            most = out > most ? out : most, other = out < other ? out : other, pm = dm, pl = dl;
        }
    }
    bad += most > 0x1p-24 * (1 + 0x1p-9) || -other > 0x1p-24 * (1 + 0x1p-9);
    printf("split: left out at most %.3g and %.3g, mismatches %d\n", most, other, bad);
    return bad;
}

// Rows times taps and grid positions of all tiles.
static double tile_cost(int rows, int taps, int64_t tb, int64_t th, int64_t tw, int grid) { return (double)tb * th * tw * (rows * (double)taps + grid); }

static int check_tiles() {
    int bad = 0;
    double worst = 1.0;
    uint64_t state = 88172645463325252ull;
    auto draw = [&](int lo, int hi) { state ^= state << 13, state ^= state >> 7, state ^= state << 17; return lo + (int)(state % (uint64_t)(hi - lo + 1)); };
    for (int i = 0; i < 2000; ++i) {
        const int64_t B = draw(1, 300);
        const int h = draw(1, 80), w = draw(1, 80), ny = draw(1, 5), nx = draw(1, 5), rows = draw(0, 1) ? 256 : 128;
        const int np = rows == 128 ? 256 : draw(0, 1) ? 384 : 512;
        double best = 1e300;
        for (int TH = 1; TH <= std::min(h, rows); ++TH)
            for (int TW = 1; TW <= std::min(w, rows / TH); ++TW)
                for (int TB = (int)std::min<int64_t>(B, rows / (TH * TW)); TB >= 1; TB /= 2) {
                    const int grid = TB * (TH + ny - 1) * (TW + nx - 1);
                    if (grid <= np) best = std::min(best, tile_cost(rows, ny * nx, (B + TB - 1) / TB, (h + TH - 1) / TH, (w + TW - 1) / TW, grid));
                }
        SplitPlan s;
        SplitSides hs, ws;
        split_sides(hs, h, w), split_sides(ws, w, h);
        const int64_t tiles = split_tiles(s, rows, np, B, hs, ws, ny, nx);
        const SplitParams& p = s.p;
        if (tiles == 0) {
            bad += best < 1e300;
            continue;
        }
        const int grid = p.TB * (p.TH + ny - 1) * (p.TW + nx - 1);
        const int64_t tb = (B + p.TB - 1) / p.TB;
        bad += grid > np || p.TB * p.TH * p.TW > rows || p.tiles_h * p.TH < h || p.tiles_w * p.TW < w || tiles != tb * p.tiles_h * p.tiles_w;
        worst = std::max(worst, tile_cost(rows, ny * nx, tb, p.tiles_h, p.tiles_w, grid) / best);
    }
    bad += worst > 1.05;
    int most = 0;   // pairs of sides that a plan looks at (all of them: up to 1400)
    for (int hw = 16; hw <= 224; ++hw) {
        SplitSides sides;
        split_sides(sides, hw, hw);
        int pairs = 0;
        for (int i = 0; i < sides.count; ++i)
            for (int j = 0; j < sides.count; ++j) pairs += sides.side[i] * sides.side[j] <= 256;
        most = std::max(most, pairs);
    }
    bad += most > 500;
    double best_us = 1e9;
    for (int k = 0; k < 20; ++k) {
        const auto begin = std::chrono::steady_clock::now();
        for (int x = 0; x < 20; ++x) {
            SplitPlan s;
            bad += !split_plan(s, 16, 112, 112, 64, 64, 3, 3, 1, 1, 2, 4);
        }
        best_us = std::min(best_us, std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - begin).count() / 20);
    }
    printf("tiles: worst %.3f of the best, up to %d pairs of sides, a plan at 112x112 takes %.2f us, mismatches %d\n", worst, most, best_us, bad);
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

int main(int argc, char** argv) {
    if (argc == 12) {
        int v[11];
        for (int i = 0; i < 11; ++i) v[i] = std::atoi(argv[i + 1]);
        SplitPlan s;
        if (!split_plan(s, v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8], v[9], v[10])) printf("none\n");
        else printf("%d %d %d %d %d\n", s.rows, s.np, s.p.TB, s.p.TH, s.p.TW);
        return 0;
    }
    const int total = check_slots() + check_sides() + check_split() + check_tiles() + check_limits();
    printf("total mismatches %d\n", total);
    return total != 0;
}

// Planner of the small-problem backward-data kernel.
#include "bwd_small.h"

namespace sdgp {

int launch_small_dense(const SmallParams& p, hipStream_t stream);
int launch_small_m4(const SmallParams& p, int rk, hipStream_t stream);
int launch_small_m8(const SmallParams& p, int rk, hipStream_t stream);
int launch_small_m16(const SmallParams& p, int rk, hipStream_t stream);
int launch_small_m32(const SmallParams& p, int rk, hipStream_t stream);

int bwd_pw_way(int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out, int R, int S, int stride, int pad, int n, int m, int rk,
               const void* workspace, size_t workspace_bytes);

namespace {

// Up to how many tiles this kernel is the faster one; 256 tiles are one round of the compute units, and time steps up
// with every further round begun.  Against what takes the problem otherwise (this kernel's time over the other's,
// smallest to largest over channels of 32 to 2048 and seven patterns; 12000 calls measured):
//
// 1x1, stride 1: the pointwise kernel takes 64 tiles of its own, 256 or 512 of these; `way` says how.
//   it declines (bwd_tiled): 0.06-0.48 up to 512 tiles.
//   dense: one round and C_out 512 0.89-0.91 (1.13 at C_in 64), 1024 0.79-1.00, 256 1.20-1.52; two rounds and C_out 2048
//     0.84-0.90 from C_in 1024 on, 1.2-1.3 at 256 and 512; C_out 1024 1.0-1.8.
//   ranked ahead: one round and C_out <= 128 0.87-1.00, 256 1.03-1.15, 512 on 0.72-0.94; two rounds 1.18-1.54.
//   ranked in the kernel, n <= 2: one round and C_out 512 on 0.37-0.77, Rescaled 256 0.85-0.97, else 0.94-1.50; two rounds
//     and C_out 2048 0.59-0.99, 1024 0.67-0.99 (Magnitude 0.79-1.13).
//   ranked in the kernel, others: one round and C_out 128 on 0.18-1.02 (160 at C_in 64 1.08-1.13), else 0.98-1.73; two and
//     C_out 1024 on 0.33-0.81.
//   C_out no multiple of its chunk (6955 calls, hardly a difference between C_in of 64 to 2048):
//     dense: one round and C_out 40 to 250 1.19-1.40, 256 to 520 0.90-1.14, 650 on 0.35-1.02; two and 2000 on 0.68-1.40 (from C_in 1024
//       on 0.81-0.98), 1496 and C_in 2048 0.81-0.84, else 1.0-2.3; three 1.07-3.3.
//     n <= 2, Magnitude: one and 40 to 200 1.01-1.27, 200 to 256 0.95-1.12, from there on 0.35-0.90; two and 1300 on 0.75-1.06, else
//       0.92-2.0; three 0.96-2.6.
//     n <= 2, Random and Rescaled: one and 40 to 160 0.94-1.29, 200 0.83-1.08, on 0.26-0.85; two and 800 on 0.44-1.03, else 0.84-2.0;
//       three and 1300 on 0.65-1.24, else 0.83-2.6.
//     general n: one and 40 to 160 0.90-1.22, 200 0.81-1.02, on 0.26-0.80; two and 800 on 0.55-0.97 (Rescaled 650 0.85-0.98), else
//       0.79-1.9; three and 1000 on 0.55-1.13, else 0.82-2.5.
//     more than 2^24 elements (the pointwise kernel on its usual tiles), two rounds: dense and Magnitude 1000 on 0.67-0.99.
//     four rounds: 0.77-4.05, below 1 for few.
//   the same where fewer than 64 tiles of more elements are left to bwd_tiled: four rounds 0.38-0.70.
// Other filters, stride 1: one round 0.16-0.86 whatever takes them.
//   bwd_row, which takes them from about 480 tiles on: 1.0-1.9 (groups of 32 0.33-0.99, at C_in 96 1.02-1.14).
//   bwd_conv3 (C_out a multiple of 64, dense or n <= 2), two rounds: dense and C_in > 64 0.69-0.91, n <= 2 and C_in > 64 0.81-1.0 where
//     C_out >= 256 and 0.93-1.14 below; C_in <= 64 1.0-1.46, half of every tile being columns that do not exist.
//   bwd_tiled, two rounds: C_in > 64 0.38-0.98; C_in <= 64 and nine taps 0.62-0.92 (C_out 48 and 56 1.08-1.22, 64, n > 2
//     1.12-1.28), more taps up to 1.52; C_out 40 and 48 at 25 and 49 taps 0.97-1.12; groups of 32 0.20-0.92 (49 taps at C_in 24 1.23).
// Strided filters (the parity classes of the pointwise kernel take them from about 900 tiles on, 0.79-2.77), bwd_tiled:
//   1x1: C_in > 64 0.11-0.80 up to four rounds; C_in <= 64 three 0.19-0.98, four 0.21-1.25.
//   wider: C_in > 64 two rounds 0.17-0.81, three 0.22-0.99 where C_out >= 128 or the filter has at most nine taps and
//     up to 1.16 otherwise, four 0.53-0.82 where C_out >= 256 and at most nine taps, up to 1.49 otherwise; C_in <= 64 two rounds
//     0.21-0.94 at nine taps, up to 1.10 beyond, three 0.32-1.65.  Groups of 32 0.20-0.97 up to four rounds.
constexpr int64_t kRound = 256;

int64_t most_pointwise(int way, bool whole_chunks, int64_t C_in, int64_t C_out, int n, int m, int rk) {
    const bool sparse = n <= 2 && m <= 16;
    if (!whole_chunks) {
        if (way < 0) return 4 * kRound;
        if (n == m) {
            const bool two = C_out >= (way == 0 ? 1000 : C_in >= 2048 ? 1400 : 2000) && (way == 0 || C_in >= 1024);
            return two ? 2 * kRound : C_out >= 320 ? kRound : 0;
        }
        if (sparse && rk == kGreedy) return C_out >= (way == 0 ? 1000 : 1300) ? 2 * kRound : C_out >= 200 ? kRound : 0;
        return C_out >= (sparse ? 1300 : 1000) ? 3 * kRound : C_out >= (!sparse && rk == kAdjusted ? 650 : 800) ? 2 * kRound : C_out >= 160 ? kRound : 0;
    }
    if (way < 0) return 2 * kRound;
    if (n == m) return C_out >= 2048 && C_in >= 1024 ? 2 * kRound : C_out >= 1024 || (C_out >= 512 && C_in > 64) ? kRound : 0;
    if (way == 1) return C_out <= 128 || C_out >= 512 ? kRound : 0;
    if (sparse) return C_out >= (rk == kGreedy ? 2048 : 1024) ? 2 * kRound : C_out >= (rk == kAdjusted ? 256 : 512) ? kRound : 0;
    return C_out >= 1024 ? 2 * kRound : C_out >= (C_in > 64 ? 128 : 256) ? kRound : 0;
}

// first: nobody else was asked; otherwise the kernels in front of bwd_conv3 and bwd_tiled have declined.
int64_t most_filter(bool first, int64_t C_in, int64_t C_out, int taps, int n, int m) {
    const bool dense = n == m, sparse = !dense && n <= 2 && m <= 16;
    if (!dense && m == 32 && (first ? C_in >= 128 : C_in > 64 || taps <= 25)) return 2 * kRound;
    if (first || (taps > 9 && (C_in <= 64 || C_out < 64))) return kRound;
    if (C_out % 64 == 0 && taps >= 4 && taps <= 49 && (dense || sparse)) return C_in > 64 && (dense || C_out >= 256) ? 2 * kRound : kRound;
    return C_in > 64 || C_out <= 40 || C_out >= 256 ? 2 * kRound : kRound;
}

int64_t most_strided(bool first, int64_t C_in, int64_t C_out, int taps, int n, int m) {
    int64_t rounds;
    if (n != m && m == 32) rounds = 4;
    else if (taps == 1) rounds = C_in > 64 ? 4 : 3;
    else if (C_in > 64) rounds = taps <= 9 && C_out >= 256 ? 4 : taps <= 9 || C_out >= 128 ? 3 : 2;
    else rounds = taps <= 9 ? 2 : 1;
    return (first && rounds > 2 ? 2 : rounds) * kRound;
}

}  // namespace

// A positive value: the problem does not fit, or is one for the other kernels.  The dispatch asks three times: first of all
// (turn 0), when the kernels for larger problems have declined (1), and when nobody but the plain kernel is left (2: strides of
// three and four, filters of more than 49 taps), which is slower by more than rounds can make up for.
int bwd_small_launch(int turn, const void* dO, const void* W, void* dD, int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out,
                     int R, int S, int stride, int pad, int n, int m, int rk, uint64_t seed, const void* workspace, size_t workspace_bytes,
                     hipStream_t stream) {
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
    const int64_t tiles = row_tiles * col_tiles * stride * stride;
    const bool first = turn == 0, pointwise = R == 1 && S == 1 && stride == 1;
    const int64_t most = turn == 2   ? 4 * kRound
                         : pointwise ? most_pointwise(bwd_pw_way(B, H, Wd, C_in, C_out, R, S, stride, pad, n, m, rk, workspace, workspace_bytes),
                                                    C_out % 32 == 0, C_in, C_out, n, m, rk)
                         : stride == 1 ? most_filter(first, C_in, C_out, R * S, n, m)
                                       : most_strided(first, C_in, C_out, R * S, n, m);
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

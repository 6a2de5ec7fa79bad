// Host side of the pointwise kernel: 1x1 convolutions without padding (any stride) and linear layers whose channel
// counts fit (both multiples of 8); chooses the tile shape and launches.
#include <climits>

#include "bwd_pw_launch.h"

namespace sdgp {

int launch_pw_dense(const PwParams& p, int shape, hipStream_t stream);
int launch_pw_sparse_m4(const PwParams& p, int shape, int rk, hipStream_t stream);
int launch_pw_sparse_m8(const PwParams& p, int shape, int rk, hipStream_t stream);
int launch_pw_sparse_m16(const PwParams& p, int shape, int rk, hipStream_t stream);
int launch_pw_masked_m4(const PwParams& p, int shape, int rk, hipStream_t stream);
int launch_pw_masked_m8(const PwParams& p, int shape, int rk, hipStream_t stream);
int launch_pw_masked_m16(const PwParams& p, int shape, int rk, hipStream_t stream);
int launch_pw_masked_m32(const PwParams& p, int shape, int rk, hipStream_t stream);
int launch_pw_classes_dense(const PwClasses& all, int ncls, int shape, hipStream_t stream);
int launch_pw_classes_sparse_m4(const PwClasses& all, int ncls, int shape, int rk, hipStream_t stream);
int launch_pw_classes_sparse_m8(const PwClasses& all, int ncls, int shape, int rk, hipStream_t stream);
int launch_pw_classes_sparse_m16(const PwClasses& all, int ncls, int shape, int rk, hipStream_t stream);
int launch_pw_classes_masked_m4(const PwClasses& all, int ncls, int shape, int rk, hipStream_t stream);
int launch_pw_classes_masked_m8(const PwClasses& all, int ncls, int shape, int rk, hipStream_t stream);
int launch_pw_classes_masked_m16(const PwClasses& all, int ncls, int shape, int rk, hipStream_t stream);
int launch_pw_classes_masked_m32(const PwClasses& all, int ncls, int shape, int rk, hipStream_t stream);
int launch_pw_pre(const PwParams& p, int shape, hipStream_t stream);
int launch_pw_classes_pre(const PwClasses& all, int ncls, int shape, hipStream_t stream);
int bwd_stride2_launch(int classes, const void* dO, const void* W, void* dD, int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out,
                       int R, int S, int stride, int pad, int n, int m, int rk, uint64_t seed, hipStream_t stream);
size_t compress_meta_offset(int64_t rows, int64_t C_out);
size_t compress_bytes(int64_t rows, int64_t C_out);
int compress_launch(const void* dO, int64_t rows, int64_t C_out, int n, int m, int rk, uint64_t seed, void* workspace,
                    hipStream_t stream);

namespace {

// 0: dense (n == m); 2: at most two survivors per aligned quad, the structured-sparse instruction; 1: any other n of
// m in {4, 8, 16, 32}, pruned rows stored dense with zeros; -1: not for this kernel
int pw_mode(int n, int m) {
    if (n == m) return 0;
    if (n <= 2 && (m == 4 || m == 8 || m == 16)) return 2;
    if (m == 4 || m == 8 || m == 16 || m == 32) return 1;
    return -1;
}

int launch_pw_any(const PwParams& p, int mode, int m, int shape, int rk, hipStream_t stream) {
    if (mode == 0) return launch_pw_dense(p, shape, stream);
    if (mode == 2) {
        if (m == 4) return launch_pw_sparse_m4(p, shape, rk, stream);
        if (m == 8) return launch_pw_sparse_m8(p, shape, rk, stream);
        return launch_pw_sparse_m16(p, shape, rk, stream);
    }
    if (m == 4) return launch_pw_masked_m4(p, shape, rk, stream);
    if (m == 8) return launch_pw_masked_m8(p, shape, rk, stream);
    if (m == 16) return launch_pw_masked_m16(p, shape, rk, stream);
    return launch_pw_masked_m32(p, shape, rk, stream);
}

int launch_pw_classes_any(const PwClasses& all, int ncls, int mode, int m, int shape, int rk, hipStream_t stream) {
    if (mode == 0) return launch_pw_classes_dense(all, ncls, shape, stream);
    if (mode == 2) {
        if (m == 4) return launch_pw_classes_sparse_m4(all, ncls, shape, rk, stream);
        if (m == 8) return launch_pw_classes_sparse_m8(all, ncls, shape, rk, stream);
        return launch_pw_classes_sparse_m16(all, ncls, shape, rk, stream);
    }
    if (m == 4) return launch_pw_classes_masked_m4(all, ncls, shape, rk, stream);
    if (m == 8) return launch_pw_classes_masked_m8(all, ncls, shape, rk, stream);
    if (m == 16) return launch_pw_classes_masked_m16(all, ncls, shape, rk, stream);
    return launch_pw_classes_masked_m32(all, ncls, shape, rk, stream);
}

// Tile shape of the fused and dense kernels.  Workgroups of four wavefronts, two or more to a CU, so that one's loads
// and stores overlap the other's arithmetic.  Dense: 128 x 128 tiles measured fastest (column tiles of one row tile run side
// by side on one XCD and find the gradient rows in its L2).  Pruning: 256 columns, so that a gradient row is ranked once
// per 256, or 128, of which two workgroups more fit a CU.  Time with 128 columns over that with 256, 1x1 layers:
//   general n of m up to 16: 0.57-0.97 (424 and 960 columns 1.04, 1.08), whose kernel with 256 leaves one workgroup to a CU;
//     Rescaled, up to 256 columns and C_out 1152 1.23;
//   n <= 2: columns rounded up to 128 fewer than to 256 0.75-0.97 up to 512 of them, from there on 0.74-0.94 in groups of 4
//     with the magnitude rankers and 0.98-1.12 otherwise; fewer than 128 tiles of 256 0.65-0.84; otherwise 0.89-1.32;
//   groups of 32: 1.09-1.51, fewer than 64 tiles (which went elsewhere) 0.66.
// 129 to 256 tiles of 256 columns are one workgroup on a CU; where that makes more than 256 tiles of 128, some CUs get two and the
// rest wait for them: 1.05-1.29 (C_out up to 192 0.96-1.01), 0.70-0.85 where it makes 256 or fewer.
// Parity classes rank an element once per tap and column tile: 1.04-1.52, where fewer than 64 tiles went elsewhere 0.48-0.68.
int pw_shape(int mode, int64_t C_in, int64_t C_out, int m, int rk, int64_t row_tiles, bool classes) {
    if (C_in <= 64) return 2;   // 128 x 64: 256-row tiles measured the same or slower (fewer workgroups, a longer last round)
    if (mode == 0 || C_in <= 128 || C_out <= 64) return 1;   // (64 channels to rank: ranking them per 128 columns costs less than the third workgroup per CU gains)
    const int64_t wide = (C_in + 255) / 256, narrow = (C_in + 127) / 128, tiles = row_tiles * wide;
    if (tiles < 64) return 1;
    if (classes || m == 32 || (mode == 1 && rk == kAdjusted && wide == 1 && C_out > 512)) return 0;
    if (tiles < 128) return 1;
    if (tiles <= 256) return row_tiles * narrow > 256 ? 0 : 1;
    return mode == 1 || (narrow < 2 * wide && (wide <= 2 || (m == 4 && rk != kRandom))) ? 1 : 0;
}
// How many column tiles of the fused kernel would rank a gradient element, as the choice below counts them.
int pw_times_ranked(int mode, int64_t C_in, int64_t C_out) {
    const int bn = C_in <= 64 ? 64 : mode != 0 && C_in > 128 && C_out > 64 ? 256 : 128;
    return (int)((C_in + bn - 1) / bn);
}
// Tile shape when the gradient arrives compressed (nothing is ranked in the kernel): the dense kernel's.
int pw_pre_shape(int64_t C_in) { return C_in <= 64 ? 2 : 1; }

// Whether a pass that ranks and compresses the gradient first (csrc/compress.hip) pays: the fused kernel would rank
// every gradient element `times` times, the pass reads it once and writes half of it, and the product that follows
// runs 1.15-1.25 times as fast as the dense one.  Measured on the layers of ResNet-50 at batch 256: from two times on
// with the random ranker (the hash makes ranking dearer), from four on with the magnitude rankers.
bool pre_pays(int mode, int64_t C_out, int64_t rows_dO, int times, int rk) {
    const int least = rk == kRandom ? 2 : 4;
    return mode == 2 && (C_out % 64) == 0 && times >= least && rows_dO * (C_out / 16) < ((int64_t)1 << 31);
}

struct PwPlan {
    PwParams p;
    int mode, shape;
    bool pre;       // rank and compress first, then MODE 3 (needs the workspace)
    size_t bytes;   // workspace of the pre path
};

// 0 and the plan, or 1 when the pointwise kernel does not take the problem.
int pw_plan(int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out, int R, int S, int stride, int pad, int n, int m,
            int rk, PwPlan& out, int force_shape = -1) {
    const int mode = pw_mode(n, m);
    if (mode < 0) return 1;
    if (R != 1 || S != 1 || stride < 1 || stride > 255 || pad != 0 || (C_out % 8) != 0 || (C_in % 8) != 0) return 1;
    if (mode != 0 && (C_out % m) != 0) return 1;
    const int64_t P = (H - 1) / stride + 1, Q = (Wd - 1) / stride + 1;  // gradient image
    const int64_t rows = B * P * Q;
    if (stride > 1 && (B * H * Wd >= INT_MAX || H < 1 || Wd < 1)) return 1;
    if (rows < 1 || C_out < 8 || C_in < 8 || C_out >= (1 << 24) || C_in >= (1 << 24)) return 1;

    // (the random ranker's sixteen channels of a short chunk must not straddle a carry into the index's high word)
    if (rk == kRandom && mode != 0 && C_out % 16 != 0 && rows > (int64_t)0xFFFFFFFFu / C_out) return 1;

    PwParams p{};
    p.rows = rows, p.C_out = (int)C_out, p.C_in = (int)C_in;
    p.n = n;
    p.stride = stride, p.P = (int)P, p.Q = (int)Q, p.H = (int)H, p.Wd = (int)Wd;
    p.rows_dO = rows, p.gather = 0, p.ntaps = 1, p.w_taps = 1;
    if (stride > 1) p.by_image = fast_div((uint32_t)(P * Q)), p.by_line = fast_div((uint32_t)Q);   // (rows below 2^31 then)

    int shape = force_shape >= 0 ? force_shape : pw_shape(mode, C_in, C_out, m, rk, (rows + 127) / 128, false);
    out.pre = force_shape < 0 && pre_pays(mode, C_out, rows, pw_times_ranked(mode, C_in, C_out), rk);
    if (out.pre) shape = pw_pre_shape(C_in);
    const int bn = kPwShapes[shape].bn, rows_per = kPwShapes[shape].rows;
    const int64_t blocks = ((rows + rows_per - 1) / rows_per) * ((C_in + bn - 1) / bn);
    // too small to be worth a matrix-core launch of this shape (a forced shape: the caller has decided)
    if ((blocks < 64 && force_shape < 0) || blocks < 1 || blocks >= INT_MAX) return 1;
    p.ntiles_n = (int)((C_in + bn - 1) / bn);
    p.nblocks = (int)blocks;
    out.p = p, out.mode = mode, out.shape = shape;
    out.bytes = out.pre ? compress_bytes(rows, C_out) : 0;
    return 0;
}

// ---- small 1x1 / linear problems whose C_out is a multiple of 8 but not of the chunk (a classifier's 1000 outputs).  The kernel
// takes them as they are; they are worth it below the 64 tiles that other layers need, since bwd_tiled is what is left for them.
// Copies of gradient and filter with C_out rounded up, and the kernel on those, took 1.3-2.6 times as long (136->144 at
// 25x25, batch 92, 2:4 Rescaled 32.8 us against 12.9, 1536->392 at 25x25, batch 20, 1:4 74.9 against 35.9).

// Whether the problem is one: plain 1x1 stride 1, at most 16 M elements in gradient and filter.
bool small_short_chunk(int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out, int R, int S, int stride, int pad, int n, int m) {
    if (R != 1 || S != 1 || stride != 1 || pad != 0) return false;
    if (C_out < kPwKC || (C_out % kPwKC) == 0 || (C_out % 8) != 0 || (C_in % 8) != 0 || C_in < 8) return false;
    if (pw_mode(n, m) < 0 || (n != m && (C_out % m) != 0)) return false;
    const int64_t rows = B * H * Wd, Kp = (C_out + kPwKC - 1) / kPwKC * kPwKC;
    return rows >= 1 && rows * Kp <= ((int64_t)1 << 24) && Kp * C_in <= ((int64_t)1 << 24);
}
// Their tiles: with fewer than 256 of the usual shape 128 x 64, the most workgroups; with more the usual one took 0.64-0.97
// of the time of 128 x 64 (1.17 at 432->120, 17x17, batch 117).
int small_short_chunk_shape(int mode, int64_t C_in, int64_t C_out, int m, int rk, int64_t rows) {
    const int shape = pw_shape(mode, C_in, C_out, m, rk, (rows + 127) / 128, false);
    const int64_t rows_per = kPwShapes[shape].rows, bn = kPwShapes[shape].bn;
    return ((rows + rows_per - 1) / rows_per) * ((C_in + bn - 1) / bn) < 256 ? 2 : shape;
}
// The workspace that the query names for them.  Nothing reads it, and a call may leave it out; the size stays as programs know it.
size_t small_short_chunk_bytes(int64_t rows, int64_t C_in, int64_t C_out) {
    const size_t Kp = (size_t)((C_out + kPwKC - 1) / kPwKC * kPwKC);
    return (((size_t)rows * Kp * 2u + 255u) & ~(size_t)255u) + Kp * (size_t)C_in * 2u;
}

}  // namespace

// Workspace bytes with which bwd_pw_launch / bwd_gather_launch rank the gradient once, in a pass of their own (0: the
// fused kernel is used, or neither takes the problem).
size_t bwd_pw_workspace(int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out, int R, int S, int stride, int pad, int n,
                        int m);

// Whether no kernel reads the workspace that the query names for a bf16 problem.
bool bwd_pw_workspace_unread(int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out, int R, int S, int stride, int pad, int n, int m) {
    return small_short_chunk(B, H, Wd, C_in, C_out, R, S, stride, pad, n, m);
}

// How bwd_pw_launch runs a problem with aligned pointers: -1 not at all, 0 as it is, 1 with the gradient ranked ahead, 2 a small
// one with a short last chunk.
int bwd_pw_way(int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out, int R, int S, int stride, int pad, int n, int m, int rk,
               const void* workspace, size_t workspace_bytes) {
    const size_t room = workspace != nullptr && is_aligned16(workspace) ? workspace_bytes : 0;
    if (small_short_chunk(B, H, Wd, C_in, C_out, R, S, stride, pad, n, m)) return 2;
    PwPlan plan{};
    if (pw_plan(B, H, Wd, C_in, C_out, R, S, stride, pad, n, m, rk, plan) != 0) return -1;
    if (!plan.pre) return 0;
    if (room >= plan.bytes) return 1;
    const PwShape& shape = kPwShapes[pw_shape(plan.mode, C_in, C_out, m, rk, (plan.p.rows + 127) / 128, false)];
    return ((plan.p.rows + shape.rows - 1) / shape.rows) * ((C_in + shape.bn - 1) / shape.bn) < 64 ? -1 : 0;
}

// SDGP_OK after launching, a positive value when the problem does not fit, or a negative sdgp_status.  With a
// workspace of at least bwd_pw_workspace(...) bytes the gradient is ranked once, in a pass of its own, where that
// pays; with less the fused kernel runs.
int bwd_pw_launch(const void* dO, const void* W, void* dD, int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out,
                  int R, int S, int stride, int pad, int n, int m, int rk, uint64_t seed, void* workspace, size_t workspace_bytes,
                  hipStream_t stream) {
    if (!is_aligned16(dO) || !is_aligned16(W) || !is_aligned16(dD)) return 1;
    const int shape = small_short_chunk(B, H, Wd, C_in, C_out, R, S, stride, pad, n, m)
                          ? small_short_chunk_shape(pw_mode(n, m), C_in, C_out, m, rk, B * H * Wd)
                          : -1;
    PwPlan plan{};
    if (pw_plan(B, H, Wd, C_in, C_out, R, S, stride, pad, n, m, rk, plan, shape) != 0) return 1;
    if (plan.pre && (workspace == nullptr || workspace_bytes < plan.bytes || !is_aligned16(workspace))) {
        // no room for the compressed gradient: the fused kernel
        const int shape = pw_shape(plan.mode, C_in, C_out, m, rk, (plan.p.rows + 127) / 128, false);
        const int bn = kPwShapes[shape].bn, rows_per = kPwShapes[shape].rows;
        const int64_t blocks = ((plan.p.rows + rows_per - 1) / rows_per) * ((C_in + bn - 1) / bn);
        if (blocks < 64 || blocks >= INT_MAX) return 1;
        plan.p.ntiles_n = (int)((C_in + bn - 1) / bn), plan.p.nblocks = (int)blocks;
        plan.shape = shape, plan.pre = false;
    }
    PwParams& p = plan.p;
    p.W = static_cast<const uint16_t*>(W);
    p.dD = static_cast<uint16_t*>(dD);
    p.mix = seed_mix(seed);
    if (plan.pre) {
        const int rc = compress_launch(dO, p.rows_dO, C_out, n, m, rk, seed, workspace, stream);
        if (rc != SDGP_OK) return rc;
        p.dO = static_cast<const uint16_t*>(workspace);
        p.meta = static_cast<const unsigned char*>(workspace) + compress_meta_offset(p.rows_dO, C_out);
        return launch_pw_pre(p, plan.shape, stream);
    }
    p.dO = static_cast<const uint16_t*>(dO);
    return launch_pw_any(p, plan.mode, m, plan.shape, rk, stream);
}

// Strided filters wider than 1x1 (the stride-2 3x3 layers of a ResNet): the input pixels split into stride x stride
// parity classes; class (a, b) -- pixels (i*stride + a, j*stride + b) -- is a small stride-1 correlation over the
// gradient with the taps r = a + pad (mod stride), s = b + pad (mod stride), at most four of them here.  Each class is
// a GEMM of the pointwise kernel whose reduction runs over (tap, channel) and whose rows are gathered from the gradient
// pixels (i + dp, j + dq) of each tap, zeros outside; all classes go out in one launch (blockIdx.y = class).  Each
// gradient element is ranked once per tap that reads it (the kept set does not depend on who asks).
namespace {

struct GatherPlan {
    PwClasses all;
    int ncls, mode, shape;
    bool pre;
    size_t bytes;
};

// 0 and the plan for the shape the fused kernels use (pre == false) or the compressed-operand kernel uses, or 1.
int gather_plan(int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out, int R, int S, int stride, int pad, int n, int m,
                bool want_pre, GatherPlan& out) {
    const int mode = pw_mode(n, m);
    if (mode < 0) return 1;
    if (stride < 2 || stride > 4 || R < stride || S < stride || R > 2 * stride || S > 2 * stride || pad < 0) return 1;
    if (C_out < 8 || (C_out % 8) != 0 || C_in < 8 || (C_in % 8) != 0) return 1;
    if (mode != 0 && (C_out % m) != 0) return 1;
    if (H + 2 * pad < R || Wd + 2 * pad < S || H < stride || Wd < stride) return 1;
    const int64_t P = (H + 2 * pad - R) / stride + 1, Q = (Wd + 2 * pad - S) / stride + 1;
    if (B < 1 || P < 1 || Q < 1 || P >= 65536 || Q >= 32768 || H >= 65536 || Wd >= 32768 || B * (P + 8) * (Q + 8) >= (1 << 30) || B * H * Wd >= INT_MAX ||
        C_out >= (1 << 20) || (int64_t)R * S * C_in >= (1 << 20))
        return 1;

    // (the random ranker's sixteen channels of a short chunk must not straddle a carry into the index's high word)
    if (mode != 0 && C_out % 16 != 0 && B * P * Q > (int64_t)0xFFFFFFFFu / C_out) return 1;

    PwParams base{};
    base.C_out = (int)C_out, base.C_in = (int)C_in;
    base.n = n;
    base.stride = stride, base.P = (int)P, base.Q = (int)Q, base.H = (int)H, base.Wd = (int)Wd;
    base.rows_dO = B * P * Q, base.gather = 1, base.w_taps = R * S;

    // every tap of every class ranks the rows it reads: R * S times per gradient element and column tile
    out.pre = want_pre && pre_pays(mode, C_out, base.rows_dO, R * S, kRandom);
    const int64_t least_rows = B * (H / stride) * (Wd / stride);   // of the smallest class
    const int shape = out.pre ? pw_pre_shape(C_in) : pw_shape(mode, C_in, C_out, m, kRandom, (least_rows + 127) / 128, true);
    const int bn = kPwShapes[shape].bn, rows_per = kPwShapes[shape].rows;
    base.ntiles_n = (int)((C_in + bn - 1) / bn);

    // all classes first: nothing is launched unless every one of them fits
    static_assert(kPwMaxClasses >= 16, "stride up to four");
    PwParams* cls = out.all.c;
    int ncls = 0;
    for (int a = 0; a < stride; ++a)
        for (int b = 0; b < stride; ++b) {
            PwParams q = base;
            q.oa = a, q.ob = b;
            q.Pc = (int)((H - a + stride - 1) / stride), q.Qc = (int)((Wd - b + stride - 1) / stride);
            q.ntaps = 0;
            for (int r = 0; r < R; ++r) {
                if ((a + pad - r) % stride != 0) continue;
                for (int sx = 0; sx < S; ++sx) {
                    if ((b + pad - sx) % stride != 0) continue;
                    if (q.ntaps == 4) return 1;
                    q.tap_dp[q.ntaps] = (a + pad - r) / stride, q.tap_dq[q.ntaps] = (b + pad - sx) / stride;
                    q.tap_w[q.ntaps] = r * S + sx;
                    ++q.ntaps;
                }
            }
            if (q.ntaps == 0) return 1;
            q.rows = B * q.Pc * q.Qc;
            q.by_image = fast_div((uint32_t)(q.Pc * q.Qc)), q.by_line = fast_div((uint32_t)q.Qc);   // (both positive: H, Wd >= stride)
            const int64_t blocks = ((q.rows + rows_per - 1) / rows_per) * q.ntiles_n;
            if (q.rows < 1 || blocks < 64 || blocks >= INT_MAX) return 1;
            q.nblocks = (int)blocks;
            cls[ncls++] = q;
        }
    // classes with more taps first: their workgroups run longest, and the launch should end on the short ones
    for (int i = 1; i < ncls; ++i)
        for (int j = i; j > 0 && cls[j].ntaps > cls[j - 1].ntaps; --j) {
            const PwParams t = cls[j];
            cls[j] = cls[j - 1];
            cls[j - 1] = t;
        }
    out.ncls = ncls, out.mode = mode, out.shape = shape;
    out.bytes = out.pre ? compress_bytes(base.rows_dO, C_out) : 0;
    return 0;
}

}  // namespace

// SDGP_OK after launching, a positive value when the problem does not fit, or a negative sdgp_status.  Workspace as
// for bwd_pw_launch.
int bwd_gather_launch(const void* dO, const void* W, void* dD, int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out,
                      int R, int S, int stride, int pad, int n, int m, int rk, uint64_t seed, void* workspace, size_t workspace_bytes,
                      hipStream_t stream) {
    if (!is_aligned16(dO) || !is_aligned16(W) || !is_aligned16(dD)) return 1;
    GatherPlan plan{};
    bool planned = false;
    if (workspace != nullptr && is_aligned16(workspace)) {
        planned = gather_plan(B, H, Wd, C_in, C_out, R, S, stride, pad, n, m, true, plan) == 0 && (!plan.pre || workspace_bytes >= plan.bytes);
    }
    if (!planned && gather_plan(B, H, Wd, C_in, C_out, R, S, stride, pad, n, m, false, plan) != 0) return 1;
    // 3x3 of stride 2: the kernel that ranks a gradient element once for all four classes, where it is the faster one
    const int rc2 = bwd_stride2_launch(plan.pre ? 2 : 1, dO, W, dD, B, H, Wd, C_in, C_out, R, S, stride, pad, n, m, rk, seed, stream);
    if (rc2 <= 0) return rc2;
    const int64_t rows_dO = plan.all.c[0].rows_dO;
    const void* grad = dO;
    const unsigned char* meta = nullptr;
    if (plan.pre) {
        const int rc = compress_launch(dO, rows_dO, C_out, n, m, rk, seed, workspace, stream);
        if (rc != SDGP_OK) return rc;
        grad = workspace;
        meta = static_cast<const unsigned char*>(workspace) + compress_meta_offset(rows_dO, C_out);
    }
    for (int i = 0; i < plan.ncls; ++i) {
        PwParams& q = plan.all.c[i];
        q.dO = static_cast<const uint16_t*>(grad), q.meta = meta;
        q.W = static_cast<const uint16_t*>(W), q.dD = static_cast<uint16_t*>(dD);
        q.mix = seed_mix(seed);
    }
    if (plan.pre) return launch_pw_classes_pre(plan.all, plan.ncls, plan.shape, stream);
    return launch_pw_classes_any(plan.all, plan.ncls, plan.mode, m, plan.shape, rk, stream);
}

size_t bwd_pw_workspace(int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out, int R, int S, int stride, int pad, int n,
                        int m) {
    if (small_short_chunk(B, H, Wd, C_in, C_out, R, S, stride, pad, n, m)) return small_short_chunk_bytes(B * H * Wd, C_in, C_out);
    PwPlan one{};
    // (the ranker that takes the pass soonest: the size is enough for any)
    if (pw_plan(B, H, Wd, C_in, C_out, R, S, stride, pad, n, m, kRandom, one) == 0) return one.bytes;
    GatherPlan many{};
    if (gather_plan(B, H, Wd, C_in, C_out, R, S, stride, pad, n, m, true, many) == 0) return many.bytes;
    return 0;
}

}  // namespace sdgp

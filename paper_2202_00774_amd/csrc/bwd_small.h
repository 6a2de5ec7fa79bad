// Backward-data kernel for bf16 problems too small to fill the chip with the tiles of the other matrix-core kernels:
// dL/dD[rows, C_in] = sum over taps of prune(dL/dO)[gathered rows, C_out] . W[:, tap, :] (Fig. 2, Fig. 3; Sec. II-A).
//
// Such a call is bound by latency: a few dozen workgroups walk a long reduction, every step of it a round trip to
// memory.  So a tile is small (32 rows x 128 columns), the eight wavefronts of its workgroup split the reduction, and a
// wavefront loads both operands from global memory straight into the registers v_mfma_f32_32x32x16_bf16 reads, the next
// step's loads in flight while one is ranked and multiplied: no LDS round trip and no barrier until the sums are added.
//   * Rows: lane l holds row l % 32.  Half h = l / 32 of the wavefront takes CH consecutive channels of the pixel (the
//     order of the reduction is free as long as both operands agree), so every m-group is ranked (Sec. III-B) in the lane
//     that holds it.
//   * Columns: lane l of column tile j holds column 4 * (l % 32) + j.  A lane reads 8 bytes (its four columns) of eight
//     rows of W in its native layout and turns them into the four tiles' fragments with sixteen byte permutations.
//   * The wavefronts add their sums through LDS in a fixed order; a result row leaves as 8 bytes per lane, 256 a row.
// Each XCD takes a run of the tiles in column order, so that its L2 serves one part of W.
// Strided filters: blockIdx.y is the parity class of the input pixels, whose taps are a sub-grid of the filter.
// Channels past C_out are zeros on both sides; taps outside the gradient and rows past the end are zero rows.  Zero times a
// non-finite weight is NaN where the definition has no term at all, so a NaN result of a row with taps outside the gradient
// is summed again without them.
#pragma once

#include <type_traits>

#include "lds_copy.h"
#include "parity_axis.h"

namespace sdgp {

#ifndef SDGP_GLOBAL
#define SDGP_GLOBAL __attribute__((address_space(1)))
#endif

constexpr int kSmallDense = 3;    // n == m: nothing is ranked
constexpr int kSmallWaves = 8, kSmallRows = 32, kSmallCols = 128;

static __device__ const uint32_t kSmallZeros[4] __attribute__((aligned(16))) = {};

struct SmallParams {
    const uint16_t* dO;
    const uint16_t* W;
    uint16_t* dD;
    int64_t B;
    int H, Wd, P, Q, C_in, C_out, R, S, stride, pad, n;
    int col_tiles, row_tiles;   // row tiles of the largest parity class
    uint32_t mix;
};

// The four results of row `row` at channel c0, some of them NaN: those that a weight of a tap outside the gradient can have
// made NaN are summed again over the taps inside.  Rare, so it is short rather than fast and reads the kernel's arguments
// again, so that none of it holds a register during the main loop: with the kernel's own ranker and registers every call
// was 4 % slower (calls of 5 to 70 us; 10 % at 4:32), like this 0.6 %.
template <int M, int RK>
__device__ __forceinline__ void sum_inside(int row, int c0, float (&v)[4]) {
    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
    uint64_t args = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    const auto& p = *reinterpret_cast<const __attribute__((address_space(4))) SmallParams*>(args);
    const ParityAxis<int> ay = parity_axis<int>(p.H, p.R, p.stride, p.pad, (int)blockIdx.y / p.stride);
    const ParityAxis<int> ax = parity_axis<int>(p.Wd, p.S, p.stride, p.pad, (int)blockIdx.y % p.stride);
    const int b = row / (ay.n * ax.n), rem = row - b * (ay.n * ax.n);
    const int gi = rem / ax.n + ay.shift, gj = rem % ax.n + ax.shift;
    const int64_t kstep = (int64_t)p.R * p.S * p.C_in;
    auto weights = [&](int u, int t) { return p.W + ((ay.r0 + u * p.stride) * p.S + ax.r0 + t * p.stride) * p.C_in + c0; };
    auto inside = [&](int u, int t) { return (unsigned)(gi - u) < (unsigned)p.P && (unsigned)(gj - t) < (unsigned)p.Q; };
    uint32_t brought = 0;   // columns with a non-finite weight in a tap outside
#pragma nounroll
    for (int u = 0; u < ay.count; ++u)
#pragma nounroll
        for (int t = 0; t < ax.count; ++t) {
            if (inside(u, t)) continue;
            const uint16_t* w = weights(u, t);
#pragma unroll 4
            for (int k = 0; k < p.C_out; ++k, w += kstep) {
                const u32x2_t x = *reinterpret_cast<const u32x2_t*>(w);
#pragma unroll
                for (int z = 0; z < 2; ++z)
                    brought |= ((x[z] & 0x7F80u) == 0x7F80u ? 1u << (2 * z) : 0u) | ((x[z] & 0x7F800000u) == 0x7F800000u ? 2u << (2 * z) : 0u);
            }
        }
    float sum[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    auto settled = [&]() {   // nothing left to find out: not a column of these, or a NaN of its own
        bool all = true;
#pragma unroll
        for (int z = 0; z < 4; ++z) all = all && (v[z] == v[z] || !((brought >> z) & 1u) || sum[z] != sum[z]);
        return all;
    };
#pragma nounroll
    for (int u = 0; u < ay.count; ++u)
#pragma nounroll
        for (int t = 0; t < ax.count; ++t) {
            if (!inside(u, t)) continue;
            const int64_t row0 = (int64_t)((b * p.P + gi - u) * p.Q + gj - t) * p.C_out;
            const uint16_t* w = weights(u, t);
#pragma nounroll
            for (int k = 0; k < p.C_out && !settled(); k += M) {
                const uint16_t* const g = p.dO + row0 + k;
                const uint32_t mask = RK == kSmallDense ? ~0u : keep_by_count<M, RK>(g, p.n, p.mix, (uint64_t)(row0 + k));
                float scale = 1.0f;
                if constexpr (RK == kAdjusted) {
                    float total = 0.0f, kept = 0.0f;
#pragma nounroll
                    for (int j = 0; j < M; ++j) {
                        const float a = bf16_to_float((uint32_t)g[j] & 0x7FFFu);
                        total = __fadd_rn(total, a);
                        if ((mask >> j) & 1u) kept = __fadd_rn(kept, a);
                    }
                    if (kept != 0.0f) scale = __fdiv_rn(total, kept);
                }
#pragma nounroll
                for (int j = 0; j < M; ++j, w += kstep) {
                    float x = (mask >> j) & 1u ? bf16_to_float(g[j]) : 0.0f;
                    if constexpr (RK == kAdjusted) {
                        if ((mask >> j) & 1u) x = bf16_to_float(float_to_bf16(__fmul_rn(x, scale)));
                    }
                    const u32x2_t y = *reinterpret_cast<const u32x2_t*>(w);
                    sum[0] = fmaf(x, bf16_to_float(y[0] & 0xFFFFu), sum[0]);
                    sum[1] = fmaf(x, bf16_to_float(y[0] >> 16), sum[1]);
                    sum[2] = fmaf(x, bf16_to_float(y[1] & 0xFFFFu), sum[2]);
                    sum[3] = fmaf(x, bf16_to_float(y[1] >> 16), sum[3]);
                }
            }
        }
#pragma unroll
    for (int z = 0; z < 4; ++z)
        if (v[z] != v[z] && ((brought >> z) & 1u)) v[z] = sum[z];
}

template <int M, int RK, bool NLE2>
__global__ void __launch_bounds__(64 * kSmallWaves) bwd_small(const SmallParams p) {
    constexpr int CH = M > 16 ? M : 16;   // channels per lane and step
    constexpr int NQ = CH / 8;            // 16-byte gradient loads and matrix steps
    typedef const SDGP_GLOBAL uint16_t* gptr_t;
    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int ca = (int)blockIdx.y / p.stride, cb = (int)blockIdx.y % p.stride;
    const ParityAxis<int> ay = parity_axis<int>(p.H, p.R, p.stride, p.pad, ca), ax = parity_axis<int>(p.Wd, p.S, p.stride, p.pad, cb);
    const int rows = (int)p.B * ay.n * ax.n;
    // workgroups go to the XCDs in turn: each takes a run of the tiles, which are in column order
    const int per_xcd = (int)gridDim.x >> 3, logical = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
    const int ct = logical / p.row_tiles, tile = logical - ct * p.row_tiles;
    if (ct >= p.col_tiles || tile * kSmallRows >= rows) return;   // (the whole workgroup: no barrier is missed)
    const int c0 = ct * kSmallCols + 4 * l32;
    const int cw = c0 < p.C_in ? c0 : p.C_in - 4;                 // (columns past the end repeat the last ones)

    int row = tile * kSmallRows + l32;
    const bool live = row < rows;
    if (!live) row = rows - 1;
    const int b = row / (ay.n * ax.n), rem = row - b * (ay.n * ax.n);
    const int i = rem / ax.n, j = rem - i * ax.n;
    const int opix = (b * p.H + i * p.stride + ca) * p.Wd + j * p.stride + cb;
    const int gi = i + ay.shift, gj = j + ax.shift;               // gradient position of the class's first tap

    const int pairs = (p.C_out + 2 * CH - 1) / (2 * CH);
    const int steps = ay.count * ax.count * pairs;                // one step: 2 CH channels of one tap
    const int per = (steps + kSmallWaves - 1) / kSmallWaves;
    const int first = wave * per, last = first + per < steps ? first + per : steps;
    const int kstep = p.R * p.S * p.C_in;                         // elements from one output channel of W to the next

    f32x16_t acc[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[u][e] = 0.0f;

    struct Step {
        gptr_t g[NQ];        // this lane's gradient values, eight channels each, or zeros
        gptr_t w[NQ];        // W[channel][tap][cw] of the first of the eight, or zeros
        int kstep[NQ];
        uint64_t e0;
    };
    int tu = 0, tv = 0, pair = 0, step = first;
    if (first < last) pair = first % pairs, tv = first / pairs % ax.count, tu = first / pairs / ax.count;
    // the step the walk stands at, past the last one nothing but zeros; the walk moves on
    auto locate = [&]() {
        const int pp = gi - tu, qq = gj - tv;
        const bool within = step < last;
        const bool in = within && live && (unsigned)pp < (unsigned)p.P && (unsigned)qq < (unsigned)p.Q;
        const int k0 = (pair * 2 + half) * CH;
        const int64_t goff = (int64_t)((b * p.P + pp) * p.Q + qq) * p.C_out + k0;
        const int64_t woff = (int64_t)k0 * kstep + ((ay.r0 + tu * p.stride) * p.S + ax.r0 + tv * p.stride) * p.C_in + cw;
        Step s;
        s.e0 = (uint64_t)goff;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const bool exists = within && k0 + 8 * q < p.C_out;
            s.g[q] = in && exists ? (gptr_t)p.dO + (goff + 8 * q) : (gptr_t)kSmallZeros;
            s.w[q] = exists ? (gptr_t)p.W + (woff + (int64_t)(8 * q) * kstep) : (gptr_t)kSmallZeros;
            s.kstep[q] = exists ? kstep : 0;
        }
        ++step;
        const bool np = ++pair == pairs;
        pair = np ? 0 : pair;
        tv += np ? 1 : 0;
        const bool nt = tv == ax.count;
        tv = nt ? 0 : tv;
        tu += nt ? 1 : 0;
        return s;
    };
    auto load_g = [&](const Step& s, u32x4_t (&g)[NQ]) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) g[q] = *reinterpret_cast<const SDGP_GLOBAL u32x4_t*>(s.g[q]);
    };
    auto load_w = [&](const Step& s, int q, u32x2_t (&w)[8]) {
#pragma unroll
        for (int x = 0; x < 8; ++x) w[x] = *reinterpret_cast<const SDGP_GLOBAL u32x2_t*>(s.w[q] + (int64_t)x * s.kstep[q]);
    };
    auto prune = [&](u32x4_t (&g)[NQ], uint64_t e0) {
        if constexpr (RK == kSmallDense) {
        } else if constexpr (M <= 16) {
            prune16_dense<M, RK, NLE2>(g, p.n, p.mix, e0);
        } else if constexpr (RK != kRandom) {
            uint32_t in[M / 2], out[M / 2];
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int x = 0; x < 4; ++x) in[4 * q + x] = g[q][x];
            prune_packed<M, RK>(in, p.n, out);
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int x = 0; x < 4; ++x) g[q][x] = out[4 * q + x];
        } else {
            uint32_t raw[M], out[M];
            bool keep[M];
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int x = 0; x < 4; ++x) raw[8 * q + 2 * x] = g[q][x] & 0xFFFFu, raw[8 * q + 2 * x + 1] = g[q][x] >> 16;
            prune_group<kBF16, M, RK, NLE2>(raw, p.n, hash_row(p.mix, (uint32_t)(e0 >> 32)), (uint32_t)e0, keep, out);
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int x = 0; x < 4; ++x) g[q][x] = out[8 * q + 2 * x] | (out[8 * q + 2 * x + 1] << 16);
        }
    };

    // Gradient and weights of the next step are in flight during a step; two steps per turn of the loop, so that the
    // register sets change places without copies.
    u32x4_t ga[NQ], gb[NQ];
    u32x2_t w[2][2][8];      // [step parity][matrix step parity][row]: M = 32 has four matrix steps and fetches two late
    Step cur, next;
    auto body = [&](u32x4_t (&g)[NQ], u32x4_t (&gnext)[NQ], auto par) {
        constexpr int PAR = decltype(par)::value;
        next = locate();
        load_g(next, gnext);
        load_w(next, 0, w[PAR ^ 1][0]);
        load_w(next, 1, w[PAR ^ 1][1]);
        __builtin_amdgcn_sched_barrier(0);
        prune(g, cur.e0);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            u32x2_t late[8];
            if (q >= 2) load_w(cur, q, late);
            const u32x2_t(&wq)[8] = q >= 2 ? late : w[PAR][q & 1];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t sel = (u & 1) ? 0x07060302u : 0x05040100u;
                const u32x4_t bv = {__builtin_amdgcn_perm(wq[1][u >> 1], wq[0][u >> 1], sel), __builtin_amdgcn_perm(wq[3][u >> 1], wq[2][u >> 1], sel),
                                    __builtin_amdgcn_perm(wq[5][u >> 1], wq[4][u >> 1], sel), __builtin_amdgcn_perm(wq[7][u >> 1], wq[6][u >> 1], sel)};
                acc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, g[q]), __builtin_bit_cast(bf16x8_t, bv), acc[u], 0, 0, 0);
            }
        }
        cur = next;
    };
    if (first < last) {
        cur = locate();
        load_g(cur, ga);
        load_w(cur, 0, w[0][0]);
        load_w(cur, 1, w[0][1]);
        for (int s = first; s < last; s += 2) {
            body(ga, gb, std::integral_constant<int, 0>{});
            body(gb, ga, std::integral_constant<int, 1>{});
        }
    }

    // every wavefront parks its sums; wavefront w then adds result registers 2w and 2w + 1 over all of them
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    float* const part = reinterpret_cast<float*>(lds);   // [wave][column tile][register][lane]
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < 16; ++e) part[((wave * 4 + u) * 16 + e) * 64 + lane] = acc[u][e];
    __syncthreads();
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const int e = wave * 2 + x;
        const int rr = 8 * (e >> 2) + 4 * half + (e & 3);                   // the row of this result register
        const int pix = __shfl(opix, rr);
        const bool stored = tile * kSmallRows + rr < rows && c0 < p.C_in;
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            v[u] = 0.0f;
#pragma unroll
            for (int k = 0; k < kSmallWaves; ++k) v[u] += part[((k * 4 + u) * 16 + e) * 64 + lane];
        }
        if (__builtin_expect(stored && (v[0] != v[0] || v[1] != v[1] || v[2] != v[2] || v[3] != v[3]), 0)) {
            sum_inside<M, RK>(tile * kSmallRows + rr, c0, v);
        }
        const u32x2_t out = {float2_to_bf16x2(v[0], v[1]), float2_to_bf16x2(v[2], v[3])};
        if (stored) *reinterpret_cast<u32x2_t*>(p.dD + (int64_t)pix * p.C_in + c0) = out;
    }
}

}  // namespace sdgp

// Backward-data kernel for fp32 problems (Fig. 2, Fig. 3; Sec. II-A) on the fp32 matrix instruction
// v_mfma_f32_32x32x2_f32: dL/dD[rows, C_in] = sum over taps of prune(dL/dO)[gathered rows, C_out] . W[:, tap, :], every
// product and sum in fp32.
//
// The instruction takes 64 cycles for two reduction steps of a 32 x 32 tile (154 TFLOP/s on the whole chip: a library
// product of 8192^3), so a wavefront has time for everything else beside it and the kernel needs no LDS: both operands
// are loaded from global memory straight into the registers the instruction reads.
//   * Rows: lane l holds row l % 32.  The half h = l / 32 of a step's two reduction positions is free to choose as long
//     as both operands agree, so half h takes a whole m-group (two of four channels): a lane's gradient values are consecutive
//     channels of one pixel, four per 16-byte load, and the group is ranked (Sec. III-B) in that lane's registers with
//     nothing exchanged.
//   * Columns: lane l of column tile j holds column CN * (l % 32) + j, so the CN tiles of a reduction position come from
//     one load of CN consecutive channels of W in its native layout, and the result of a row leaves as CN consecutive
//     values per lane: whole 128- or 512-byte runs.
//   * A wavefront owns 32 rows x 32 CN columns.  WK = 1: the WV wavefronts of a workgroup take consecutive row tiles of
//     one column block (they read the same W through the L1).  WK > 1 (few tiles): the wavefronts share a tile, split
//     the reduction and add their sums through LDS in a fixed order.
// Bound by the matrix pipe's issue: 3x3 128 -> 128 channels at 16x16, batch 128, 2:4 Magnitude 99 us = 98 TFLOP/s (20151
// us with one thread per element; 195 us while every step waited for its own loads); linear 256 x 128 -> 256 67 -> 10.5
// us back to back.
// Strided filters: blockIdx.z is the parity class of the input pixels, whose taps are a sub-grid of the filter.
// Taps outside the gradient and rows past the end multiply zeros.  Zero times a non-finite weight is NaN where the
// definition has no term at all, so a NaN result of a row that has such taps is summed again with those taps left out.
#pragma once

#include <type_traits>

#include "parity_axis.h"
#include "ranker.h"

namespace sdgp {

typedef float f32v2_t __attribute__((ext_vector_type(2)));
typedef float f32v4_t __attribute__((ext_vector_type(4)));
typedef float f32v16_t __attribute__((ext_vector_type(16)));

#define SDGP_GLOBAL __attribute__((address_space(1)))

constexpr int kDenseRanker = 3;   // n == m: nothing is ranked

// What a lane reads instead of a gradient group outside the gradient or a weight of a group past the last one: the loads
// need no branch and no select behind them, either of which would wait for the data in front of the multiplies.
static __device__ const float kF32Zeros[32] __attribute__((aligned(128))) = {};

struct F32Params {
    const float* dO;
    const float* W;
    float* dD;
    int64_t B, H, Wd, P, Q, C_in, C_out;
    int R, S, stride, pad, n;
    uint32_t mix;
};

// raw[0..M) of the group that starts at flat element e0 -> the pruned values
template <int M, int RK, bool NLE2>
__device__ __forceinline__ void prune_f32(uint32_t (&raw)[M], int n, uint32_t mix, uint64_t e0) {
    if constexpr (RK != kDenseRanker) {
        bool keep[M];
        uint32_t out[M];
        prune_group<kF32, M, RK, NLE2>(raw, n, hash_row(mix, (uint32_t)(e0 >> 32)), (uint32_t)e0, keep, out);
#pragma unroll
        for (int j = 0; j < M; ++j) raw[j] = out[j];
    }
}

// The CN stored results of row `row` at channel c0, some of them NaN: where taps of the row lie outside the gradient, the NaNs
// are summed again over the taps inside.  It reads the kernel's arguments again, so that nothing of it is kept in registers
// during the main loop.
template <int M, int RK, bool NLE2, int CN>
__device__ __forceinline__ void sum_inside_f32(int64_t row, int64_t c0) {
    typedef float vcn_t __attribute__((ext_vector_type(CN)));
    uint64_t args = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    const auto& p = *reinterpret_cast<const __attribute__((address_space(4))) F32Params*>(args);
    const int ca = (int)(blockIdx.z / p.stride), cb = (int)(blockIdx.z % p.stride);
    const ParityAxis<int64_t> ay = parity_axis<int64_t>(p.H, p.R, p.stride, p.pad, ca), ax = parity_axis<int64_t>(p.Wd, p.S, p.stride, p.pad, cb);
    const int64_t b = row / (ay.n * ax.n), rem = row - b * (ay.n * ax.n), i = rem / ax.n, j = rem - i * ax.n;
    const int64_t gi = i + ay.shift, gj = j + ax.shift;
    if (gi < p.P && gi - ay.count >= -1 && gj < p.Q && gj - ax.count >= -1) return;   // every tap inside: a NaN of its own
    float* const at = p.dD + ((b * p.H + i * p.stride + ca) * p.Wd + j * p.stride + cb) * p.C_in + c0;
    const vcn_t v = *reinterpret_cast<const vcn_t*>(at);
    vcn_t sum = vcn_t(0.0f);
    const int64_t kstep = (int64_t)p.R * p.S * p.C_in;
    bool open = true;   // some NaN result may still turn out not to be one: a NaN of the taps inside stays one
#pragma nounroll
    for (int t = 0; t < ay.count * ax.count && open; ++t) {
        const int u = t / ax.count, s = t - u * ax.count;
        const int64_t pp = gi - u, qq = gj - s;
        if (pp < 0 || pp >= p.P || qq < 0 || qq >= p.Q) continue;
        const uint64_t e0 = (uint64_t)(((b * p.P + pp) * p.Q + qq) * p.C_out);
        const float* w = p.W + (((int64_t)(ay.r0 + u * p.stride) * p.S + ax.r0 + s * p.stride) * p.C_in + c0);
#pragma nounroll
        for (int64_t k = 0; k < p.C_out && open; k += M) {
            uint32_t raw[M];
#pragma unroll
            for (int y = 0; y < M; ++y) raw[y] = float_to_bits(p.dO[e0 + k + y]);
            prune_f32<M, RK, NLE2>(raw, p.n, p.mix, e0 + (uint64_t)k);
#pragma unroll
            for (int y = 0; y < M; ++y) sum += bits_to_float(raw[y]) * *reinterpret_cast<const vcn_t*>(w + (k + y) * kstep);
            open = false;
#pragma unroll
            for (int x = 0; x < CN; ++x) open = open || (v[x] != v[x] && sum[x] == sum[x]);
        }
    }
    vcn_t out;
#pragma unroll
    for (int x = 0; x < CN; ++x) out[x] = v[x] != v[x] ? sum[x] : v[x];
    *reinterpret_cast<vcn_t*>(at) = out;
}

template <int M, int RK, bool NLE2, int CN, int WV, int WK>
__global__ void __launch_bounds__(64 * WV, CN == 2 ? 2 : 1) bwd_f32(const F32Params p) {
    static_assert(WK == 1 || WK == WV, "the wavefronts share rows or the reduction");
    static_assert(M % 4 == 0 && (CN == 2 || CN == 4), "16-byte gradient loads, 8- or 16-byte weight loads");
    constexpr int CH = M > 8 ? M : 8;   // channels per lane and step: one group, or two of four
    constexpr int JS = CH / 4;          // sub-steps of 4 channels
    typedef float vcn_t __attribute__((ext_vector_type(CN)));
    typedef const SDGP_GLOBAL float* gptr_t;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int ca = (int)(blockIdx.z / p.stride), cb = (int)(blockIdx.z % p.stride);
    const ParityAxis<int64_t> ay = parity_axis<int64_t>(p.H, p.R, p.stride, p.pad, ca), ax = parity_axis<int64_t>(p.Wd, p.S, p.stride, p.pad, cb);
    const int64_t rows = p.B * ay.n * ax.n;
    const int64_t tile = (int64_t)blockIdx.x * (WK == 1 ? WV : 1) + (WK == 1 ? wave : 0);
    if (tile * 32 >= rows) return;   // (with WK > 1 the whole workgroup leaves: no barrier is missed)
    const int64_t c0 = (int64_t)blockIdx.y * (32 * CN) + CN * l32;          // this lane's first column
    const int64_t cw = c0 < p.C_in ? c0 : p.C_in - CN;                      // (columns past the end repeat the last ones)

    // this lane's row: image, position in the class
    int64_t row = tile * 32 + l32;
    const bool live = row < rows;
    if (!live) row = rows - 1;
    const int64_t b = row / (ay.n * ax.n), rem = row % (ay.n * ax.n);
    const int64_t i = rem / ax.n, j = rem % ax.n;
    const int64_t opix = (b * p.H + i * p.stride + ca) * p.Wd + j * p.stride + cb;

    const int ntaps = ay.count * ax.count;
    const int npairs = (int)((p.C_out + 2 * CH - 1) / (2 * CH));
    const int steps = ntaps * npairs;                                       // one step: 2 CH channels of one tap
    const int per = (steps + WK - 1) / WK;
    const int first = WK == 1 ? 0 : wave * per, last = WK == 1 ? steps : (first + per < steps ? first + per : steps);
    const int kstep = p.R * p.S * (int)p.C_in;                              // elements from one output channel of W to the next
    const int gi = (int)i + ay.shift, gj = (int)j + ax.shift;               // gradient position of the class's first tap
    const int P = (int)p.P, Q = (int)p.Q, C_out = (int)p.C_out;
    const int64_t image = b * p.P * p.Q * p.C_out;                          // (an image and the filter are below 2^31 elements)

    f32v16_t acc[CN];
#pragma unroll
    for (int u = 0; u < CN; ++u)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[u][e] = 0.0f;

    struct Step {
        gptr_t g[JS];         // this lane's gradient values, four channels each, or zeros
        gptr_t w[JS];         // W[channel][tap][cw] of the first of the four, or zeros
        int kstep[JS];        // elements from one channel's weights to the next
        uint64_t e0;
    };
    // where the walk over (tap row, tap column, channels) stands: uniform over the wavefront
    int tu = 0, tv = 0, pair = 0, step = first;
    if constexpr (WK > 1) {
        if (first < last) pair = first % npairs, tv = (first / npairs) % ax.count, tu = first / npairs / ax.count;
    }
    // the step the walk stands at, past the last one nothing but zeros; the walk moves on
    auto locate = [&]() {
        const int pp = gi - tu, qq = gj - tv;
        const bool in = (unsigned)pp < (unsigned)P && (unsigned)qq < (unsigned)Q;
        const bool within = step < last;
        const int k0 = (pair * 2 + half) * CH;
        const int goff = (pp * Q + qq) * C_out + k0;
        const int woff = k0 * kstep + ((ay.r0 + tu * p.stride) * p.S + ax.r0 + tv * p.stride) * (int)p.C_in + (int)cw;
        Step s;
        s.e0 = (uint64_t)(image + goff);
#pragma unroll
        for (int q = 0; q < JS; ++q) {
            const bool exists = within && k0 + 4 * q < C_out;
            s.g[q] = in && live && exists ? (gptr_t)p.dO + (image + goff + 4 * q) : (gptr_t)kF32Zeros;
            s.w[q] = exists ? (gptr_t)p.W + (woff + 4 * q * kstep) : (gptr_t)kF32Zeros;
            s.kstep[q] = exists ? kstep : 0;
        }
        ++step;
        const bool np = ++pair == npairs;
        pair = np ? 0 : pair;
        tv += np ? 1 : 0;
        const bool nt = tv == ax.count;
        tv = nt ? 0 : tv;
        tu += nt ? 1 : 0;
        return s;
    };
    auto load_g = [&](const Step& s, uint32_t (&raw)[CH]) {
#pragma unroll
        for (int q = 0; q < JS; ++q) {
            const f32v4_t v = *reinterpret_cast<const SDGP_GLOBAL f32v4_t*>(s.g[q]);
#pragma unroll
            for (int x = 0; x < 4; ++x) raw[4 * q + x] = float_to_bits(v[x]);
        }
    };
    auto load_w = [&](const Step& s, int q, vcn_t (&w)[4]) {
#pragma unroll
        for (int x = 0; x < 4; ++x) w[x] = *reinterpret_cast<const SDGP_GLOBAL vcn_t*>(s.w[q] + x * s.kstep[q]);
    };

    // The gradient of the next step is in flight during a step, the weights of the two sub-steps after the current one
    // during a sub-step (4 CN matrix instructions, 64 cycles each): no load is waited for behind its own request.  Two
    // steps per turn of the loop, so that the register sets change places without copies; an odd last one is followed by
    // a step of zeros.
    constexpr int RING = 4;
    vcn_t w[RING][4];
    uint32_t ga[CH], gb[CH];
    Step cur, next;
    auto body = [&](uint32_t (&g)[CH], uint32_t (&gnext)[CH], auto par) {
        constexpr int W0 = (decltype(par)::value * JS) % RING;
        next = locate();
        load_g(next, gnext);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < JS; ++q) {
            if (q + 2 < JS) load_w(cur, q + 2, w[(W0 + q + 2) % RING]);
            else load_w(next, q + 2 - JS, w[(W0 + q + 2) % RING]);
            __builtin_amdgcn_sched_barrier(0);
            if (q % (M / 4) == 0) {
                uint32_t grp[M];
#pragma unroll
                for (int x = 0; x < M; ++x) grp[x] = g[4 * q + x];
                prune_f32<M, RK, NLE2>(grp, p.n, p.mix, cur.e0 + (uint64_t)(4 * q));
#pragma unroll
                for (int x = 0; x < M; ++x) g[4 * q + x] = grp[x];
            }
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int u = 0; u < CN; ++u)
                    acc[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(bits_to_float(g[4 * q + x]), w[(W0 + q) % RING][x][u], acc[u], 0, 0, 0);
        }
        cur = next;
    };
    if (first < last) {
        cur = locate();
        load_g(cur, ga);
        load_w(cur, 0, w[0]);
        load_w(cur, 1, w[1]);
        for (int s = first; s < last; s += 2) {
            body(ga, gb, std::integral_constant<int, 0>{});
            body(gb, ga, std::integral_constant<int, 1>{});
        }
    }

    if constexpr (WK > 1) {
        // every wavefront parks its sums; wavefront w then adds result registers w, w + WK, ... over all of them
        static_assert(16 % WK == 0, "the result registers are dealt evenly");
        __shared__ float part[WK][CN][16][64];
#pragma unroll
        for (int u = 0; u < CN; ++u)
#pragma unroll
            for (int e = 0; e < 16; ++e) part[wave][u][e][lane] = acc[u][e];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < CN; ++u)
#pragma unroll
            for (int x = 0; x < 16 / WK; ++x) {
                float sum = 0.0f;
#pragma unroll
                for (int k = 0; k < WK; ++k) sum += part[k][u][wave * (16 / WK) + x][lane];
                acc[u][x] = sum;
            }
    }

    uint32_t nans = 0;   // which of this lane's results hold a NaN
#pragma unroll
    for (int x = 0; x < 16 / WK; ++x) {
        const int e = WK == 1 ? x : wave * (16 / WK) + x;
        const int rr = 8 * (e >> 2) + 4 * half + (e & 3);                   // the row of this result register
        const int64_t pix = __shfl(opix, rr);
        if (tile * 32 + rr >= rows || c0 >= p.C_in) continue;
        vcn_t v;
        bool nan = false;
#pragma unroll
        for (int u = 0; u < CN; ++u) v[u] = acc[u][x], nan = nan || v[u] != v[u];
        nans |= (uint32_t)nan << x;
        *reinterpret_cast<vcn_t*>(p.dD + pix * p.C_in + c0) = v;
    }
    if (__builtin_expect(nans != 0, 0)) {
        for (; nans != 0; nans &= nans - 1) {
            const int e = (WK == 1 ? 0 : wave * (16 / WK)) + __ffs((int)nans) - 1;
            sum_inside_f32<M, RK, NLE2, CN>(tile * 32 + 8 * (e >> 2) + 4 * half + (e & 3), c0);
        }
    }
}

}  // namespace sdgp

// Backward-data kernel for fp32 problems (Fig. 2, Fig. 3; Sec. II-A) on the fp32 matrix instruction
// v_mfma_f32_32x32x2_f32: dL/dD[rows, C_in] = sum over taps of prune(dL/dO)[gathered rows, C_out] . W[:, tap, :], every
// product and sum in fp32.
//
// The instruction takes 64 cycles for two reduction steps of a 32 x 32 tile (154 TFLOP/s on the whole chip: a library
// product of 8192^3), so a wavefront has time for everything else beside it and the kernel needs no LDS: both operands
// are loaded from global memory straight into the registers the instruction reads.
//   * Rows: lane l holds row l % 32.  The half h = l / 32 of a step's two reduction positions is free to choose as long
//     as both operands agree, so half h takes the whole m-group 2g + h: a lane's gradient values are M consecutive
//     channels of one pixel, four per 16-byte load, and the group is ranked (Sec. III-B) in that lane's registers with
//     nothing exchanged.
//   * Columns: lane l of column tile j holds column CN * (l % 32) + j, so the CN tiles of a reduction position come from
//     one load of CN consecutive channels of W in its native layout, and the result of a row leaves as CN consecutive
//     values per lane: whole 128- or 512-byte runs.
//   * A wavefront owns 32 rows x 32 CN columns.  WK = 1: the WV wavefronts of a workgroup take consecutive row tiles of
//     one column block (they read the same W through the L1).  WK > 1 (few tiles): the wavefronts share a tile, split
//     the reduction and add their sums through LDS in a fixed order.
// Strided filters: blockIdx.z is the parity class of the input pixels, whose taps are a sub-grid of the filter.
// Taps outside the gradient and rows past the end multiply zeros.  Zero times a non-finite weight is NaN where the
// definition has no term at all, so a result that is NaN is summed again element by element with those taps left out.
#pragma once

#include "ranker.h"

namespace sdgp {

typedef float f32v2_t __attribute__((ext_vector_type(2)));
typedef float f32v4_t __attribute__((ext_vector_type(4)));
typedef float f32v16_t __attribute__((ext_vector_type(16)));

constexpr int kDenseRanker = 3;   // n == m: nothing is ranked

struct F32Params {
    const float* dO;
    const float* W;
    float* dD;
    int64_t B, H, Wd, P, Q, C_in, C_out;
    int R, S, stride, pad, n;
    uint32_t mix;
};

// One parity class of input pixels along one axis: pixel i*stride + a meets filter positions r0, r0 + stride, ...
// (count of them) at gradient positions i + shift, i + shift - 1, ...
struct F32Axis {
    int r0, count, shift;
    int64_t n;
};
__device__ __forceinline__ F32Axis f32_axis(int64_t size, int filter, int stride, int pad, int a) {
    F32Axis x;
    x.r0 = (a + pad) % stride;
    x.count = x.r0 < filter ? (filter - x.r0 + stride - 1) / stride : 0;
    x.shift = (a + pad - x.r0) / stride;
    x.n = size > a ? (size - a + stride - 1) / stride : 0;
    return x;
}

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

template <int M, int RK, bool NLE2, int CN, int WV, int WK>
__global__ void __launch_bounds__(64 * WV) bwd_f32(const F32Params p) {
    static_assert(WK == 1 || WK == WV, "the wavefronts share rows or the reduction");
    static_assert(M % 4 == 0 && (CN == 2 || CN == 4), "16-byte gradient loads, 8- or 16-byte weight loads");
    constexpr int JS = M / 4;   // reduction sub-steps of 4 channels per half
    typedef float vcn_t __attribute__((ext_vector_type(CN)));
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int ca = (int)(blockIdx.z / p.stride), cb = (int)(blockIdx.z % p.stride);
    const F32Axis ay = f32_axis(p.H, p.R, p.stride, p.pad, ca), ax = f32_axis(p.Wd, p.S, p.stride, p.pad, cb);
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
    const int64_t ngroups = p.C_out / M;
    const int npairs = (int)((ngroups + 1) / 2);
    const int steps = ntaps * npairs;                                       // one step: a pair of groups of one tap
    const int per = (steps + WK - 1) / WK;
    const int first = WK == 1 ? 0 : wave * per, last = WK == 1 ? steps : (first + per < steps ? first + per : steps);
    const int64_t kstep = (int64_t)p.R * p.S * p.C_in;                      // elements from one output channel of W to the next

    f32v16_t acc[CN];
#pragma unroll
    for (int u = 0; u < CN; ++u)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[u][e] = 0.0f;

    // position of a step, advanced without divisions
    struct At {
        int tap, pair;
    };
    struct Step {
        const float* g;       // this lane's gradient group, or null: zeros
        const float* w;       // W[first channel of the group][tap][cw]
        uint64_t e0;
        bool wok;             // the group exists
    };
    bool outside = false;     // some tap of this lane's row lies outside the gradient
    auto locate = [&](const At& a) {
        const int u = a.tap / ax.count, v = a.tap - u * ax.count;
        const int64_t pp = i + ay.shift - u, qq = j + ax.shift - v;
        const bool in = pp >= 0 && pp < p.P && qq >= 0 && qq < p.Q;
        outside |= !in;
        const int64_t grp = 2 * (int64_t)a.pair + half;
        Step s;
        s.wok = grp < ngroups;
        const int64_t gr = s.wok ? grp : ngroups - 1;
        s.e0 = (uint64_t)(((b * p.P + pp) * p.Q + qq) * p.C_out + gr * M);
        s.g = in && live && s.wok ? p.dO + s.e0 : nullptr;
        s.w = p.W + (gr * M * kstep + ((int64_t)(ay.r0 + u * p.stride) * p.S + ax.r0 + v * p.stride) * p.C_in + cw);
        return s;
    };
    auto advance = [&](At& a) {
        if (++a.pair == npairs) a.pair = 0, ++a.tap;
    };
    auto load_g = [&](const Step& s, uint32_t (&raw)[M]) {
#pragma unroll
        for (int q = 0; q < JS; ++q) {
            f32v4_t v = {0.0f, 0.0f, 0.0f, 0.0f};
            if (s.g != nullptr) v = *reinterpret_cast<const f32v4_t*>(s.g + 4 * q);
#pragma unroll
            for (int x = 0; x < 4; ++x) raw[4 * q + x] = float_to_bits(v[x]);
        }
    };
    auto load_w = [&](const Step& s, int q, vcn_t (&w)[4]) {
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            w[x] = *reinterpret_cast<const vcn_t*>(s.w + (4 * q + x) * kstep);
            if (!s.wok) w[x] = vcn_t(0.0f);
        }
    };

    if (first < last) {
        At at{first / npairs, first % npairs};
        Step cur = locate(at);
        uint32_t g[M], gnext[M];
        vcn_t w[2][4];
        load_g(cur, g);
        load_w(cur, 0, w[0]);
        for (int s = first; s < last; ++s) {
            advance(at);
            const bool more = s + 1 < last;
            const Step next = more ? locate(at) : cur;
            if (more) load_g(next, gnext);
            prune_f32<M, RK, NLE2>(g, p.n, p.mix, cur.e0);
#pragma unroll
            for (int q = 0; q < JS; ++q) {
                // the weights of the next sub-step are in flight while this one is multiplied
                if constexpr (JS % 2 == 0) {
                    if (q + 1 < JS) load_w(cur, q + 1, w[(q + 1) & 1]);
                    else if (more) load_w(next, 0, w[0]);
#pragma unroll
                    for (int x = 0; x < 4; ++x)
#pragma unroll
                        for (int u = 0; u < CN; ++u)
                            acc[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(bits_to_float(g[4 * q + x]), w[q & 1][x][u], acc[u], 0, 0, 0);
                } else {   // one sub-step per step: the two register sets change places by copying
                    vcn_t wn[4];
                    if (more) load_w(next, 0, wn);
#pragma unroll
                    for (int x = 0; x < 4; ++x)
#pragma unroll
                        for (int u = 0; u < CN; ++u)
                            acc[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(bits_to_float(g[x]), w[0][x][u], acc[u], 0, 0, 0);
#pragma unroll
                    for (int x = 0; x < 4; ++x) w[0][x] = wn[x];
                }
            }
            cur = next;
#pragma unroll
            for (int x = 0; x < M; ++x) g[x] = gnext[x];
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

    const bool redo_taps = ntaps > 0 && __any(outside) != 0;
#pragma unroll
    for (int x = 0; x < 16 / WK; ++x) {
        const int e = WK == 1 ? x : wave * (16 / WK) + x;
        const int rr = 8 * (e >> 2) + 4 * half + (e & 3);                   // the row of this result register
        const int64_t pix = __shfl(opix, rr);
        if (tile * 32 + rr >= rows || c0 >= p.C_in) continue;
        vcn_t v;
#pragma unroll
        for (int u = 0; u < CN; ++u) v[u] = acc[u][x];
        if (WK > 1 || redo_taps) {
            bool nan = false;
#pragma unroll
            for (int u = 0; u < CN; ++u) nan = nan || v[u] != v[u];
            if (nan && (p.R > 1 || p.S > 1)) {
                const int64_t r2 = tile * 32 + rr, b2 = r2 / (ay.n * ax.n), m2 = r2 % (ay.n * ax.n), i2 = m2 / ax.n, j2 = m2 % ax.n;
                v = vcn_t(0.0f);
                for (int u = 0; u < ay.count; ++u)
                    for (int t = 0; t < ax.count; ++t) {
                        const int64_t pp = i2 + ay.shift - u, qq = j2 + ax.shift - t;
                        if (pp < 0 || pp >= p.P || qq < 0 || qq >= p.Q) continue;
                        const uint64_t e0 = (uint64_t)(((b2 * p.P + pp) * p.Q + qq) * p.C_out);
                        const float* w = p.W + (((int64_t)(ay.r0 + u * p.stride) * p.S + ax.r0 + t * p.stride) * p.C_in + c0);
                        for (int64_t k = 0; k < p.C_out; k += M) {
                            uint32_t raw[M];
#pragma unroll
                            for (int y = 0; y < M; ++y) raw[y] = float_to_bits(p.dO[e0 + k + y]);
                            prune_f32<M, RK, NLE2>(raw, p.n, p.mix, e0 + (uint64_t)k);
#pragma unroll
                            for (int y = 0; y < M; ++y) v += bits_to_float(raw[y]) * *reinterpret_cast<const vcn_t*>(w + (k + y) * kstep);
                        }
                    }
            }
        }
        *reinterpret_cast<vcn_t*>(p.dD + pix * p.C_in + c0) = v;
    }
}

}  // namespace sdgp

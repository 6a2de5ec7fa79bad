// fp32 backward-data products on the bf16 matrix instructions (Fig. 2, Fig. 3; Sec. II-A), for problems large enough to
// pay for a pass over the operands.
//
// An fp32 value is the sum of three bf16 values: the nearest one, the one nearest to what is left, which is at most 2^-8 of the
// whole, and the rest, at most 2^-17 and exact.  A product of two such sums is nine bf16 products, each exact in fp32; the
// three smallest are together at most 2^-24 of the whole, of either sign, and are left out.  So six bf16 instructions replace
// the fp32 one, which takes 16 times as long for the same work, and every sum stays fp32, in fewer steps.  Operands are scaled by
// 2^24 on the way in and results by 2^-48 on the way out, so that parts of the smallest values are normal numbers too.
// The products of the first parts and the five smaller ones have sums of their own, so that a sum that counts is rounded once per
// chunk and tap.  Error against 64 bits over that of the fp32 instruction, 762 products of 4 to 4608 terms, three distributions:
// 0.05 to 0.81 (3x3 128 -> 128 at 16x16, batch 128, 2:4 Magnitude 1.3e-7 against 4.1e-7; parts by truncation, whose loss is
// towards zero, and one sum: 3.6e-7 there, up to 12 times the fp32 instruction's on same-sign data).
//   1. split_operands ranks the gradient (Sec. III-B) and writes its three planes -- kept values only, with their
//      positions, where at most two of four channels stay -- and W's, in the order in which the product reads its fragments.
//      Bound by latency and memory: 6.3 us there.
//   2. f32_split multiplies: a workgroup of 16 (8) wavefronts owns 256 (128) rows x 64 columns of one parity class of the
//      input pixels, a wavefront 32 x 32.  Per chunk of channels the gradient positions its taps reach come into LDS once (a
//      grid with the image's borders as zeros, so that a tap is a constant distance); W's slabs of one to three taps per
//      stage pass through a ring of three sets; everything by direct-to-LDS copies, a stage ahead of the stage before its
//      use, so that a wavefront requests a stage's first fragments before its barrier.  64 columns and 256 rows move the
//      fewest bytes per multiplication that still give 256 workgroups to ResNet-9's 3x3 layers at batch 128.
//      Bound by fragment reads and matrix instructions, which take equal time and overlap by half: 7 us per 32 channels
//      and nine taps, 10 us of prologue, first copies and stores.
// 3x3 128 -> 128 at 16x16, batch 128, 2:4 Magnitude: 96.6 us on the fp32 instruction, 43.4 here.
// Values that scaling takes out of the range, infinite and NaN ones have parts that make NaN of every result they reach
// (split3), and sums may leave the range on the way: where split_operands notes an operand that can have done so, results that are
// not finite are summed again term by term.  (A NaN gradient alone costs nothing: its NaN is the result.)  A dropped channel meets
// no weight here, where the definition multiplies it by zero: the columns of W with a non-finite weight are noted too, and
// summed again.
#pragma once

#include "bwd_f32.h"
#include "lds_copy.h"

#define SDGP_CONSTANT __attribute__((address_space(4)))

namespace sdgp {

struct SplitParams {
    const float* dO;
    const float* W;
    float* dD;
    // the workspace
    unsigned char* planes;   // [chunk][plane][half][pixel] 16 bytes: 8 bf16
    uint16_t* idx;           // [chunk][pixel][half] 2-bit positions (compressed planes)
    unsigned char* wimg;     // [64 columns][32 channels][part][slot][32 columns][plane][lane] 16 bytes; slot: the filter's taps
                             // class by class, so that a stage's slabs lie behind each other
    uint32_t* wnotes;        // [64 columns][32 channels][part][slot][32 columns] two words: bit c set, column c has a non-finite
                             // weight there; not zero, a weight is large
    uint32_t* gnotes;        // one word per workgroup of the first pass that has gradient: a large value is kept
    int64_t npix;
    int B, H, Wd, P, Q, C_in, C_out, R, S, stride, pad, n;
    uint32_t mix;
    int gblocks, wblocks, nchunks, nc32;
    int TB, TH, TW, tiles_h, tiles_w, ntiles_n, nblocks;
    int slot0[16];           // class_slots
};

// W's slots hold the taps of one parity class after another, so that a stage's slabs lie behind each other: class i has the taps
// that begin at filter position (i / stride, i % stride), row by row, from slot0[i] on.  A filter narrower than the stride
// leaves classes without taps, which begin where the next class does.
__host__ __device__ __forceinline__ void class_slots(int R, int S, int stride, int (&slot0)[16]) {
    for (int i = 0, at = 0; i < stride * stride; ++i) {
        slot0[i] = at;
        const int r0 = i / stride, s0 = i % stride;
        at += (r0 < R ? (R - r0 + stride - 1) / stride : 0) * (s0 < S ? (S - s0 + stride - 1) / stride : 0);
    }
}
// The tap (r, s) of a slot: of the last class with taps that begins at or before it.
__host__ __device__ __forceinline__ void slot_tap(const int (&slot0)[16], int R, int S, int stride, int slot, int& r, int& s) {
    int cl = 0;   // (always has taps)
    for (int i = 1; i < stride * stride; ++i) cl = i / stride < R && i % stride < S && slot0[i] <= slot ? i : cl;
    const int nx = (S - cl % stride + stride - 1) / stride;
    r = cl / stride + (slot - slot0[cl]) / nx * stride, s = cl % stride + (slot - slot0[cl]) % nx * stride;
}

// Grid positions along one side of a tile of `side` pixels whose class has `count` taps on that axis.  (A class without taps
// copies none; a side of at least one position keeps the divisions by it defined.)
__host__ __device__ __forceinline__ int grid_side(int side, int count) { return count > 0 ? side + count - 1 : side; }

constexpr int kSlab = 6 * 1024;       // W for one tap, 16 channels and 64 columns: 2 column tiles x 3 planes

// Tile of ROWS rows on a grid of at most NP positions (64 per wavefront: one copy unit each); W: three sets of kGroup taps.
template <bool SPARSE, int ROWS, int NP>
struct SplitLayout {
    static constexpr int kParts = SPARSE ? 2 : 1;                   // 16 channels each
    static constexpr int kPlane = NP * 16;                          // one plane's half chunk
    static constexpr int kABytes = 6 * kPlane + (SPARSE ? NP * 4 : 0);
    static constexpr int kGroup = SPARSE ? (NP > 384 ? 1 : 2) : 3;  // taps per stage
    static constexpr int kWSet = kParts * kGroup * kSlab;
    static constexpr int kOffA = ROWS * 4 + 64;                     // behind the row table and the notes
    static constexpr int kOffW = kOffA + 2 * kABytes;
    static constexpr int kTotal = kOffW + 3 * kWSet;
    static_assert(kTotal <= 160 * 1024 && NP <= 512, "fits the LDS, and eight wavefronts copy it");
};

// An operand's scale: parts of the smallest fp32 value are then normal numbers of bf16, whatever the instructions do with others.
constexpr float kSplitScale = 0x1p24f, kSplitUnscale = 0x1p-48f;

struct Split3 {
    uint32_t h, m, l;   // fp32 patterns whose lower halves are zero: x 2^24 = h + m + l
};
// A value that bf16 cannot hold then (infinite, NaN, from 2^104 on) has a NaN for h, which makes NaN of every result it reaches,
// and its own two halves for m and l (split_join).
__host__ __device__ __forceinline__ Split3 split3(uint32_t x) {
    auto nearest = [](uint32_t u) { return (u + 0x7FFFu + ((u >> 16) & 1u)) & 0xFFFF0000u; };
    const float v = bits_to_float(x) * kSplitScale;
    Split3 s;
    s.h = nearest(float_to_bits(v));
    const float rest = v - bits_to_float(s.h);
    s.m = nearest(float_to_bits(rest));
    s.l = float_to_bits(rest - bits_to_float(s.m));   // (at most seven bits are left)
    if ((s.h & 0x7F800000u) == 0x7F800000u || (x & 0x7F800000u) == 0x7F800000u) s.h = 0x7FC00000u, s.m = x & 0xFFFF0000u, s.l = x << 16;
    return s;
}
// From 2^24 on, and infinite.  Without such operands no sum leaves the range: products are below 2^48, and a filter has fewer than
// 2^27 taps and channels, which makes less than 2^75, scaled 2^123.
__host__ __device__ __forceinline__ bool is_large(uint32_t x) { return (x & 0x7FFFFFFFu) - 0x4B800000u <= 0x7F800000u - 0x4B800000u; }
// The value of three parts given as bf16.
__host__ __device__ __forceinline__ float split_join(uint32_t h, uint32_t m, uint32_t l) {
    if (h == 0x7FC0u) return bits_to_float(m << 16 | l);
    return (bits_to_float(l << 16) + bits_to_float(m << 16) + bits_to_float(h << 16)) * (1.0f / kSplitScale);
}
// eight values -> eight bf16 of each plane
__device__ __forceinline__ void split8(const uint32_t (&x)[8], u32x4_t (&out)[3]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const Split3 a = split3(x[2 * i]), b = split3(x[2 * i + 1]);
        out[0][i] = __builtin_amdgcn_perm(b.h, a.h, 0x07060302u);
        out[1][i] = __builtin_amdgcn_perm(b.m, a.m, 0x07060302u);
        out[2][i] = __builtin_amdgcn_perm(b.l, a.l, 0x07060302u);
    }
}

// First pass.  Workgroups below wblocks: one (tap, 32 channels, 32 columns, part) of W per wavefront.  The others: 64 channels
// of 256 / (64 / IC) pixels at a time, IC channels per thread, so that the threads of a pixel read 256 consecutive bytes
// and those of a channel group write 16 consecutive bytes per pixel.
template <int M, int RK, bool NLE2, bool SPARSE>
__global__ void __launch_bounds__(256) split_operands(const SplitParams p) {
    if ((int)blockIdx.x < p.wblocks) {
        const int lane = threadIdx.x & 63, taps = p.R * p.S;
        const int unit = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // (slab, column tile)
        if (unit >= p.ntiles_n * p.nc32 * 2 * taps * 2) return;
        const int slab = unit >> 1, slot = slab % taps, part = slab / taps & 1, c32 = slab / taps / 2 % p.nc32, nt = slab / taps / 2 / p.nc32;
        int r, q;
        slot_tap(p.slot0, p.R, p.S, p.stride, slot, r, q);
        const int col = nt * 64 + (unit & 1) * 32 + (lane & 31), k0 = c32 * 32 + part * 16 + (lane >> 5) * 8;
        uint32_t x[8];
        bool bad = false, large = false;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            x[j] = 0u;
            if (k0 + j < p.C_out && col < p.C_in) x[j] = float_to_bits(p.W[((size_t)(k0 + j) * taps + r * p.S + q) * p.C_in + col]);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) bad = bad || (x[j] & 0x7F800000u) == 0x7F800000u, large = large || is_large(x[j]);
        u32x4_t out[3];
        split8(x, out);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<u32x4_t*>(p.wimg + ((size_t)unit * 3 + pl) * 1024 + lane * 16) = out[pl];
        const uint64_t cols = __ballot(bad), larges = __ballot(large);
        if (lane == 0) p.wnotes[2 * unit] = (uint32_t)cols | (uint32_t)(cols >> 32), p.wnotes[2 * unit + 1] = larges != 0;
        return;
    }
    constexpr int IC = M > 16 ? M : 16;               // channels per thread
    constexpr int TPP = 64 / IC, PX = 256 / TPP;      // threads per pixel, pixels at a time
    const int wg = (int)blockIdx.x - p.wblocks;
    const uint32_t cblocks = (uint32_t)(p.C_out + 63) / 64u, tiles = (uint32_t)((p.npix + PX - 1) / PX) * cblocks;   // (below 2^31)
    bool large = false;
    for (uint32_t t = (uint32_t)wg; t < tiles; t += (uint32_t)p.gblocks) {
        const int64_t pix = (int64_t)(t / cblocks) * PX + threadIdx.x / TPP;
        const int ch = (int)(t % cblocks) * 64 + (int)(threadIdx.x % TPP) * IC;
        if (pix >= p.npix || ch >= p.nchunks * (SPARSE ? 32 : 16)) continue;
        uint32_t raw[IC];
        const uint64_t e0 = (uint64_t)pix * (uint32_t)p.C_out + (uint32_t)ch;
#pragma unroll
        for (int q = 0; q < IC / 4; ++q) {
            u32x4_t v = {0u, 0u, 0u, 0u};
            if (ch + 4 * q < p.C_out) v = *reinterpret_cast<const u32x4_t*>(p.dO + e0 + 4 * q);
#pragma unroll
            for (int x = 0; x < 4; ++x) raw[4 * q + x] = v[x];
        }
        uint32_t keep = 0;   // one bit per channel
#pragma unroll
        for (int g = 0; g < IC / M; ++g) {
            uint32_t in[M], out[M];
            bool k[M];
#pragma unroll
            for (int j = 0; j < M; ++j) in[j] = raw[g * M + j], k[j] = true;
            const uint64_t eg = e0 + (uint64_t)(g * M);
            if constexpr (RK != kDenseRanker) {
                prune_group<kF32, M, RK, NLE2>(in, p.n, hash_row(p.mix, (uint32_t)(eg >> 32)), (uint32_t)eg, k, out);
#pragma unroll
                for (int j = 0; j < M; ++j) in[j] = out[j];
            }
#pragma unroll
            for (int j = 0; j < M; ++j) raw[g * M + j] = in[j], keep |= (k[j] ? 1u : 0u) << (g * M + j), large = large || is_large(in[j]);
        }
        const size_t plane = (size_t)p.npix * 16;
        if constexpr (SPARSE) {
            uint32_t kept[8], meta = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool k[4] = {(keep >> (4 * q) & 1) != 0, (keep >> (4 * q + 1) & 1) != 0, (keep >> (4 * q + 2) & 1) != 0, (keep >> (4 * q + 3) & 1) != 0};
                const uint32_t o[4] = {raw[4 * q], raw[4 * q + 1], raw[4 * q + 2], raw[4 * q + 3]};
                uint32_t pos;
                compress_quad(k, o, kept[2 * q], kept[2 * q + 1], pos);
                meta |= pos << (4 * q);
            }
            u32x4_t out[3];
            split8(kept, out);
            const int chunk = ch >> 5, half = (ch >> 4) & 1;
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
                *reinterpret_cast<u32x4_t*>(p.planes + ((size_t)chunk * 6 + pl * 2 + half) * plane + (size_t)pix * 16) = out[pl];
            p.idx[((size_t)chunk * (size_t)p.npix + (size_t)pix) * 2 + half] = (uint16_t)meta;
        } else {
#pragma unroll
            for (int e = 0; e < IC / 8; ++e) {
                uint32_t x[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) x[j] = raw[8 * e + j];
                u32x4_t out[3];
                split8(x, out);
                const int chunk = (ch >> 4) + (e >> 1), half = e & 1;
                if (chunk < p.nchunks) {
#pragma unroll
                    for (int pl = 0; pl < 3; ++pl)
                        *reinterpret_cast<u32x4_t*>(p.planes + ((size_t)chunk * 6 + pl * 2 + half) * plane + (size_t)pix * 16) = out[pl];
                }
            }
        }
    }
    const int any = __syncthreads_or(large);
    if (threadIdx.x == 0) p.gnotes[wg] = any ? 1u : 0u;
}

// Result (input pixel `pix`, column `col`) as the definition has it, term by term, from the planes (whose sums are the
// pruned values) and W itself.
template <bool SPARSE>
__device__ __attribute__((noinline)) float split_sum_again(const SDGP_CONSTANT SplitParams* args, int pix, int col) {
    const SDGP_CONSTANT SplitParams& p = *args;
    const int h = pix / p.Wd % p.H, w = pix % p.Wd, b = pix / p.Wd / p.H;
    float sum = 0.0f;
    for (int r = 0; r < p.R; ++r)
        for (int s = 0; s < p.S; ++s) {
            const int y = h + p.pad - r, x = w + p.pad - s;
            if (y < 0 || x < 0 || y % p.stride != 0 || x % p.stride != 0 || y / p.stride >= p.P || x / p.stride >= p.Q) continue;
            const size_t g = ((size_t)b * p.P + y / p.stride) * p.Q + x / p.stride;
            for (int k = 0; k < p.C_out; ++k) {
                const int chunk = SPARSE ? k >> 5 : k >> 4, half = SPARSE ? (k >> 4) & 1 : (k >> 3) & 1;
                int e = k & 7;
                if constexpr (SPARSE) {
                    const uint32_t pos = (uint32_t)p.idx[((size_t)chunk * (size_t)p.npix + g) * 2 + half] >> (k & 12);
                    const uint32_t j = (uint32_t)k & 3u;
                    e = j == (pos & 3u) ? (k & 12) >> 1 : j == ((pos >> 2) & 3u) ? ((k & 12) >> 1) + 1 : -1;
                }
                float v = 0.0f;
                if (e >= 0) {
                    const uint16_t* const at = reinterpret_cast<const uint16_t*>(p.planes) + (((size_t)chunk * 6 + half) * (size_t)p.npix + g) * 8 + (size_t)e;
                    const size_t plane = (size_t)p.npix * 16;   // (two half chunks of eight)
                    v = split_join(at[0], at[plane], at[2 * plane]);
                }
                sum += v * p.W[((size_t)k * (p.R * p.S) + r * p.S + s) * p.C_in + col];
            }
            if (sum != sum) return sum;
        }
    return sum;
}

template <bool SPARSE, int ROWS, int NP>
__global__ void __launch_bounds__(ROWS * 4) f32_split(const SplitParams p) {
    using L = SplitLayout<SPARSE, ROWS, NP>;
    constexpr int THREADS = ROWS * 4, WAVES = THREADS / 64;
    constexpr int PARTS = L::kParts, GROUP = L::kGroup;
    extern __shared__ __align__(16) unsigned char smem_generic[];
    SDGP_LDS unsigned char* smem = (SDGP_LDS unsigned char*)smem_generic;
    const uint32_t smem_base = (uint32_t)(uintptr_t)smem;
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    // consecutive tiles on one XCD (workgroups are dealt round-robin over 8): its L2 then holds their rows and W
    int lid = blockIdx.x;
    {
        const int per = p.nblocks >> 3;
        if (lid < (per << 3)) lid = (lid & 7) * per + (lid >> 3);
    }
    const int ntile = lid % p.ntiles_n, mtile = lid / p.ntiles_n;
    const int ca = (int)blockIdx.z / p.stride, cb = (int)blockIdx.z % p.stride;
    const ParityAxis<int> ay = parity_axis<int>(p.H, p.R, p.stride, p.pad, ca), ax = parity_axis<int>(p.Wd, p.S, p.stride, p.pad, cb);
    const int b0 = mtile / (p.tiles_w * p.tiles_h) * p.TB, i0 = mtile / p.tiles_w % p.tiles_h * p.TH, j0 = mtile % p.tiles_w * p.TW;
    if (i0 >= ay.n || j0 >= ax.n) return;           // (the other classes have a row or column more; the whole workgroup leaves)
    const int ny = ay.count, nx = ax.count, ntaps = ny * nx;
    const int GH = grid_side(p.TH, ny), GW = grid_side(p.TW, nx), npad = p.TB * GH * GW;

    SDGP_LDS int* rowpix = (SDGP_LDS int*)smem;                          // input pixel of a tile row, -1: none
    SDGP_LDS uint32_t* notes = (SDGP_LDS uint32_t*)(smem + ROWS * 4);    // columns with a non-finite weight

    // the gradient pixel of the grid position this lane copies; positions outside the gradient copy zeros
    const unsigned char* src_plane = reinterpret_cast<const unsigned char*>(kF32Zeros);
    const unsigned char* src_idx = src_plane;
    uint64_t step_plane = 0, step_idx = 0;
    {
        const int pos = wave * 64 + lane;
        const int tb = pos / (GH * GW), rem = pos % (GH * GW);
        const int b = b0 + tb, pp = i0 + ay.shift - (ny - 1) + rem / GW, qq = j0 + ax.shift - (nx - 1) + rem % GW;
        if (pos < npad && b < p.B && pp >= 0 && pp < p.P && qq >= 0 && qq < p.Q) {
            const size_t pix = ((size_t)b * p.P + pp) * p.Q + qq;
            src_plane = p.planes + pix * 16, step_plane = (uint64_t)p.npix * 16;
            src_idx = reinterpret_cast<const unsigned char*>(p.idx) + pix * 4, step_idx = (uint64_t)p.npix * 4;
        }
    }
    // the next chunk's grid (chunks in order)
    auto copy_a = [&](uint32_t buf) {
        if (wave * 64 >= npad) return;
#pragma unroll
        for (int s = 0; s < 6; ++s) {
            lds_copy16(src_plane, smem_base + buf + (uint32_t)(s * L::kPlane) + (uint32_t)wave * 1024u);
            src_plane += step_plane;
        }
        if constexpr (SPARSE) {
            lds_copy4(src_idx, smem_base + buf + 6u * L::kPlane + (uint32_t)wave * 256u);
            src_idx += step_idx;
        }
    };
    const int taps = p.R * p.S;
    // W of the stage two ahead: up to GROUP taps of a chunk.  Copy unit i of a set is (part, tap, KB of the slab), this wavefront
    // takes units wave, wave + WAVES, ...
    constexpr int UNITS = PARTS * GROUP * 6, PER = (UNITS + WAVES - 1) / WAVES;
    const int chunks = ntaps > 0 ? p.nchunks : 0;
    int ahead_c = 0, ahead_tap = 0;
    uint32_t ahead = L::kOffW;
    const unsigned char* ahead_src = p.wimg + ((size_t)ntile * p.nc32 * 2 * taps + p.slot0[ay.r0 * p.stride + ax.r0]) * kSlab;
    uint32_t unit_src[PER];
    int unit_tap[PER];
#pragma unroll
    for (int x = 0; x < PER; ++x) {
        const int i = wave + x * WAVES, t = i / 6 % GROUP;
        unit_src[x] = (uint32_t)((i / (6 * GROUP) * taps + t) * kSlab + i % 6 * 1024);
        unit_tap[x] = i < UNITS ? t : GROUP;
    }
    auto copy_w = [&]() {
        if (ahead_c < chunks) {
            const int cnt = ntaps - ahead_tap;   // (of which the first GROUP)
#pragma unroll
            for (int x = 0; x < PER; ++x)
                if (unit_tap[x] < GROUP && unit_tap[x] < cnt)
                    lds_copy16(ahead_src + unit_src[x], (uint32_t)lane * 16u, smem_base + ahead + (uint32_t)((wave + x * WAVES) * 1024));
            ahead = ahead == L::kOffW + 2 * L::kWSet ? L::kOffW : ahead + L::kWSet;
            const bool wrap = cnt <= GROUP;      // the chunk's last taps
            ahead_src += wrap ? (PARTS * taps - ahead_tap) * kSlab : GROUP * kSlab;
            ahead_tap = wrap ? 0 : ahead_tap + GROUP;
            ahead_c += wrap ? 1 : 0;
        }
    };
    if (chunks > 0) copy_a(L::kOffA);
    copy_w();
    copy_w();
    if (tid < 2) notes[tid] = 0u;
    uint32_t lane_a, lane_i;   // this lane's row: grid position of the last tap of both axes
    {
        const int m = tid;
        if (m < ROWS) {
            int pix = -1;
            const int tb = m / (p.TH * p.TW), rem = m % (p.TH * p.TW), i = i0 + rem / p.TW, j = j0 + rem % p.TW;
            if (tb < p.TB && b0 + tb < p.B && i < ay.n && j < ax.n) pix = ((b0 + tb) * p.H + i * p.stride + ca) * p.Wd + j * p.stride + cb;
            rowpix[m] = pix;
        }
        {
            const int r = wm * 32 + (lane & 31);
            const int tb = r / (p.TH * p.TW), rem = r % (p.TH * p.TW);
            const int pos = tb < p.TB ? (tb * GH + rem / p.TW) * GW + rem % p.TW : 0;
            lane_a = (uint32_t)(half * L::kPlane) + (uint32_t)pos * 16u;
            lane_i = 6u * L::kPlane + (uint32_t)pos * 4u + (uint32_t)half * 2u;
        }
    }
    __syncthreads();
    {
        const int n = p.nc32 * 2 * taps * 2;
        for (int i = tid; i < n; i += THREADS) {
            const uint32_t cols = p.wnotes[2 * ((size_t)ntile * n + i)];
            if (cols) atomicOr((uint32_t*)(smem_generic + ROWS * 4 + 4 * (i & 1)), cols);
        }
    }

    f32x16_t acc, low;   // the products of the first parts, the five smaller ones
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = low[e] = 0.0f;

    struct Frags {
        u32x4_t a[3];
        int idx;
        u32x4_t b[3][PARTS];
    };
    const uint32_t b_lane = (uint32_t)(wn * 3 * 1024 + lane * 16);
    // tap t of a stage, `at` grid positions after a row's base
    auto load = [&](Frags& f, uint32_t abuf, uint32_t wbuf, int at, int t) {
        SDGP_LDS unsigned char* const a = smem + (abuf + lane_a + (uint32_t)at * 16u);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) f.a[pl] = *(SDGP_LDS u32x4_t*)(a + pl * 2 * L::kPlane);
        if constexpr (SPARSE) f.idx = *(SDGP_LDS uint16_t*)(smem + (abuf + lane_i + (uint32_t)at * 4u));
        SDGP_LDS unsigned char* const b = smem + (wbuf + b_lane);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl)
#pragma unroll
            for (int part = 0; part < PARTS; ++part) f.b[pl][part] = *(SDGP_LDS u32x4_t*)(b + (part * GROUP + t) * kSlab + pl * 1024);
    };
    auto multiply = [&](const Frags& f) {
        // the smallest products first
        constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const bf16x8_t a = __builtin_bit_cast(bf16x8_t, f.a[PA[q]]);
            f32x16_t& sum = q < 5 ? low : acc;
            if constexpr (SPARSE) {
                struct { u32x4_t lo, hi; } both = {f.b[PB[q]][0], f.b[PB[q]][PARTS - 1]};
                sum = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(a, __builtin_bit_cast(bf16x16_t, both), sum, f.idx, 0, 0);
            } else {
                sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(bf16x8_t, f.b[PB[q]][0]), sum, 0, 0, 0);
            }
        }
    };

    // Everything the next stage reads has landed a stage early, so its first fragments are requested before the barrier and a
    // wavefront's fragment reads run under matrix instructions, its own last ones and the other wavefronts'.  (Not the first of a
    // chunk of a single stage: that chunk's grid lands at the barrier.)
    const int first_at = (ny - 1) * GW + nx - 1;
    const bool early = ntaps > GROUP;
    uint32_t abuf = L::kOffA, wbuf = L::kOffW;
    Frags f;
    wait_lds_copies<0>();
    __syncthreads();
    if (chunks > 0) load(f, abuf, wbuf, first_at, 0);
    for (int c = 0; c < chunks; ++c) {
        const uint32_t aother = 2 * L::kOffA + L::kABytes - abuf;
        const bool more = c + 1 < chunks;
        // the walk over the taps, row by row: one grid position back per tap, GW - nx more at a row's end
        int at = first_at, v = 0;
        for (int tap0 = 0; tap0 < ntaps; tap0 += GROUP) {
            const uint32_t wnext = wbuf == L::kOffW + 2 * L::kWSet ? L::kOffW : wbuf + L::kWSet;
            if (tap0 == 0 && more) copy_a(aother);
            copy_w();
#pragma unroll
            for (int t = 0; t < GROUP; ++t) {
                if (tap0 + t < ntaps) {
                    multiply(f);
                    const bool end = ++v == nx;
                    at -= end ? GW - nx + 1 : 1;
                    v = end ? 0 : v;
                    if (tap0 + t + 1 < ntaps) load(f, abuf, t + 1 < GROUP ? wbuf : wnext, at, (t + 1) % GROUP);
                    else if (more && early) load(f, aother, wnext, first_at, 0);
                }
            }
            wait_lds_copies<0>();
            // a bare barrier: the fragments on their way are of sets that nobody overwrites before the next one
            asm volatile("s_barrier" ::: "memory");
            wbuf = wnext;
        }
        abuf = aother;
        if (more && !early) load(f, abuf, wbuf, first_at, 0);
    }

    float check = 0.0f;   // NaN: a result is not finite
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] += low[e], check = fmaf(acc[e], 0.0f, check);
    const bool unusual = check != check;
    bool large = false;   // what the first pass noted about the operands
    if (__builtin_expect(__any(unusual), 0)) {
        const int n = p.nc32 * 2 * taps * 2;
        for (int i = lane; i < p.gblocks; i += 64) large = large || p.gnotes[i] != 0;
        for (int i = lane; i < n; i += 64) large = large || p.wnotes[2 * ((size_t)ntile * n + i) + 1] != 0;
        large = __any(large);
    }
    const int col = ntile * 64 + wn * 32 + (lane & 31);
    const bool bad_col = ((notes[wn] >> (lane & 31)) & 1u) != 0;
    if (col >= p.C_in) return;
    typedef int i32x4_t __attribute__((ext_vector_type(4)));
    i32x4_t pixels[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) pixels[q] = *(SDGP_LDS i32x4_t*)(rowpix + wm * 32 + 8 * q + 4 * half);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const int pix = pixels[e >> 2][e & 3];
        if (pix >= 0) p.dD[(size_t)pix * p.C_in + col] = acc[e] * kSplitUnscale;
    }
    if (__builtin_expect((large && unusual) || bad_col, 0)) {
        for (int e = 0; e < 16; ++e) {
            const int pix = rowpix[wm * 32 + 8 * (e >> 2) + 4 * half + (e & 3)];
            if (pix < 0) continue;
            float* const at = p.dD + (size_t)pix * p.C_in + col;
            if (bad_col || (float_to_bits(*at) & 0x7F800000u) == 0x7F800000u)   // (with no large operand a NaN is the gradient's own)
                *at = split_sum_again<SPARSE>(reinterpret_cast<const SDGP_CONSTANT SplitParams*>((uint64_t)__builtin_amdgcn_kernarg_segment_ptr()), pix, col);
        }
    }
}

}  // namespace sdgp

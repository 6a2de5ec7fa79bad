// Backward-data kernel for 3x3 layers of stride 2 with one pixel of padding, fused with pruning (n <= 2 of m in {4, 8, 16}):
// dL/dD = prune(dL/dO) (*) W (Fig. 3 left; Sec. II-A).
//
// Input pixel (2i + a, 2j + b) sums the taps r of its parity -- r = 1 of gradient line i for a = 0, r = 2 of line i and r = 0 of line
// i + 1 for a = 1, the same across -- so the four parity classes are products over 1, 2, 2 and 4 taps whose gradient pixels are
// (i, j), (i, j + 1), (i + 1, j) and (i + 1, j + 1).  One workgroup computes all four classes of its grid positions:
//   * It takes BM consecutive positions (i, j) of all images.  The gradient pixels they need are a run of BM + width + 1 pixels,
//     ranked and compressed once, with all their channels, into LDS: a line of the padded gradient in which a tap is a constant
//     distance (as in bwd_line.h).
//   * Then class by class, tap by tap, 32 channels a stage: W's slab of (tap, 32 channels) streams through a ring of four slots of
//     direct-to-LDS copies, three stages ahead; every slab is read once per workgroup, whatever class it serves.  Fragments are read
//     a stage ahead, between the matrix instructions: two wavefronts on a SIMD hide no LDS latency of their own.
//   * A class leaves as soon as its taps are done, straight from the registers (store_class), while the next class's slabs arrive.
// The parity-class kernel (bwd_pw.h) needs a pass that ranks ahead, or ranks an element once per tap, and its workgroups are too short
// to hide their first loads and their stores: four and a half steps each.  128 <- 128 channels at 56x56, batch 256, 2:4 random
// 97.2 -> 76 to 79 us (94.8 -> 72.1 on another card; 16 of the old time the pass), Magnitude 101 -> 75; 192 <- 96 at 51x51, batch 60, 39 -> 21; 150 layers that kernel took
// before 0.78 of the time.  Per workgroup of 256 x 128, in cycles: 36 stages of 800 (256 of them matrix instructions, two wavefronts a
// SIMD), ranking 10 000, four stores of a class; 128 KB a workgroup go to memory.  Tried: eight wavefronts of 32 x 64 results, half
// the instructions each, and 64 channels a stage: 83 us, bound by the fragments' LDS reads.
#pragma once

#include "fastdiv.h"
#include "lds_copy.h"
#include "quad_rows.h"

namespace sdgp {

struct Stride2Params {
    const uint16_t* dO;
    const uint16_t* W;
    uint16_t* dD;
    int pixels;                  // B * P * Q gradient pixels
    int P, Q, H, Wd, C_out, C_in;
    FastDiv by_line, by_image, by_parts;
    int parts;                   // items of sixteen channels per pixel, the missing ones of a short last chunk included
    int w_row;                   // elements per W row: 9 * C_in
    int n;
    uint32_t mix;
    int npos;                    // positions of the line that a tile's taps reach, at most
    int ntiles_n, nblocks;
};

__device__ __align__(16) const uint32_t kStride2Zeros[4] = {0, 0, 0, 0};   // rows of W past the last channel

constexpr int kStride2Threads = 256;
constexpr int kStride2KC = 32;     // reduction channels per stage
constexpr int kStride2Slots = 4;   // slabs of W in the ring

// The nine taps by class -- (1, 1), (1, 0), (0, 1), (0, 0) -- a nibble each: the filter tap 3 r + s, and the gradient pixel it
// reads, one line down (bit 1) and one pixel on (bit 0).
constexpr uint64_t kStride2Tap = 0x435170268ull;
constexpr uint64_t kStride2Shift = 0x010203210ull;

template <int BN, int TM>
struct Stride2Layout {
    static constexpr int kRows = 4 * 32 * TM * 64 / BN;    // four wavefronts of (32 TM) x 64 results
    static constexpr int kWRow = BN * 2;
    static constexpr int kWSlab = kStride2KC * kWRow;
    __host__ __device__ static int plane_a(int npos) { return ((npos * 16 + 127) & ~255) + 128; }
    __host__ __device__ static int plane_m(int npos) { return (npos * 2 + 63) & ~63; }
    __host__ __device__ static int off_rows() { return kStride2Slots * kWSlab; }
    __host__ __device__ static int off_a() { return off_rows() + kRows * 4; }
    __host__ __device__ static int off_m(int npos, int parts) { return off_a() + parts * plane_a(npos); }
    __host__ __device__ static int total(int npos, int parts) { return off_m(npos, parts) + parts * plane_m(npos); }
    // the longest run of the padded line from a tile's first position to the last one its taps read
    static int positions(int P, int Q) {
        const int between = kRows - 1;
        return between + (Q - 1 + between) / Q + (int)(((int64_t)P * Q - 1 + between) / ((int64_t)P * Q)) * (Q + 1) + Q + 1 + 2;
    }
};

// TAIL: C_out is no multiple of a stage's channels
template <int BN, int TM, int M, int RK, bool TAIL>
__global__ void __launch_bounds__(kStride2Threads, 2) bwd_stride2(const Stride2Params p) {
    using L = Stride2Layout<BN, TM>;
    constexpr int BM = L::kRows;
    constexpr int WAVES_N = BN / 64;
    constexpr int TN = 2;
    constexpr int CPR = BN / 8;                 // 16-byte columns per W row
    constexpr int RPU = 1024 / L::kWRow;        // W rows per copy unit of 1 KB
    constexpr int COPIES = L::kWSlab / 4096;    // units per wavefront and stage
    constexpr int WSW = BN >= 128 ? 4 : 2;      // swizzle of the W slab, as in bwd_row.h
    extern __shared__ __align__(16) unsigned char smem_generic[];
    SDGP_LDS unsigned char* smem = (SDGP_LDS unsigned char*)smem_generic;
    const uint32_t smem_base = (uint32_t)(uintptr_t)smem;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;

    // consecutive logical ids stay on one XCD (workgroups are dealt round-robin over 8 XCDs)
    int lid = blockIdx.x;
    {
        const int per = p.nblocks >> 3;
        if (lid < (per << 3)) lid = (lid & 7) * per + (lid >> 3);
    }
    const int ntile = lid % p.ntiles_n;
    const int n0 = ntile * BN;
    const int t0 = lid / p.ntiles_n * BM;
    const int GW = p.Q + 1;                     // a line of the padded gradient: one zero behind
    auto line_pos = [&](int px) {
        const uint32_t row = divide((uint32_t)px, p.by_line);
        return px + (int)row + (int)divide(row, p.by_image) * GW;
    };
    const int base = line_pos(t0);
    const uint32_t plane_a = (uint32_t)L::plane_a(p.npos), plane_m = (uint32_t)L::plane_m(p.npos);
    const uint32_t off_m = (uint32_t)L::off_m(p.npos, p.parts);

    // ---- copies of W
    const int w_lrow = wave * RPU + lane / CPR;      // of a slab's rows, and 4 RPU further with every copy
    uint32_t w_voff;
    {
        int col = n0 + (((lane % CPR) ^ (WSW * (w_lrow & 3))) * 8);
        if (col > p.C_in - 8) col = p.C_in - 8;  // columns past C_in feed accumulators that are never stored
        w_voff = (uint32_t)(w_lrow * p.w_row + col) * 2u;
    }
    uint32_t w_unit[COPIES];                     // this lane's byte of each of its wavefront's copies, from the slab's first row
#pragma unroll
    for (int i = 0; i < COPIES; ++i) w_unit[i] = w_voff + (uint32_t)(4 * i * RPU) * (uint32_t)p.w_row * 2u;
    const unsigned char* const gWb = reinterpret_cast<const unsigned char*>(p.W);
    const int nk = (p.C_out + kStride2KC - 1) / kStride2KC;
    const int total = 9 * nk;
    const size_t chunkB = (size_t)kStride2KC * p.w_row * 2;
    uint64_t c_taps = kStride2Tap;               // the slab to be asked for next: its tap is the lowest nibble
    int c_left = p.C_out;                        // ... and the channels from it on
    const unsigned char* c_slab = gWb + (size_t)(kStride2Tap & 15) * p.C_in * 2;
    uint32_t c_dst = smem_base + (uint32_t)wave * 1024u;
    const uint32_t c_end = c_dst + (uint32_t)(kStride2Slots * L::kWSlab);
    auto copy_unit = [&](int i) {
        if (!TAIL || c_left >= kStride2KC) lds_copy16(c_slab, w_unit[i], c_dst + 4096u * i);
        else lds_copy16(w_lrow + 4 * i * RPU < c_left ? c_slab + w_unit[i] : reinterpret_cast<const unsigned char*>(kStride2Zeros), c_dst + 4096u * i);
    };
    auto copied = [&]() {                        // on to the next slab
        c_dst += L::kWSlab;
        if (c_dst == c_end) c_dst -= (uint32_t)(kStride2Slots * L::kWSlab);
        c_left -= kStride2KC;
        c_slab += chunkB;
        if (c_left <= 0) {
            c_taps >>= 4;
            c_left = p.C_out;
            c_slab = gWb + (size_t)(uint32_t)((int)(c_taps & 15) * p.C_in * 2);
        }
    };
#pragma unroll
    for (int j = 0; j < kStride2Slots - 1; ++j) {   // (nine stages or more)
#pragma unroll
        for (int i = 0; i < COPIES; ++i) copy_unit(i);
        copied();
    }

    // ---- zeros, and the table of the tile's rows: pixel (2i, 2j) of position (i, j), and what of its block lies in the image
    SDGP_LDS uint32_t* const rows = (SDGP_LDS uint32_t*)(smem + L::off_rows());
    {
        const u32x4_t z = {0u, 0u, 0u, 0u};
        const uint32_t end = (uint32_t)L::total(p.npos, p.parts);
        for (uint32_t o = (uint32_t)L::off_a() + (uint32_t)tid * 16u; o < end; o += kStride2Threads * 16u) *(SDGP_LDS u32x4_t*)(smem + o) = z;
        if (tid < BM) {
            const int px = t0 + tid;
            uint32_t e = 3u << 30;               // no such position
            if (px < p.pixels) {
                const int row = (int)divide((uint32_t)px, p.by_line), img = (int)divide((uint32_t)row, p.by_image);
                const int i = row - img * p.P, j = px - row * p.Q;
                e = (uint32_t)((img * p.H + 2 * i) * p.Wd + 2 * j) | (2 * i + 1 < p.H ? 0u : 1u << 31) | (2 * j + 1 < p.Wd ? 0u : 1u << 30);
                if (e >= 3u << 30) e = (e & 0x1FFFFFFFu) | 1u << 29 | 3u << 30;   // the last pixel of an odd image: class (0, 0) only
            }
            rows[tid] = e;
        }
    }
    __syncthreads();

    // ---- rank and compress the window, all channels
    {
        const int last = min(BM + GW, p.pixels - t0);
        const int items = last * p.parts;
        const unsigned char* const first = reinterpret_cast<const unsigned char*>(p.dO) + (size_t)t0 * p.C_out * 2;
        constexpr int U = 5;                     // a tile of 256 positions at 28 pixels a line and 128 channels in two rounds
        for (int it = tid; it < items; it += U * kStride2Threads) {
            u32x4_t v[U][2];
            int px[U], part[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int item = min(it + u * kStride2Threads, items - 1);
                px[u] = (int)divide((uint32_t)item, p.by_parts);
                part[u] = item - px[u] * p.parts;
                const int c = part[u] * 16;
                const unsigned char* const src = first + ((uint32_t)px[u] * (uint32_t)p.C_out + (uint32_t)c) * 2u;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const bool in = c + 8 * h < p.C_out;
                    v[u][h] = *reinterpret_cast<const u32x4_t*>(in ? src + 16 * h : first);
                    if (!in) v[u][h] = u32x4_t{0u, 0u, 0u, 0u};
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (it + u * kStride2Threads < items) {
                    const uint64_t e0 = (uint64_t)(t0 + px[u]) * (uint64_t)p.C_out + (uint64_t)(part[u] * 16);
                    uint32_t packed[4], meta;
                    prune16_compressed<M, RK>(v[u], p.n, p.mix, e0, packed, meta);
                    const uint32_t pos = (uint32_t)(line_pos(t0 + px[u]) - base);
                    if (pos < (uint32_t)p.npos) {
                        *(SDGP_LDS u32x4_t*)(smem + L::off_a() + (uint32_t)part[u] * plane_a + pos * 16u) = u32x4_t{packed[0], packed[1], packed[2], packed[3]};
                        *(SDGP_LDS uint16_t*)(smem + off_m + (uint32_t)part[u] * plane_m + pos * 2u) = (uint16_t)meta;
                    }
                }
            }
        }
    }

    // ---- fragments
    // Column n of tile u is 8 (n / 4) + 4 (u ^ (n / 16)) + n % 4 of the wavefront's 64: the lanes of a quad then hold eight consecutive
    // columns in their two tiles, sixteen bytes of a row.  (The halves of a transposing read's lanes take different halves of the
    // sixteen bytes, or they would meet in the same banks.)
    uint32_t b_lane[TN];
#pragma unroll
    for (int u = 0; u < TN; ++u) {
        const int L16 = lane & 15, upper = (lane >> 4) & 1;
        const int chunk = 8 * wn + 4 * upper + (L16 & 3);
        b_lane[u] = (uint32_t)((8 * (lane >> 5) + (L16 >> 2)) * L::kWRow + ((chunk ^ (WSW * (L16 >> 2))) * 16) + (u ^ upper) * 8);
    }
    const uint32_t half = (uint32_t)(lane >> 5);
    uint32_t lane_a[TM], lane_m[TM];
#pragma unroll
    for (int t = 0; t < TM; ++t) {
        const int px = t0 + (wm * TM + t) * 32 + (lane & 31);
        const uint32_t pos = px < p.pixels ? (uint32_t)(line_pos(px) - base) : 0u;
        lane_a[t] = (uint32_t)L::off_a() + half * plane_a + pos * 16u;
        lane_m[t] = off_m + half * plane_m + pos * 2u;
    }
    struct Frags {
        u32x4_t a[TM];
        int meta[TM];
        bf16x16_t b[TN];
    };
    auto load_a = [&](Frags& f, int t, uint32_t at, uint32_t at_m) {
        f.a[t] = *(SDGP_LDS u32x4_t*)(smem + lane_a[t] + at);
        f.meta[t] = *(SDGP_LDS uint16_t*)(smem + lane_m[t] + at_m);
    };
    auto load_b = [&](Frags& f, int u, uint32_t slab_off) {
        SDGP_LDS unsigned char* wb = smem + b_lane[u] + slab_off;
        s16x4_t q[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            q[i] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((SDGP_LDS s16x4_t*)(wb + ((i >> 1) * 16 + (i & 1) * 4) * L::kWRow));
        typedef short s16x16_t __attribute__((ext_vector_type(16)));
        const s16x16_t all = {q[0][0], q[0][1], q[0][2], q[0][3], q[1][0], q[1][1], q[1][2], q[1][3],
                              q[2][0], q[2][1], q[2][2], q[2][3], q[3][0], q[3][1], q[3][2], q[3][3]};
        f.b[u] = __builtin_bit_cast(bf16x16_t, all);
    };
    f32x16_t acc[TM][TN];
    auto clear = [&]() {
#pragma unroll
        for (int t = 0; t < TM; ++t)
#pragma unroll
            for (int u = 0; u < TN; ++u)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[t][u][r] = 0.0f;
    };
    clear();

    // ---- a finished class: out of the registers, a store is eight whole 128-byte rows.  (Through LDS, sixteen rows of a wavefront at a
    // time, a class took 8000 cycles of waiting for its own reads and writes; stores of half a line each cost the memory a quarter of
    // the whole call's time.)
    auto store_class = [&](int a, int b) __attribute__((always_inline)) {
        const uint32_t outside = (a ? 1u << 31 : 0u) | (b ? 1u << 30 : 0u);
        const int col = n0 + wn * 64 + 2 * (lane & 28);
        const bool in = col < p.C_in;
        uint32_t place[TM][4];
#pragma unroll
        for (int t = 0; t < TM; ++t)
#pragma unroll
            for (int g = 0; g < 4; ++g) place[t][g] = rows[(wm * TM + t) * 32 + 8 * g + 4 * (lane >> 5) + (lane & 3)];
#pragma unroll
        for (int t = 0; t < TM; ++t)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const u32x4_t out = quad_rows(acc[t][0], acc[t][1], g, lane);
                const uint32_t e = place[t][g];
                if (in && e != 3u << 30 && (e & outside) == 0u) {
                    const size_t pix = (size_t)((e & 0x1FFFFFFFu) + (uint32_t)(a * p.Wd + b));
                    __builtin_nontemporal_store(out, reinterpret_cast<u32x4_t*>(p.dD + pix * p.C_in + col));
                }
            }
    };

    wait_lds_copies<COPIES>();                   // two slabs have landed (and the compressed gradient lies where it belongs)
    __syncthreads();

    // A stage reads the next one's fragments between its matrix instructions: the next slab landed a barrier ago, the compressed
    // gradient stays where it is.
    Frags f0, f1;
    auto stage = [&](const Frags& cur, Frags& nxt, int tap, int k, int x) __attribute__((always_inline)) {
        const bool more = x + kStride2Slots - 1 < total, tap_done = k + 1 == nk;
        const int next_tap = tap_done ? tap + 1 : tap, next_k = tap_done ? 0 : k + 1;
        const uint32_t sh = (uint32_t)(kStride2Shift >> (4 * next_tap)) & 3u, place = (sh >> 1) * (uint32_t)GW + (sh & 1u);
        const uint32_t at = place * 16u + (uint32_t)(2 * next_k) * plane_a, at_m = place * 2u + (uint32_t)(2 * next_k) * plane_m;
        const uint32_t slot = (uint32_t)((x + 1) % kStride2Slots) * L::kWSlab;
        // (behind the last stage the reads stay inside the LDS, and nobody uses what they bring)
#pragma unroll
        for (int g = 0; g < TM * TN; ++g) {
            const int t = g / TN, u = g % TN;
            __builtin_amdgcn_sched_barrier(0);
            acc[t][u] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(__builtin_bit_cast(bf16x8_t, cur.a[t]), cur.b[u], acc[t][u], cur.meta[t], 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (g < TN) load_b(nxt, g, slot);
            else if (g - TN < TM) load_a(nxt, g - TN, at, at_m);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (more) {
#pragma unroll
            for (int i = 0; i < COPIES; ++i) copy_unit(i);
            copied();
            wait_lds_copies<COPIES>();
        } else {
            wait_lds_copies<0>();
        }
        __syncthreads();                         // the slab after the next has landed, and everybody is done with this one
        if (tap_done && (tap == 3 || tap == 5 || tap >= 7)) {
            store_class(tap == 3 || tap == 5, tap == 3 || tap == 7);
            clear();
        }
    };
#pragma unroll
    for (int t = 0; t < TM; ++t) load_a(f0, t, 0u, 0u);
#pragma unroll
    for (int u = 0; u < TN; ++u) load_b(f0, u, 0u);
    int tap = 0, k = 0;
    for (int x = 0; x < total; x += 2) {
        stage(f0, f1, tap, k, x);
        if (++k == nk) k = 0, ++tap;
        if (x + 1 == total) break;
        stage(f1, f0, tap, k, x + 1);
        if (++k == nk) k = 0, ++tap;
    }
}

}  // namespace sdgp

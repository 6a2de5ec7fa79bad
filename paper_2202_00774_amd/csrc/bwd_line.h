// Backward-data kernel for 3x3 stride-1 layers with one pixel of padding, fused with pruning or unpruned (then also the forward pass):
// dL/dD = prune(dL/dO) (*) W as an implicit GEMM (Fig. 3 left; Sec. II-A), rows = input pixels, columns = input channels.
//
// The pixels of all images lie behind each other in one line, and a workgroup takes 256 consecutive ones wherever lines and images
// begin: no tile is chosen for the image's shape and none is cut by its border.  The gradient pixels that their nine taps reach are
// a run of 256 + 2 (width + 1) consecutive pixels.  In LDS they lie in a line of the padded image -- a zero in front of every image
// line, a line of zeros between images -- where a tap is a constant distance: no tables, no tests in the loop.
//   * The reduction runs in chunks of 32 channels; a stage = (chunk, filter row) = three taps between two barriers, as in bwd_row.h.
//   * A lane ranks the same three pixels' halves (items of sixteen channels) in every chunk, one per stage, for the chunk after the
//     current one; it asks for an item's 32 bytes one stage ahead, straight into registers.  Output: the operand of
//     v_smfmac_f32_32x32x32_bf16, two values + two 2-bit positions per quad.
//   * The ranker runs between the stage's matrix instructions, five or six of its instructions after each (NoGap in ranker.h), and
//     so do the requests for the next fragments and the copies of W's next slabs.
//   * Four wavefronts of 128 x 64 (128 columns) or 64 x 64 results (64 columns).  More than one workgroup on a CU lets one's first loads,
//     ranking and stores run beside the other's matrix instructions; bwd_row has one workgroup of 512 pixels there, whose prologue and
//     epilogue (7 us a round) nothing hides.  The LDS leaves two of 128 columns on images 4 to 60 pixels wide, three of 64 on 5 to 46 and two
//     to 63, of the whole gradient two on 4 to 57; a single one beyond that and on images of few lines (bwd_line_choice.h).
//   * W through a two-set ring of direct-to-LDS copies, fragments by transposing reads, as in bwd_row.h.
//   * Patterns with more than two of a quad, groups of 32 and the unpruned gradient lie in LDS whole, eight channels a plane, and use
//     the dense instruction; their rankers (none, or a sorting network) run in front of the stage's matrix instructions.
// What bounds it: the matrix and vector instructions share a SIMD's issue (a structured-sparse instruction takes 13 cycles of it and
// 32 of the matrix pipe) and the clock, which falls from 2.4 to 1.6 - 1.9 GHz under them.  Measured against bwd_row, whole calls: 128 <- 256
// channels at 16x16, batch 512, 2:4 Magnitude 51.9 -> 46.5 to 48.3 us, 64 <- 128 at 32x32 80.8 -> 64.5, 128 <- 128 at 28x28, batch 128,
// 31 -> 24.8; 400 drawn layers 0.70 of the time, a hundred of one of m 0.76;
// of general n:m 0.76 (80 layers), unpruned 0.79 (70; 128 <- 320 at 28x28, batch 112, 88.7 -> 60.5 us; the slowest
// of 700 more 1.04: 128 <- 384 at 14x14, batch 567, one round of bwd_row).
#pragma once

#include <type_traits>

#include "fastdiv.h"
#include "lds_copy.h"
#include "quad_rows.h"

namespace sdgp {

struct LineParams {
    const uint16_t* dO;
    const uint16_t* W;
    uint16_t* dD;
    int pixels;                  // B * H * Wd: as many gradient pixels as input pixels
    int H, Wd, C_out, C_in;
    FastDiv by_line, by_image;   // a pixel's line, a line's image
    int w_row;                   // elements per W row: 9 * C_in
    int n;
    uint32_t mix;
    int npos;                    // positions of the line that a tile's taps reach, at most
    int ntiles_n, nblocks;
};

__device__ __align__(16) const uint32_t kLineZeros[4] = {0, 0, 0, 0};   // what a short last chunk lacks

constexpr int kLineKC = 32;         // reduction channels per chunk
constexpr int kLineThreads = 256;

constexpr int kLineRows = 256;      // pixels of a workgroup tile
// a lane ranks one item (sixteen channels of a gradient pixel) per stage; the three stages of a chunk cover the window
constexpr int kLineMaxWindow = 3 * kLineThreads / 2;
constexpr int kLineMaxWidth = (kLineMaxWindow - kLineRows) / 2 - 1;

__host__ __device__ inline int line_window(int Wd) { return kLineRows + 2 * (Wd + 1); }

// Whether bwd_line is built with 128 columns for n <= 2 (one: one of m; cut: the last chunk is short; one of m is built for all channel
// counts).  The magnitude rankers that sort keys leave no registers for them where the last chunk is cut.
constexpr bool line_has_128(int m, int rk, bool one, bool cut) {
    return !((one || cut) && rk != kRandom && (m > 4 || (one && rk == kGreedy)));
}

// The longest run of the padded line, from the first to the last position that some tile's taps read.
inline int line_positions(int H, int Wd) {
    const int between = kLineRows - 1;
    const int lines = (Wd - 1 + between) / Wd;                                                // line ends between a tile's first and last pixel
    const int images = (int)(((int64_t)H * Wd - 1 + between) / ((int64_t)H * Wd));            // image ends
    return between + lines + images * (Wd + 1) + 2 * (Wd + 2) + 1;
}

template <int BN, int MODE>
struct LineLayout {
    static constexpr int kWRow = BN * 2;
    static constexpr int kWSlab = kLineKC * kWRow;
    static constexpr int kWSet = 3 * kWSlab;               // the slabs of one filter row
    // value planes (16 bytes per position and half chunk) and planes of their 2-bit positions (2 bytes), with one position more, which
    // takes what no tap reads; sizes are 128 modulo 256 bytes, so that the two halves of a wavefront read different halves of the banks
    __host__ __device__ static int plane_a(int npos) { return (((npos + 1) * 16 + 127) & ~255) + 128; }
    __host__ __device__ static int plane_m(int npos) { return (((npos + 1) * 2 + 127) & ~255) + 128; }
    __host__ __device__ static int off_a() { return 2 * kWSet; }
    // (the whole gradient, MODE 0 and 1: four planes, eight channels each)
    __host__ __device__ static int buf_bytes(int npos) { return MODE == 2 ? 2 * plane_a(npos) + 2 * plane_m(npos) : 4 * plane_a(npos); }
    __host__ __device__ static int total(int npos) { return off_a() + 2 * buf_bytes(npos); }
};

// keeps the computation of a value in front of what follows in the program
template <class T>
__device__ __forceinline__ void pin_value(T& x) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(x));
#endif
}

// MODE 2: at most two of a quad stay (TWO: two of m, else one), the structured-sparse instruction; 1: any n of m up to 32, stored with
// zeros, the dense one; 0: unpruned.
template <int BN, int MODE, int M, int RK, bool TAIL, bool TWO>
__global__ void __launch_bounds__(kLineThreads, MODE == 2 && BN == 64 ? 3 : 2) bwd_line(const LineParams p) {
    using L = LineLayout<BN, MODE>;
    constexpr bool SPARSE = MODE == 2;
    constexpr int KSTEPS = SPARSE ? 3 : 6;      // of a stage
    constexpr bool WHOLE = MODE == 1 && M == 32;   // an item is a pixel's 32 channels, and two of them cover the window
    constexpr int ITEMS = WHOLE ? 2 : 3;
    constexpr int KC = kLineKC;
    constexpr int BM = kLineRows;
    constexpr int WAVES_N = BN / 64;
    constexpr int WAVES_M = 4 / WAVES_N;
    constexpr int WM = BM / WAVES_M;
    constexpr int TM = WM / 32;
    constexpr int TN = 2;
    constexpr int CPR = BN / 8;                 // 16-byte columns per W row
    constexpr int RPU = 1024 / L::kWRow;        // W rows per copy unit of 1 KB
    constexpr int UPS = L::kWSlab / 1024;       // units per slab
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
    const int mtile = lid / p.ntiles_n;
    const int n0 = ntile * BN;
    const int t0 = mtile * BM;
    const int nchunks = TAIL ? (p.C_out + KC - 1) / KC : p.C_out / KC;
    const int tail = p.C_out - (nchunks - 1) * KC;      // channels of the last chunk
    // every workgroup walks the chunks in its own rotation: the sum does not care, and the workgroups of an XCD then ask its L2 for
    // different W slabs at a given moment
    const int c_rot = mtile % nchunks;

    const int GW = p.Wd + 1;   // a line of the padded image: one zero in front
    auto line_pos = [&](int px) {
        const uint32_t row = divide((uint32_t)px, p.by_line);
        return px + (int)row + ((int)divide(row, p.by_image) + 1) * GW + 1;
    };
    const int base = line_pos(t0) - GW - 1;    // line position of LDS position 0
    const uint32_t plane_a = (uint32_t)L::plane_a(p.npos), plane_m = (uint32_t)L::plane_m(p.npos);
    const uint32_t buf_bytes = (uint32_t)L::buf_bytes(p.npos);
    const unsigned char* const gWb = reinterpret_cast<const unsigned char*>(p.W);

    // ---- copies of W
    const int w_lrow = (wave % UPS) * RPU + lane / CPR;
    uint32_t w_voff;
    {
        int col = n0 + (((lane % CPR) ^ (WSW * (w_lrow & 3))) * 8);
        if (col > p.C_in - 8) col = p.C_in - 8;  // columns past C_in feed accumulators that are never stored
        w_voff = (uint32_t)(w_lrow * p.w_row + col) * 2u;
    }
    const uint32_t tapB = (uint32_t)p.C_in * 2u;
    const uint32_t chunkB = (uint32_t)KC * (uint32_t)p.w_row * 2u;
    const uint32_t unitB = (uint32_t)(4 * RPU) * (uint32_t)p.w_row * 2u;   // four units further down the slab
    constexpr int WCOPIES = 3 * UPS / 4;        // copies of this wavefront per stage
    auto copy_w = [&](int pc, int pr, uint32_t set_off, int i) {
        const int j = i / (UPS / 4), k = i % (UPS / 4);
        const unsigned char* const src = gWb + ((size_t)pc * chunkB + (size_t)(pr * 3 + j) * tapB + (size_t)k * unitB);
        const uint32_t dst = smem_base + set_off + (uint32_t)j * L::kWSlab + (uint32_t)(wave + 4 * k) * 1024u;
        if (TAIL && pc == nchunks - 1)
            lds_copy16(w_lrow + 4 * RPU * k < tail ? src + w_voff : reinterpret_cast<const unsigned char*>(kLineZeros), dst);
        else
            lds_copy16(src, w_voff, dst);
    };

    // ---- this lane's items: the same pixels in every chunk
    const int64_t g0 = (int64_t)t0 - GW;                       // first pixel of the window
    const int half_i = WHOLE ? 0 : tid & 1;
    uint32_t it_voff[ITEMS];                                  // byte offset from the window's first pixel
    uint32_t it_pos[ITEMS];                                   // LDS position; npos, which no tap reads: no pixel, or one that no tap reaches
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int w = WHOLE ? k * kLineThreads + tid : (k * kLineThreads + tid) >> 1;
        const int64_t px = g0 + w;
        uint32_t pos = (uint32_t)p.npos, at = (uint32_t)GW;
        if (w < line_window(p.Wd) && px >= 0 && px < p.pixels) {
            const uint32_t q = (uint32_t)(line_pos((int)px) - base);
            at = (uint32_t)w;
            if (q < (uint32_t)p.npos) pos = q;
        }
        it_pos[k] = pos;
        it_voff[k] = at * (uint32_t)p.C_out * 2u + (uint32_t)half_i * 32u;
    }
    const unsigned char* const window = reinterpret_cast<const unsigned char*>(p.dO) + g0 * p.C_out * 2;
    struct Raw {
        u32x4_t v[WHOLE ? 4 : 2];
    };
    auto load_item = [&](int k, int pc) {
        Raw r;
        const unsigned char* const src = window + (size_t)pc * (KC * 2);
        if (TAIL && pc == nchunks - 1) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const bool in = half_i * 16 + i * 8 < tail;
                r.v[i] = *reinterpret_cast<const u32x4_t*>((in ? src : window) + it_voff[k] + (in ? i * 16 : -half_i * 32));
                if (!in) r.v[i] = u32x4_t{0u, 0u, 0u, 0u};
            }
        } else {
#pragma unroll
            for (int i = 0; i < (WHOLE ? 4 : 2); ++i) r.v[i] = *reinterpret_cast<const u32x4_t*>(src + it_voff[k] + 16 * i);
        }
        return r;
    };
    const uint64_t e_first = (uint64_t)(g0 * p.C_out);
    auto rank_item = [&](const Raw& r, int k, int pc, uint32_t abuf, auto&& gap) __attribute__((always_inline)) {
        const uint64_t e0 = e_first + (uint64_t)(it_voff[k] >> 1) + (uint64_t)(pc * KC);
        if constexpr (SPARSE) {
            uint32_t packed[4], meta;
            prune16_compressed<M, RK>(r.v, TWO ? 2 : 1, p.mix, e0, packed, meta, gap);
            *(SDGP_LDS u32x4_t*)(smem + abuf + (uint32_t)half_i * plane_a + it_pos[k] * 16u) = u32x4_t{packed[0], packed[1], packed[2], packed[3]};
            *(SDGP_LDS uint16_t*)(smem + abuf + 2u * plane_a + (uint32_t)half_i * plane_m + it_pos[k] * 2u) = (uint16_t)meta;
        } else {
            Raw o = r;
            if constexpr (WHOLE) prune32_dense<RK, false>(o.v, p.n, p.mix, e0);
            else if constexpr (MODE == 1) prune16_dense<M, RK, false>(o.v, p.n, p.mix, e0);
#pragma unroll
            for (int i = 0; i < (WHOLE ? 4 : 2); ++i)
                *(SDGP_LDS u32x4_t*)(smem + abuf + (uint32_t)(2 * half_i + i) * plane_a + it_pos[k] * 16u) = o.v[i];
        }
    };

    // ---- prologue
    int pc = c_rot;
    int pc1 = pc + 1 == nchunks ? 0 : pc + 1;
#pragma unroll
    for (int i = 0; i < WCOPIES; ++i) copy_w(pc, 0, 0u, i);
    Raw raw;
    {
        Raw first[ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) first[k] = load_item(k, pc);
        const u32x4_t z = {0u, 0u, 0u, 0u};
        for (uint32_t o = (uint32_t)tid * 16u; o < 2u * buf_bytes; o += kLineThreads * 16u) *(SDGP_LDS u32x4_t*)(smem + L::off_a() + o) = z;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) rank_item(first[k], k, pc, (uint32_t)L::off_a(), NoGap{});
        if (nchunks > 1) raw = load_item(0, pc1);
    }

    f32x16_t acc[TM][TN];
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int u = 0; u < TN; ++u)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][u][r] = 0.0f;

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
    // where this lane's rows lie in the buffer and at the filter row of the current stage; tap s is 2 - s positions further
    uint32_t a_stage[TM], m_stage[TM];
#pragma unroll
    for (int t = 0; t < TM; ++t) {
        const int px = t0 + wm * WM + t * 32 + (lane & 31);
        const uint32_t pos = (uint32_t)((px < p.pixels ? line_pos(px) - base - GW - 1 : 0) + 2 * GW);
        a_stage[t] = (uint32_t)L::off_a() + half * plane_a + pos * 16u;
        m_stage[t] = (uint32_t)L::off_a() + 2u * plane_a + half * plane_m + pos * 2u;
    }
    struct Frags {
        u32x4_t a[TM];
        int meta[TM];
        typename std::conditional<SPARSE, bf16x16_t, bf16x8_t>::type b[TN];
    };
    // of k-step q: tap q, or tap q / 2 and its sixteen channels q % 2
    auto load_a = [&](Frags& f, int t, int q) {
        if constexpr (SPARSE) {
            f.a[t] = *(SDGP_LDS u32x4_t*)(smem + a_stage[t] + (2 - q) * 16);
            f.meta[t] = *(SDGP_LDS uint16_t*)(smem + m_stage[t] + (2 - q) * 2);
        } else {
            f.a[t] = *(SDGP_LDS u32x4_t*)(smem + a_stage[t] + (2 - q / 2) * 16 + (q & 1 ? 2u * plane_a : 0u));
        }
    };
    auto load_b = [&](Frags& f, int u, uint32_t set, int q) {
        SDGP_LDS unsigned char* wb = smem + b_lane[u] + set;
        if constexpr (SPARSE) {
            s16x4_t x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                x[i] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((SDGP_LDS s16x4_t*)(wb + q * L::kWSlab + ((i >> 1) * 16 + (i & 1) * 4) * L::kWRow));
            typedef short s16x16_t __attribute__((ext_vector_type(16)));
            const s16x16_t all = {x[0][0], x[0][1], x[0][2], x[0][3], x[1][0], x[1][1], x[1][2], x[1][3],
                                  x[2][0], x[2][1], x[2][2], x[2][3], x[3][0], x[3][1], x[3][2], x[3][3]};
            f.b[u] = __builtin_bit_cast(bf16x16_t, all);
        } else {
            s16x4_t x[2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
                x[i] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((SDGP_LDS s16x4_t*)(wb + (q / 2) * L::kWSlab + ((q & 1) * 16 + i * 4) * L::kWRow));
            typedef short s16x8_t __attribute__((ext_vector_type(8)));
            const s16x8_t all = {x[0][0], x[0][1], x[0][2], x[0][3], x[1][0], x[1][1], x[1][2], x[1][3]};
            f.b[u] = __builtin_bit_cast(bf16x8_t, all);
        }
    };

    wait_lds_copies<0>();
    __syncthreads();

    // ---- main loop
    uint32_t set_off = 0u, abuf = (uint32_t)L::off_a(), abuf_other = (uint32_t)L::off_a() + buf_bytes;
    Frags fr[2];
    auto chunk = [&](auto more, int pc2) __attribute__((always_inline)) {
        constexpr bool has1 = decltype(more)::value;
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const uint32_t other_set = (uint32_t)L::kWSet - set_off;
#pragma unroll
            for (int t = 0; t < TM; ++t) load_a(fr[0], t, 0);
#pragma unroll
            for (int u = 0; u < TN; ++u) load_b(fr[0], u, set_off, 0);
            Raw raw_next;
            int g = 0;   // the next matrix instruction
            auto gap = [&](auto&... values) __attribute__((always_inline)) {
                (pin_value(values), ...);
                constexpr int G = TM * TN;
                if (g >= KSTEPS * G) return;
                const int q = g / G, i = g % G;
                Frags& cur = fr[q & 1];
                Frags& nxt = fr[(q & 1) ^ 1];
                const int t = i / TN, u = i % TN;
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (SPARSE)
                    acc[t][u] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(__builtin_bit_cast(bf16x8_t, cur.a[t]), cur.b[u], acc[t][u], cur.meta[t], 0, 0);
                else
                    acc[t][u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, cur.a[t]), cur.b[u], acc[t][u], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (q + 1 < KSTEPS) {
                    if (i < TN) load_b(nxt, i, set_off, q + 1);
                    else if (i - TN < TM) load_a(nxt, i - TN, q + 1);
                }
                if (has1 && g == 0 && (r == 2 || r + 1 < ITEMS)) raw_next = load_item(r < 2 ? r + 1 : 0, r < 2 ? pc1 : pc2);
                if (g < WCOPIES) {
                    if (r < 2) copy_w(pc, r + 1, other_set, g);
                    else if (has1) copy_w(pc1, 0, other_set, g);
                }
                __builtin_amdgcn_sched_barrier(0);
                ++g;
            };
            if (has1 && r < ITEMS) rank_item(raw, r, pc1, abuf_other, gap);
#pragma unroll
            for (int i = 0; i < KSTEPS * TM * TN; ++i) gap();
            __builtin_amdgcn_sched_barrier(0);
            wait_lds_copies<0>();
            __syncthreads();
            raw = raw_next;
            set_off = other_set;
            const uint32_t da = r < 2 ? 0u - (uint32_t)GW * 16u : (uint32_t)GW * 32u + (abuf_other - abuf);
            const uint32_t dm = r < 2 ? 0u - (uint32_t)GW * 2u : (uint32_t)GW * 4u + (abuf_other - abuf);
#pragma unroll
            for (int t = 0; t < TM; ++t) a_stage[t] += da, m_stage[t] += dm;
        }
    };
    for (int c = 0; c + 1 < nchunks; ++c) {
        const int pc2 = pc1 + 1 == nchunks ? 0 : pc1 + 1;   // (in front of the last chunk nobody reads what is asked for)
        chunk(std::true_type{}, pc2);
        pc = pc1, pc1 = pc2;
        const uint32_t x = abuf; abuf = abuf_other; abuf_other = x;
    }
    chunk(std::false_type{}, 0);

    // ---- epilogue: whole 128-byte rows straight from the registers (through LDS, with a barrier: 1.01 to 1.03 of the time of a call)
    const int col = n0 + wn * 64 + 2 * (lane & 28);
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const u32x4_t out = quad_rows(acc[t][0], acc[t][1], g, lane);
            const int px = t0 + wm * WM + t * 32 + 8 * g + 4 * (lane >> 5) + (lane & 3);
            if (px < p.pixels && col < p.C_in) __builtin_nontemporal_store(out, reinterpret_cast<u32x4_t*>(p.dD + (size_t)px * p.C_in + col));
        }
}

}  // namespace sdgp

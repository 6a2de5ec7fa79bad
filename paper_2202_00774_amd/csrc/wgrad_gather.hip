// Weight gradient on the matrix cores for any filter and stride (Sec. II-A, Fig. 1), bf16, channel counts that are
// multiples of 8:
//   dW[k, tap, c] = sum over pixels of dO[pixel][k] * D[the pixel the tap reads][c]
// One workgroup takes KB output x CB input channels of one tap and a run of gradient pixels (a split), 64 pixels at a
// time.  The reduction runs over pixels, so both operands of v_mfma_f32_32x32x16_bf16 are read from [pixel][channel] tiles in
// LDS, the layout they have in memory, with the transposing read ds_read_b64_tr_b16.
//   * Bound by memory: a 1x1 layer does 2*KB*CB flops per 2*(KB+CB) bytes, so the block shape is the one that reads the
//     two tensors the fewest times over (64 x 256, 128 x 128, 256 x 64; 64 x 64 where neither side is wider).
//   * Eight wavefronts (four for 64 x 64), 32 x 64 results each: two per SIMD, so that one's copy addresses, reads and sums
//     overlap the other's matrix instructions (four wavefronts of 64 x 64 on 32-pixel chunks: 36 us against 29 on 1x1 256 ->
//     64, 69 against 39 on the gathered 3x3 168 -> 40 at 35x35, batch 32).
//   * Every byte takes the direct path into LDS (16 bytes per lane, no registers); three buffers, two chunks in flight
//     while one is multiplied, one barrier per chunk.  The 16-byte columns of a row are
//     exchanged by row on the way (the copy's source address), so that the four rows of a transposing read lie in four
//     different quarters of the 64 banks.
//   * Pixels whose tap falls outside the image, and pixels past the run's end, are zeros on BOTH sides: they add nothing
//     whatever the other side holds.  Channels past the end repeat the last ones and are not stored.
//   * The splits' partial filters (fp32) are added in a fixed order by a second kernel: the result is the same from call
//     to call.
// 1x1 256 -> 64 at 56x56, batch 64 (128 MB): 31 us with the sum of the splits, 105 ms with one workgroup per filter
// element.
#include "fastdiv.h"
#include "lds_copy.h"
#include "wgrad_gather.h"

namespace sdgp {

namespace {

constexpr int kPX = 64;      // pixels per chunk
constexpr int kSets = 3;     // LDS buffers
constexpr int kRun = 2;      // chunks summed on their own, a power of two

__device__ const uint32_t kWgradZeros[4] __attribute__((aligned(16))) = {};

struct GatherParams {
    const uint16_t* D;
    const uint16_t* dO;
    float* out;               // partial filters [nsplit][nW], or dW itself when there is one split
    int64_t nW, npix;
    int64_t per;              // pixels per split, a multiple of kPX
    int H, Wd, P, Q, C_in, C_out, S, stride, pad, ntaps;
    int kblocks, cblocks;
    FastDiv by_q, by_p;
    int plain;                // 1x1, stride 1: a gradient pixel reads the image pixel of the same index
};

template <int KB, int CB, int WVK, int WVC>
__global__ void __launch_bounds__(WVK* WVC * 64) wgrad_gather(const GatherParams p) {
    constexpr int NW = WVK * WVC, TM = KB / WVK / 32, TN = CB / WVC / 32;
    constexpr int PA = KB * 2, PB = CB * 2;                       // bytes per pixel of the two tiles
    constexpr int kSetBytes = kPX * (PA + PB);
    constexpr int CA = kPX * PA / 1024 / NW, CBC = kPX * PB / 1024 / NW;   // copies per wavefront and chunk
    static_assert(CA * NW * 1024 == kPX * PA && CBC * NW * 1024 == kPX * PB, "every wavefront copies the same number of units");
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    SDGP_LDS unsigned char* const smem = (SDGP_LDS unsigned char*)lds;
    const uint32_t smem_base = (uint32_t)(uintptr_t)smem;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wk = wave / WVC, wc = wave % WVC;

    const int tap = (int)(blockIdx.y % p.ntaps), block = (int)(blockIdx.y / p.ntaps);
    const int kb = block / p.cblocks, cb = block % p.cblocks;
    const int r = tap / p.S, s = tap - r * p.S;
    const int64_t pix0 = (int64_t)blockIdx.x * p.per;
    const int64_t pix1 = pix0 + p.per < p.npix ? pix0 + p.per : p.npix;
    const int nchunks = (int)((pix1 - pix0 + kPX - 1) / kPX);

    // 16-byte column exchange: rows of 128 bytes lie two to a bank window, longer ones start a window each
    auto swz = [](int row, int pitch) { return pitch == 128 ? ((row >> 1) & 1) * 4 : (row & 3) * 4; };

    // The lane's part of a copy of 1024 bytes: row (pixel) and first channel, clamped to the tensor's last 8.
    constexpr int RA = 1024 / PA, RB = 1024 / PB;
    const int ra = lane / (PA / 16), rb = lane / (PB / 16);
    int ca[CA], cc[CBC];
#pragma unroll
    for (int i = 0; i < CA; ++i) {
        const int row = (wave * CA + i) * RA + ra;
        const int c = kb * KB + ((lane % (PA / 16)) ^ swz(row, PA)) * 8;
        ca[i] = c <= p.C_out - 8 ? c : p.C_out - 8;
    }
#pragma unroll
    for (int i = 0; i < CBC; ++i) {
        const int row = (wave * CBC + i) * RB + rb;
        const int c = cb * CB + ((lane % (PB / 16)) ^ swz(row, PB)) * 8;
        cc[i] = c <= p.C_in - 8 ? c : p.C_in - 8;
    }
    // image pixel that gradient pixel `pix` reads through this tap, or -1
    auto source = [&](int64_t pix) -> int64_t {
        if (pix >= pix1) return -1;
        if (p.plain) return pix;
        const uint32_t n = (uint32_t)pix, row = divide(n, p.by_q), q = n - row * (uint32_t)p.Q;
        const uint32_t b = divide(row, p.by_p), pp = row - b * (uint32_t)p.P;
        const int h = (int)pp * p.stride + r - p.pad, w = (int)q * p.stride + s - p.pad;
        if ((unsigned)h >= (unsigned)p.H || (unsigned)w >= (unsigned)p.Wd) return -1;
        return ((int64_t)b * p.H + h) * p.Wd + w;
    };
    auto copy_chunk = [&](int chunk, int set) {
        const uint32_t base = smem_base + (uint32_t)(set * kSetBytes);
#pragma unroll
        for (int i = 0; i < CA; ++i) {
            const int64_t pix = pix0 + (int64_t)chunk * kPX + (wave * CA + i) * RA + ra;
            const void* src = source(pix) >= 0 ? (const void*)(p.dO + pix * p.C_out + ca[i]) : (const void*)kWgradZeros;
            lds_copy16(src, base + (uint32_t)(wave * CA + i) * 1024u);
        }
#pragma unroll
        for (int i = 0; i < CBC; ++i) {
            const int64_t pix = pix0 + (int64_t)chunk * kPX + (wave * CBC + i) * RB + rb;
            const int64_t at = source(pix);
            const void* src = at >= 0 ? (const void*)(p.D + at * p.C_in + cc[i]) : (const void*)kWgradZeros;
            lds_copy16(src, base + (uint32_t)(kPX * PA) + (uint32_t)(wave * CBC + i) * 1024u);
        }
    };

    f32x16_t acc[TM][TN];
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int u = 0; u < TN; ++u)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[t][u][e] = 0.0f;

    // lane's part of a transposing read: 16-lane group g takes pixels 8*(g/2) + (lane%16)/4 (and those plus 4) and the
    // four channels 16*(g%2) + 4*(lane%4) of a 32-channel tile
    const int g = lane >> 4, l16 = lane & 15;
    const int prow = 8 * (g >> 1) + (l16 >> 2);
    const int x16 = 2 * (g & 1) + ((l16 & 3) >> 1), b8 = (l16 & 1) * 8;
    uint32_t fa[TM], fb[TN];
#pragma unroll
    for (int t = 0; t < TM; ++t) fa[t] = (uint32_t)(prow * PA + ((((wk * TM + t) * 4 + x16) ^ swz(prow, PA)) * 16) + b8);
#pragma unroll
    for (int u = 0; u < TN; ++u) fb[u] = (uint32_t)(kPX * PA + prow * PB + ((((wc * TN + u) * 4 + x16) ^ swz(prow, PB)) * 16) + b8);
    auto frag = [&](uint32_t at, int pitch) {
        const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((SDGP_LDS s16x4_t*)(smem + at));
        const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((SDGP_LDS s16x4_t*)(smem + at + 4 * pitch));
        typedef short s16x8_t __attribute__((ext_vector_type(8)));
        const s16x8_t all = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        return __builtin_bit_cast(bf16x8_t, all);
    };

    // Runs of kRun chunks are summed on their own and added to an fp64 total: a chain of fp32 additions errs by its length.
    // (Relative error over thirty shapes 5.4e-8 to 7.2e-8; 6.6e-8 to 1.6e-7 as one chain, 5.5e-8 to 1.4e-7 for the plain
    // kernel's short chains; 2 us of the call below.)
    double total[TM][TN][16];
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int u = 0; u < TN; ++u)
#pragma unroll
            for (int e = 0; e < 16; ++e) total[t][u][e] = 0.0;

    copy_chunk(0, 0);
    copy_chunk(1, 1);
    int set = 0, next_set = 2;
    for (int chunk = 0; chunk < nchunks; ++chunk) {
        // this chunk has landed (the copies of the one after it may stay in flight), for every wavefront; the set that
        // the next copies go to was read one chunk ago, before this barrier
        wait_lds_copies<CA + CBC>();
        __syncthreads();
        copy_chunk(chunk + 2, next_set);   // (past the run's end: zeros)
        const uint32_t base = (uint32_t)(set * kSetBytes);
#pragma unroll
        for (int st = 0; st < kPX / 16; ++st) {
            bf16x8_t a[TM], b[TN];
#pragma unroll
            for (int t = 0; t < TM; ++t) a[t] = frag(base + fa[t] + st * 16 * PA, PA);
#pragma unroll
            for (int u = 0; u < TN; ++u) b[u] = frag(base + fb[u] + st * 16 * PB, PB);
#pragma unroll
            for (int t = 0; t < TM; ++t)
#pragma unroll
                for (int u = 0; u < TN; ++u) acc[t][u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[t], b[u], acc[t][u], 0, 0, 0);
        }
        if ((chunk & (kRun - 1)) == kRun - 1) {
#pragma unroll
            for (int t = 0; t < TM; ++t)
#pragma unroll
                for (int u = 0; u < TN; ++u)
#pragma unroll
                    for (int e = 0; e < 16; ++e) total[t][u][e] += (double)acc[t][u][e], acc[t][u][e] = 0.0f;
        }
        set = set == kSets - 1 ? 0 : set + 1;
        next_set = next_set == kSets - 1 ? 0 : next_set + 1;
    }
    wait_lds_copies<0>();   // no copy may land in LDS that another workgroup owns by then

    // result register e of lane l: output channel 8*(e/4) + 4*(l/32) + e%4, input channel l%32 of the tile
    float* const out = p.out + (int64_t)blockIdx.x * p.nW;
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int u = 0; u < TN; ++u)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int k = kb * KB + (wk * TM + t) * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
                const int c = cb * CB + (wc * TN + u) * 32 + (lane & 31);
                if (k < p.C_out && c < p.C_in) out[((int64_t)k * p.ntaps + tap) * p.C_in + c] = (float)(total[t][u][e] + (double)acc[t][u][e]);
            }
}

struct Shape {
    int kb, cb, per_cu;   // channels of a block, workgroups per compute unit
};
constexpr Shape kShapes[] = {{64, 64, 3}, {64, 256, 1}, {128, 128, 1}, {256, 64, 1}};

template <int KB, int CB, int WVK, int WVC>
int launch(const GatherParams& p, const WgradGatherPlan& pl, hipStream_t stream) {
    constexpr int lds = kSets * kPX * (KB + CB) * 2;
    auto kern = wgrad_gather<KB, CB, WVK, WVC>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return SDGP_ERR_HIP;
    hipLaunchKernelGGL(kern, dim3((unsigned)pl.nsplit, (unsigned)(p.kblocks * p.cblocks * p.ntaps)), dim3(WVK * WVC * 64), lds, stream, p);
    return launch_status();
}

}  // namespace

WgradGatherPlan wgrad_gather_plan(int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out, int R, int S, int stride,
                                  int pad, int dt) {
    WgradGatherPlan pl{};
    const int64_t P = (H + 2 * pad - R) / stride + 1, Q = (Wd + 2 * pad - S) / stride + 1;
    const int64_t limit = (int64_t)1 << 30;
    if (dt != SDGP_BF16 || C_in <= 0 || C_out <= 0 || C_in % 8 != 0 || C_out % 8 != 0 || C_in > (1 << 20) || C_out > (1 << 20)) return pl;
    if (H > (1 << 20) || Wd > (1 << 20) || P <= 0 || Q <= 0 || B <= 0) return pl;
    if (P * Q > limit / B) return pl;
    const int64_t npix = B * P * Q, chunks = (npix + kPX - 1) / kPX;
    // A filter of a few blocks' results and a few chunks of pixels leave the chip idle here, and the plain kernel's
    // workgroup per filter element is the faster one.  Measured (this kernel's time over the plain one's): 576 elements 1.3
    // at 128 pixels, 2.2 at 512, 1.34 at 2048, 1.02 at 3072; 1600 (5x5) 1.06, 1.6, 0.83; 2304 (3x3) 0.90, 1.32, 0.57 and 1.07 at 768;
    // 1x1 1024 1.06, 1.36, 0.79, 2048 0.86, 0.85, 0.36 (of 256 x 8 channels 1.12, 1.35, 1.02 at 1024); 32 pixels and 512 elements 1.16, 64 pixels
    // 0.91-1.08 and less from 1600 elements on.
    const int64_t nW = C_out * R * S * C_in;
    if (nW <= (R * S > 1 || C_in < 32 || C_out < 32 ? 2304 : 1024) && (npix >= 128 || nW <= 600) && npix < 4096 && nW * npix <= 1800000) return pl;
    // channels read per pixel and tap, over all blocks
    int64_t best = -1;
    for (int i = 0; i < 4; ++i) {
        const Shape& sh = kShapes[i];
        const int64_t reads = ((C_out + sh.kb - 1) / sh.kb) * ((C_in + sh.cb - 1) / sh.cb) * (sh.kb + sh.cb);
        if (best < 0 || reads < best) best = reads, pl.shape = i;
    }
    const Shape& sh = kShapes[pl.shape];
    pl.kblocks = (C_out + sh.kb - 1) / sh.kb, pl.cblocks = (C_in + sh.cb - 1) / sh.cb;
    const int64_t blocks = pl.kblocks * pl.cblocks * R * S;
    if (blocks > 65535) return pl;
    // One round of workgroups, none with fewer than four chunks, most with eight or more.  One of the large blocks per compute
    // unit: every split writes and reads a partial filter (1x1 256 -> 64 at 56x56, batch 64, four-wavefront workgroups: 38 us
    // with two per unit, 31 with one; 1024 -> 256 at 14x14 25 / 20).  Blocks of 64 x 64 take 48 KB of LDS, so three fit; a
    // fourth begins a second round (2x2 64 -> 64 at 56x56, batch 64 40.8 us with four, 30.9 with three; 3x3 64 -> 40 at 28x28
    // 25.4, 22.6; 7x7 stride 2 32.1, 29.4; fifty shapes of one round 0.98-1.02).  Large 3x3 layers are faster with it all the
    // same, for a reason that was not found (64 -> 64 stride 2 at 56x56, batch 256 61.5, 77.3; 56 -> 56 209, 256).
    const int per_cu = pl.shape == 0 && R * S == 9 && chunks >= 3000 ? 4 : sh.per_cu;
    int64_t ns = 256 * per_cu / blocks;
    if (ns > (chunks + 7) / 8) ns = (chunks + 7) / 8;
    if (ns < 1) ns = 1;
    pl.per = (chunks + ns - 1) / ns * kPX;
    pl.nsplit = (npix + pl.per - 1) / pl.per;
    pl.ok = true;
    return pl;
}

int wgrad_gather_launch(const WgradGatherPlan& pl, const void* D, const void* dO, float* out, int64_t B, int64_t H, int64_t Wd,
                        int64_t C_in, int64_t C_out, int R, int S, int stride, int pad, hipStream_t stream) {
    GatherParams p{};
    p.D = static_cast<const uint16_t*>(D), p.dO = static_cast<const uint16_t*>(dO), p.out = out;
    p.H = (int)H, p.Wd = (int)Wd, p.P = (int)((H + 2 * pad - R) / stride + 1), p.Q = (int)((Wd + 2 * pad - S) / stride + 1);
    p.nW = C_out * R * S * C_in, p.npix = B * p.P * p.Q, p.per = pl.per;
    p.C_in = (int)C_in, p.C_out = (int)C_out, p.S = S, p.stride = stride, p.pad = pad, p.ntaps = R * S;
    p.kblocks = (int)pl.kblocks, p.cblocks = (int)pl.cblocks;
    p.by_q = fast_div((uint32_t)p.Q), p.by_p = fast_div((uint32_t)p.P);
    p.plain = R == 1 && S == 1 && stride == 1 && pad == 0;
    switch (pl.shape) {
        case 0: return launch<64, 64, 2, 2>(p, pl, stream);
        case 1: return launch<64, 256, 2, 4>(p, pl, stream);
        case 2: return launch<128, 128, 4, 2>(p, pl, stream);
        default: return launch<256, 64, 8, 1>(p, pl, stream);
    }
}

}  // namespace sdgp

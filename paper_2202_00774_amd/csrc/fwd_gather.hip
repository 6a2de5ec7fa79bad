// Forward convolution on the matrix cores for any filter and stride (Sec. II-A, Fig. 1), bf16, channel counts that are
// multiples of 8:
//   O[pixel, k] = sum over taps and channels of D[the pixel the tap reads, c] * W[k, tap, c]
// A GEMM whose rows are output pixels and whose reduction walks (tap, 32 channels) steps.  Both operands lie along the
// reduction in memory, so a fragment of v_mfma_f32_32x32x16_bf16 is one 16-byte LDS read on either side and W is taken
// as it is (no transposed copy, no workspace).
//   * Workgroup = 4 wavefronts on 128 pixels x BN output channels, each wavefront 64 x 64 or 64 x 32.
//   * Both tiles of a step take the direct path into LDS (16 bytes per lane); the next step's copies are in flight while
//     a step is multiplied, SETS buffers and several workgroups per CU cover the rest of their latency.  A lane's image
//     pixel of every row it copies is kept in registers, so a step costs one 64-bit addition per copy and a new tap a
//     bounds check.
//   * 16-byte columns of a row are exchanged by row so that the sixteen lanes of a fragment read meet all 64 banks.
//   * Consecutive tiles share image rows, and the column tiles of one row tile all of them: tiles are dealt to the eight
//     XCDs in runs, so that each one's L2 serves its own part of the image.
// 3x3 stride 2 128 -> 128 at 56x56, batch 128: 60 us a call = 490 TFLOP/s (53 in the kernel; a wavefront waits half of its
// time, for copies between two barriers); one thread per output element took 50.1 ms.
// Pixels outside the image are zeros.  Zero times a non-finite weight is NaN where the definition has no term, so a NaN
// of a pixel whose window leaves the image is summed again without those taps.
#include "lds_copy.h"

namespace sdgp {

namespace {

constexpr int kRows = 128, kKC = 32;
__device__ const uint32_t kFwdZeros[4] __attribute__((aligned(16))) = {};

struct FwdParams {
    const uint16_t* D;
    const uint16_t* W;
    uint16_t* O;
    int64_t rows;          // output pixels
    int H, Wd, P, Q, C_in, C_out, R, S, stride, pad;
    int col_tiles, nblocks, per_xcd;
};

template <int BN, int SETS>
struct FwdLayout {
    static constexpr int kSet = (kRows + BN) * kKC * 2, kOutPitch = BN * 2 + 16;
    static constexpr int kTotal = SETS * kSet > kRows * kOutPitch ? SETS * kSet : kRows * kOutPitch;
};

template <int BN, int SETS>
__global__ void __launch_bounds__(256) fwd_gather(const FwdParams p) {
    using L = FwdLayout<BN, SETS>;
    constexpr int WVN = 2, TM = 2, TN = BN / WVN / 32, NA = kRows / 64, NB = BN / 64;   // copies per wavefront and step
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    SDGP_LDS unsigned char* const smem = (SDGP_LDS unsigned char*)lds;
    const uint32_t smem_base = (uint32_t)(uintptr_t)smem;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WVN, wn = wave % WVN;

    const int logical = (int)(blockIdx.x & 7) * p.per_xcd + (int)(blockIdx.x >> 3);
    if (logical >= p.nblocks) return;
    const int64_t m0 = (int64_t)(logical / p.col_tiles) * kRows;
    const int n0 = logical % p.col_tiles * BN;

    // What this lane copies: 16-byte column `col` of the channels of a step, for row 16 u + lane / 4 of each of its units u
    const int crow = lane >> 2, col = ((lane & 3) ^ ((crow >> 2) & 3)) * 8;
    int hb[NA], wb[NA];                        // image position of tap (0, 0)
    const uint16_t* image[NA];
    const uint16_t* wrow[NB];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        int64_t row = m0 + (wave * NA + i) * 16 + crow;
        const bool live = row < p.rows;
        if (!live) row = p.rows - 1;
        const int64_t line = row / p.Q, b = line / p.P;
        hb[i] = live ? (int)(line - b * p.P) * p.stride - p.pad : -(1 << 20);   // (a row past the end is outside at every tap)
        wb[i] = (int)(row - line * p.Q) * p.stride - p.pad;
        image[i] = p.D + b * p.H * p.Wd * p.C_in + col;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        int k = n0 + (wave * NB + i) * 16 + crow;
        if (k >= p.C_out) k = p.C_out - 1;
        wrow[i] = p.W + (int64_t)k * p.R * p.S * p.C_in + col;
    }
    // the walk over (tap row, tap column, channels)
    int r = 0, s = 0, c = 0;
    const uint16_t* a[NA];                     // this tap's pixel, or null outside the image
    auto enter_tap = [&]() {
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int h = hb[i] + r, w = wb[i] + s;
            const bool in = (unsigned)h < (unsigned)p.H && (unsigned)w < (unsigned)p.Wd;
            a[i] = in ? image[i] + ((int64_t)h * p.Wd + w) * p.C_in : nullptr;
        }
    };
    enter_tap();
    auto copy_step = [&](int set) {
        const uint32_t base = smem_base + (uint32_t)(set * L::kSet);
        const bool has = c + col < p.C_in;     // (the last step of a tap may hold fewer than 32 channels)
#pragma unroll
        for (int i = 0; i < NA; ++i)
            lds_copy16(has && a[i] != nullptr ? (const void*)(a[i] + c) : (const void*)kFwdZeros, base + (uint32_t)(wave * NA + i) * 1024u);
#pragma unroll
        for (int i = 0; i < NB; ++i)
            lds_copy16(has ? (const void*)(wrow[i] + c) : (const void*)kFwdZeros, base + (uint32_t)(kRows * kKC * 2) + (uint32_t)(wave * NB + i) * 1024u);
        c += kKC;
        if (c >= p.C_in) {
            c = 0;
            if (++s == p.S) s = 0, ++r;
#pragma unroll
            for (int i = 0; i < NB; ++i) wrow[i] += p.C_in;
            enter_tap();
        }
    };

    f32x16_t acc[TM][TN];
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int u = 0; u < TN; ++u)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[t][u][e] = 0.0f;
    uint32_t fa[TM], fb[TN];
#pragma unroll
    for (int t = 0; t < TM; ++t) {
        const uint32_t row = (uint32_t)(wm * 64 + t * 32 + (lane & 31));
        fa[t] = row * 64u + ((((uint32_t)(lane >> 5) ^ (row >> 2)) & 3u) << 4);
    }
#pragma unroll
    for (int u = 0; u < TN; ++u) {
        const uint32_t row = (uint32_t)(wn * (TN * 32) + u * 32 + (lane & 31));
        fb[u] = (uint32_t)(kRows * kKC * 2) + row * 64u + ((((uint32_t)(lane >> 5) ^ (row >> 2)) & 3u) << 4);
    }

    const int steps = p.R * p.S * ((p.C_in + kKC - 1) / kKC);
#pragma unroll
    for (int i = 0; i < SETS - 1; ++i)
        if (i < steps) copy_step(i);
    int set = 0, next_set = SETS - 1;
    for (int st = 0; st < steps; ++st) {
        // this step's copies have landed, for every wavefront; the buffer that the next copies go to was read one step
        // ago, in front of this barrier
        if (st + SETS - 1 <= steps) wait_lds_copies<(SETS - 2) * (NA + NB)>();
        else wait_lds_copies<0>();
        __syncthreads();
        if (st + SETS - 1 < steps) copy_step(next_set);
        const uint32_t base = (uint32_t)(set * L::kSet);
#pragma unroll
        for (int ks = 0; ks < kKC / 16; ++ks) {
            bf16x8_t fragA[TM], fragB[TN];
#pragma unroll
            for (int t = 0; t < TM; ++t) fragA[t] = __builtin_bit_cast(bf16x8_t, *(SDGP_LDS u32x4_t*)(smem + base + (fa[t] ^ (uint32_t)(ks * 32))));
#pragma unroll
            for (int u = 0; u < TN; ++u) fragB[u] = __builtin_bit_cast(bf16x8_t, *(SDGP_LDS u32x4_t*)(smem + base + (fb[u] ^ (uint32_t)(ks * 32))));
#pragma unroll
            for (int t = 0; t < TM; ++t)
#pragma unroll
                for (int u = 0; u < TN; ++u) acc[t][u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fragA[t], fragB[u], acc[t][u], 0, 0, 0);
        }
        set = set + 1 == SETS ? 0 : set + 1;
        next_set = next_set + 1 == SETS ? 0 : next_set + 1;
    }
    __syncthreads();   // every wavefront has read its last fragments: the tiles' LDS becomes the result's

#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int u = 0; u < TN; ++u)
#pragma unroll
            for (int e = 0; e < 16; e += 2) {
                const int m = wm * 64 + t * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3), n = wn * (TN * 32) + u * 32 + (lane & 31);
                const uint32_t pk = float2_to_bf16x2(acc[t][u][e], acc[t][u][e + 1]);   // rows m and m + 1
                *(SDGP_LDS uint16_t*)(smem + m * L::kOutPitch + n * 2) = (uint16_t)pk;
                *(SDGP_LDS uint16_t*)(smem + (m + 1) * L::kOutPitch + n * 2) = (uint16_t)(pk >> 16);
            }
    __syncthreads();
    uint32_t nans = 0;   // which of this lane's vectors hold a NaN
#pragma unroll 4
    for (int i = 0; i < kRows * (BN / 8) / 256; ++i) {
        const int x = tid + 256 * i, m = x / (BN / 8), cc = x % (BN / 8);
        const int64_t row = m0 + m;
        if (row >= p.rows || n0 + cc * 8 >= p.C_out) continue;
        const u32x4_t v = *(SDGP_LDS u32x4_t*)(smem + m * L::kOutPitch + cc * 16);
        if (p.pad > 0) {
            bool nan = false;
#pragma unroll
            for (int y = 0; y < 4; ++y) nan = nan || (v[y] & 0x7FFFu) > 0x7F80u || (v[y] & 0x7FFF0000u) > 0x7F800000u;
            nans |= (uint32_t)nan << i;
        }
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4_t*>(p.O + row * p.C_out + n0 + cc * 8));
    }
    if (__builtin_expect(nans != 0, 0)) {
        uint64_t args = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();   // (read again: nothing below is kept in registers above)
        asm volatile("" : "+s"(args));
        const auto& q = *reinterpret_cast<const __attribute__((address_space(4))) FwdParams*>(args);
#pragma nounroll
        for (; nans != 0; nans &= nans - 1) {
            const int x = tid + 256 * (__ffs((int)nans) - 1), m = x / (BN / 8), cc = x % (BN / 8);
            const int row = (int)m0 + m, line = row / q.Q, b = line / q.P;             // (at most 2^30 rows)
            const int h0 = (line - b * q.P) * q.stride - q.pad, w0 = (row - line * q.Q) * q.stride - q.pad;
            if (h0 >= 0 && w0 >= 0 && h0 + q.R <= q.H && w0 + q.S <= q.Wd) continue;   // no tap outside
            u32x4_t v = *(SDGP_LDS u32x4_t*)(smem + m * L::kOutPitch + cc * 16);
            const int64_t wstep = (int64_t)q.R * q.S * q.C_in;
            const uint16_t* wk = q.W + (int64_t)(n0 + cc * 8) * wstep;
#pragma nounroll
            for (int y = 0; y < 4; ++y, wk += 2 * wstep) {   // two channels at a time
                uint32_t pair = v[0];
                bool lo = (pair & 0x7FFFu) > 0x7F80u, hi = (pair & 0x7FFF0000u) > 0x7F800000u;
                float s0 = 0.0f, s1 = 0.0f;
                const uint16_t* w = wk;
#pragma nounroll
                for (int t = 0; t < q.R * q.S && (lo || hi); ++t, w += q.C_in) {   // (a NaN of the taps inside stays one)
                    const int h = h0 + t / q.S, ww = w0 + t % q.S;
                    if ((unsigned)h >= (unsigned)q.H || (unsigned)ww >= (unsigned)q.Wd) continue;
                    const uint16_t* d = q.D + (((int64_t)b * q.H + h) * q.Wd + ww) * q.C_in;
#pragma nounroll
                    for (int ch = 0; ch < q.C_in && (lo || hi); ch += 4) {
                        typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
                        const u32x2_t dv = *reinterpret_cast<const u32x2_t*>(d + ch), wa = *reinterpret_cast<const u32x2_t*>(w + ch),
                                      wb = *reinterpret_cast<const u32x2_t*>(w + wstep + ch);
#pragma unroll
                        for (int z = 0; z < 2; ++z) {
                            s0 = fmaf(bf16_to_float(dv[z] & 0xFFFFu), bf16_to_float(wa[z] & 0xFFFFu), s0);
                            s0 = fmaf(bf16_to_float(dv[z] >> 16), bf16_to_float(wa[z] >> 16), s0);
                            s1 = fmaf(bf16_to_float(dv[z] & 0xFFFFu), bf16_to_float(wb[z] & 0xFFFFu), s1);
                            s1 = fmaf(bf16_to_float(dv[z] >> 16), bf16_to_float(wb[z] >> 16), s1);
                        }
                        lo = lo && s0 == s0, hi = hi && s1 == s1;
                    }
                }
                if (lo) pair = (pair & 0xFFFF0000u) | float_to_bf16(s0);
                if (hi) pair = (pair & 0xFFFFu) | (float_to_bf16(s1) << 16);
                v = u32x4_t{v[1], v[2], v[3], pair};   // (all four pairs pass the first place)
            }
            *reinterpret_cast<u32x4_t*>(q.O + (int64_t)row * q.C_out + n0 + cc * 8) = v;
        }
    }
}

template <int BN, int SETS>
int launch(const FwdParams& p, hipStream_t stream) {
    auto kern = fwd_gather<BN, SETS>;
    constexpr int lds = FwdLayout<BN, SETS>::kTotal;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return SDGP_ERR_HIP;
    hipLaunchKernelGGL(kern, dim3((unsigned)(p.per_xcd * 8)), dim3(256), lds, stream, p);
    return launch_status();
}

}  // namespace

// A positive value: the layer or the pointers do not fit.
int fwd_gather_launch(const void* D, const void* W, void* O, int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out,
                      int R, int S, int stride, int pad, int dt, hipStream_t stream) {
    if (dt != SDGP_BF16 || C_in <= 0 || C_out <= 0 || C_in % 8 != 0 || C_out % 8 != 0) return 1;
    if (!is_aligned16(D) || !is_aligned16(W) || !is_aligned16(O)) return 1;
    const int64_t P = (H + 2 * pad - R) / stride + 1, Q = (Wd + 2 * pad - S) / stride + 1;
    if (H > (1 << 18) || Wd > (1 << 18) || C_in > (1 << 24) || C_out > (1 << 24) || H * Wd > ((int64_t)1 << 40) / C_in) return 1;
    FwdParams p{};
    p.D = static_cast<const uint16_t*>(D), p.W = static_cast<const uint16_t*>(W), p.O = static_cast<uint16_t*>(O);
    p.rows = B * P * Q;
    p.H = (int)H, p.Wd = (int)Wd, p.P = (int)P, p.Q = (int)Q, p.C_in = (int)C_in, p.C_out = (int)C_out;
    p.R = R, p.S = S, p.stride = stride, p.pad = pad;
    // Tiles of 128 channels unless they leave a compute unit without one (3x3 stride 2 512 -> 512 at 14x14, batch 16: 28 such
    // tiles 66 us, 56 of 64 channels 45).  Four LDS buffers where at most two workgroups meet on a compute unit anyway (the
    // same layer 56 us with 128 channels), two where four of them fit beside each other (1x1 64 -> 256 at 56x56 47 us
    // against 55 with four buffers).
    const int64_t row_tiles = (p.rows + kRows - 1) / kRows;
    const int bn = C_out > 64 && row_tiles * ((C_out + 127) / 128) >= 256 ? 128 : 64;
    p.col_tiles = (int)((C_out + bn - 1) / bn);
    if (row_tiles > (1 << 23) / p.col_tiles) return 1;   // (a launch holds fewer than 2^32 threads)
    const int64_t blocks = row_tiles * p.col_tiles;
    p.nblocks = (int)blocks, p.per_xcd = (int)((blocks + 7) / 8);
    if (blocks <= 512) return bn == 128 ? launch<128, 4>(p, stream) : launch<64, 4>(p, stream);
    return bn == 128 ? launch<128, 2>(p, stream) : launch<64, 2>(p, stream);
}

}  // namespace sdgp

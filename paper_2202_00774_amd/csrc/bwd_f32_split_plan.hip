// Launcher of the fp32 backward-data products on the bf16 matrix instructions.
#include "bwd_f32_split_tiles.h"

namespace sdgp {

namespace {

template <int M, int RK, bool NLE2, bool SPARSE>
int first_pass(const SplitParams& p, hipStream_t stream) {
    hipLaunchKernelGGL((split_operands<M, RK, NLE2, SPARSE>), dim3((unsigned)(p.wblocks + p.gblocks)), dim3(256), 0, stream, p);
    return launch_status();
}
template <int M, bool NLE2, bool SPARSE>
int first_pass_rk(const SplitParams& p, int rk, hipStream_t stream) {
    if (rk == kRandom) return first_pass<M, kRandom, NLE2, SPARSE>(p, stream);
    if (rk == kGreedy) return first_pass<M, kGreedy, NLE2, SPARSE>(p, stream);
    return first_pass<M, kAdjusted, NLE2, SPARSE>(p, stream);
}

template <bool SPARSE, int ROWS, int NP>
int product(const SplitPlan& s, hipStream_t stream) {
    auto kern = f32_split<SPARSE, ROWS, NP>;
    constexpr int lds = SplitLayout<SPARSE, ROWS, NP>::kTotal;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return SDGP_ERR_HIP;
    hipLaunchKernelGGL(kern, dim3((unsigned)s.p.nblocks, 1, (unsigned)(s.p.stride * s.p.stride)), dim3(ROWS * 4), lds, stream, s.p);
    return launch_status();
}
template <bool SPARSE>
int product_shape(const SplitPlan& s, hipStream_t stream) {
    if (s.rows == 128) return product<SPARSE, 128, 256>(s, stream);
    return s.np == 384 ? product<SPARSE, 256, 384>(s, stream) : product<SPARSE, 256, 512>(s, stream);
}

}  // namespace

// Workspace bytes of a problem these kernels take, 0 for the others.
size_t bwd_f32_split_workspace(int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out, int R, int S, int stride, int pad, int n, int m) {
    SplitPlan s;
    return split_plan(s, B, H, Wd, C_in, C_out, R, S, stride, pad, n, m) ? s.bytes : 0;
}

// SDGP_OK after launching, a positive value when the problem does not fit or the workspace is missing or too small, or a
// negative sdgp_status.
int bwd_f32_split_launch(const void* dO, const void* W, void* dD, int64_t B, int64_t H, int64_t Wd, int64_t C_in, int64_t C_out, int R, int S,
                         int stride, int pad, int n, int m, int rk, uint64_t seed, void* workspace, size_t workspace_bytes, hipStream_t stream) {
    SplitPlan s;
    if (workspace == nullptr || !is_aligned16(workspace) || !is_aligned16(dO)) return 1;
    if (!split_plan(s, B, H, Wd, C_in, C_out, R, S, stride, pad, n, m) || workspace_bytes < s.bytes) return 1;
    SplitParams& p = s.p;
    p.dO = static_cast<const float*>(dO), p.W = static_cast<const float*>(W), p.dD = static_cast<float*>(dD);
    unsigned char* const ws = static_cast<unsigned char*>(workspace);
    p.planes = ws, p.idx = reinterpret_cast<uint16_t*>(ws + s.off_idx), p.wimg = ws + s.off_wimg;
    p.wnotes = reinterpret_cast<uint32_t*>(ws + s.off_wnotes), p.gnotes = reinterpret_cast<uint32_t*>(ws + s.off_gnotes);
    p.mix = seed_mix(seed);
    int rc;
    if (n == m) rc = first_pass<4, kDenseRanker, false, false>(p, stream);
    else if (m == 4) rc = s.sparse ? first_pass_rk<4, true, true>(p, rk, stream) : first_pass_rk<4, false, false>(p, rk, stream);
    else if (m == 8) rc = s.sparse ? first_pass_rk<8, true, true>(p, rk, stream) : first_pass_rk<8, false, false>(p, rk, stream);
    else if (m == 16) rc = s.sparse ? first_pass_rk<16, true, true>(p, rk, stream) : first_pass_rk<16, false, false>(p, rk, stream);
    else rc = n <= 2 ? first_pass_rk<32, true, false>(p, rk, stream) : first_pass_rk<32, false, false>(p, rk, stream);
    if (rc != SDGP_OK) return rc;
    return s.sparse ? product_shape<true>(s, stream) : product_shape<false>(s, stream);
}

}  // namespace sdgp

// Results of two 32 x 32 tiles side by side as rows of sixteen bytes, without a detour through LDS.
#pragma once

#include "bwd_tiled.h"

namespace sdgp {

// Registers 4 g .. 4 g + 3 of a lane are rows 8 g + 4 (lane / 32) + 0 .. 3 of one column (lane % 32) of either tile.  The four lanes of
// a quad exchange them as bf16 (rounded to nearest even): a lane ends with row lane % 4 of the quad's four columns in both tiles.  Column
// n of tile u stands for column 8 (n / 4) + 4 (u ^ (n / 16)) + n % 4 of the two tiles' 64, so these are eight consecutive ones.
__device__ __forceinline__ u32x4_t quad_rows(const f32x16_t& tile0, const f32x16_t& tile1, int g, int lane) {
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    const uint32_t row_sel = lane & 1 ? 0x03020706u : 0x05040100u;
    uint32_t quad[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const f32x16_t& x = u ? tile1 : tile0;
        const f32x2_t v01 = {x[4 * g], x[4 * g + 1]}, v23 = {x[4 * g + 2], x[4 * g + 3]};
        const uint32_t p01 = __builtin_bit_cast(uint32_t, __builtin_convertvector(v01, bf16x2_t));
        const uint32_t p23 = __builtin_bit_cast(uint32_t, __builtin_convertvector(v23, bf16x2_t));
        const uint32_t n01 = (uint32_t)__builtin_amdgcn_mov_dpp((int)p01, 0xB1, 0xF, 0xF, true);   // the neighbour's: lane ^ 1
        const uint32_t n23 = (uint32_t)__builtin_amdgcn_mov_dpp((int)p23, 0xB1, 0xF, 0xF, true);
        const uint32_t q01 = __builtin_amdgcn_perm(n01, p01, row_sel);   // even lanes: row 0 of two columns, odd ones: row 1
        const uint32_t q23 = __builtin_amdgcn_perm(n23, p23, row_sel);   // rows 2 and 3
        const uint32_t give = lane & 2 ? q01 : q23;
        const uint32_t got = (uint32_t)__builtin_amdgcn_mov_dpp((int)give, 0x4E, 0xF, 0xF, true);  // lane ^ 2
        quad[u][0] = lane & 2 ? got : q01, quad[u][1] = lane & 2 ? q23 : got;
    }
    const bool swap = (lane & 16) != 0;
    return u32x4_t{swap ? quad[1][0] : quad[0][0], swap ? quad[1][1] : quad[0][1], swap ? quad[0][0] : quad[1][0], swap ? quad[0][1] : quad[1][1]};
}

}  // namespace sdgp

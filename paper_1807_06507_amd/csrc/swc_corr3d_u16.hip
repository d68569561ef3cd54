// Instantiations of the fused 3-D kernels for MODE_U16.
#include "swc_corr3d.hpp"
#include "swc_internal.h"

namespace swc {

template <int KW>
static hipError_t go3(const P3D& g, bool block, bool vec, int grid, int wpb, hipStream_t s)
{
    if (block) {
        const dim3 gr(grid), bl(wpb * kWave);
        constexpr int kTall = block3_rows(MODE_U16, 9), kFlat = block3_rows(MODE_U16, 1);
        // (debug bit 1: the general y sums)
        if (g.ky == KW && g.sy == 1 && g.sz == 1 && !(g.force & 2))
            return launch_kernel(&corr3d_block_kernel<MODE_U16, KW, block3_rows(MODE_U16, KW), true>, gr, bl, 0, s, g);
        if (block3_rows(MODE_U16, g.ky) == kFlat)
            return launch_kernel(&corr3d_block_kernel<MODE_U16, KW, kFlat, false>, gr, bl, 0, s, g);
        return launch_kernel(&corr3d_block_kernel<MODE_U16, KW, kTall, false>, gr, bl, 0, s, g);
    }
    const size_t smem = (size_t)wpb * tile3d_lds_per_wave<MODE_U16, 2>(4);
    if (vec)
        return launch_kernel(&corr3d_kernel<MODE_U16, 4, KW, 2, true>, dim3(grid), dim3(wpb * kWave), smem, s, g);
    return launch_kernel(&corr3d_kernel<MODE_U16, 4, KW, 2, false>, dim3(grid), dim3(wpb * kWave), smem, s, g);
}

hipError_t launch_fast3d_modeu16(const P3D& g, int KW, bool block, bool vec, int grid, int wpb,
                               hipStream_t s)
{
    switch (KW) {
    case 3: return go3<3>(g, block, vec, grid, wpb, s);
    case 5: return go3<5>(g, block, vec, grid, wpb, s);
    case 7: return go3<7>(g, block, vec, grid, wpb, s);
    case 9: return go3<9>(g, block, vec, grid, wpb, s);
    default: return hipErrorNotSupported;
    }
}

}  // namespace swc

// Instantiations of the register-resident 2-D kernel for MODE_F64.
#include "swc_corr2d_fast.hpp"
#include "swc_internal.h"

namespace swc {

// Launch (occ == nullptr) or report resident workgroups per CU (occ != nullptr).
template <int R, int KW, bool SHIFT>
static hipError_t go1(const P2DF& g, int grid, int wpb, size_t smem, hipStream_t s, int* occ)
{
    if (occ)
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(
            occ, corr2d_fast_kernel<MODE_F64, R, KW, SHIFT>, wpb * kWave, smem);
    return launch_kernel(&corr2d_fast_kernel<MODE_F64, R, KW, SHIFT>, dim3(grid), dim3(wpb * kWave), smem, s, g);
}

template <int R, int KW>
static hipError_t go(const P2DF& g, bool shifted, int grid, int wpb, size_t smem, hipStream_t s, int* occ)
{
    if (shifted) return hipErrorNotSupported;    // float rows are read at any word
    return go1<R, KW, false>(g, grid, wpb, smem, s, occ);
}

hipError_t launch_fast2d_modef64(const P2DF& g, int R, int KW, bool shifted, int grid, int wpb,
                                size_t smem, hipStream_t s, int* occ)
{
    if (R == 4) {
        switch (KW) {
        case 1: return go<4, 1>(g, shifted, grid, wpb, smem, s, occ);
        case 2: return go<4, 2>(g, shifted, grid, wpb, smem, s, occ);
        case 3: return go<4, 3>(g, shifted, grid, wpb, smem, s, occ);
        case 4: return go<4, 4>(g, shifted, grid, wpb, smem, s, occ);
        case kTall3: return go<4, kTall3>(g, shifted, grid, wpb, smem, s, occ);
        case 5: return go<4, 5>(g, shifted, grid, wpb, smem, s, occ);
        case 7: return go<4, 7>(g, shifted, grid, wpb, smem, s, occ);
        case 9: return go<4, 9>(g, shifted, grid, wpb, smem, s, occ);
        case 15: return go<4, 15>(g, shifted, grid, wpb, smem, s, occ);
        case 0: return go<4, 0>(g, shifted, grid, wpb, smem, s, occ);
        case kWideKw: return go<4, kWideKw>(g, shifted, grid, wpb, smem, s, occ);
        default: break;
        }
    } else if (R == 8) {
        switch (KW) {
        case 7: return go<8, 7>(g, shifted, grid, wpb, smem, s, occ);
        case 15: return go<8, 15>(g, shifted, grid, wpb, smem, s, occ);
        case 0: return go<8, 0>(g, shifted, grid, wpb, smem, s, occ);
        case kWideKw: return go<8, kWideKw>(g, shifted, grid, wpb, smem, s, occ);
        default: break;
        }
    }
    return hipErrorNotSupported;
}

}  // namespace swc

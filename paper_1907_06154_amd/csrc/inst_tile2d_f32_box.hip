// Small 2D grids, many sweeps a launch (ssam_kernel2d_tile.h): fp32, boxes of radius 1 to 2.
#include "ssam_kernel2d_tile.h"

namespace ssam {

template <>
const Tile2DKernel* tile2d_kernels<float, false>(int R)
{
    static const Tile2DKernel list[][4] = {
        {SSAM_TILE2D_K(float, 4, 1, 2), SSAM_TILE2D_K(float, 2, 1, 2), SSAM_TILE2D_K(float, 1, 1, 2), {}},
        {SSAM_TILE2D_K(float, 4, 2, 2), SSAM_TILE2D_K(float, 2, 2, 2), SSAM_TILE2D_K(float, 1, 2, 2), {}},
    };
    return R >= 1 && R <= 2 ? list[R - 1] : nullptr;
}

}  // namespace ssam

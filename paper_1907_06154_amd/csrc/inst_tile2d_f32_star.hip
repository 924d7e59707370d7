// Small 2D grids, many sweeps a launch (ssam_kernel2d_tile.h): fp32, stars of radius 1 to 6.
#include "ssam_kernel2d_tile.h"

namespace ssam {

template <>
const Tile2DKernel* tile2d_kernels<float, true>(int R)
{
    static const Tile2DKernel list[][4] = {
        {SSAM_TILE2D_K(float, 4, 1, 1), SSAM_TILE2D_K(float, 2, 1, 1), SSAM_TILE2D_K(float, 1, 1, 1), {}},
        {SSAM_TILE2D_K(float, 4, 2, 1), SSAM_TILE2D_K(float, 2, 2, 1), SSAM_TILE2D_K(float, 1, 2, 1), {}},
        {SSAM_TILE2D_K(float, 4, 3, 1), SSAM_TILE2D_K(float, 2, 3, 1), SSAM_TILE2D_K(float, 1, 3, 1), {}},
        {SSAM_TILE2D_K(float, 4, 4, 1), SSAM_TILE2D_K(float, 2, 4, 1), SSAM_TILE2D_K(float, 1, 4, 1), {}},
        {SSAM_TILE2D_K(float, 4, 5, 1), SSAM_TILE2D_K(float, 2, 5, 1), SSAM_TILE2D_K(float, 1, 5, 1), {}},
        {SSAM_TILE2D_K(float, 4, 6, 1), SSAM_TILE2D_K(float, 2, 6, 1), SSAM_TILE2D_K(float, 1, 6, 1), {}},
    };
    return R >= 1 && R <= 6 ? list[R - 1] : nullptr;
}

}  // namespace ssam

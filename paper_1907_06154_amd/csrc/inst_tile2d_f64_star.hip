// Small 2D grids, many sweeps a launch (ssam_kernel2d_tile.h): fp64, stars of radius 1 to 6.
#include "ssam_kernel2d_tile.h"

namespace ssam {

template <>
const Tile2DKernel* tile2d_kernels<double, true>(int R)
{
    static const Tile2DKernel list[][3] = {
        {SSAM_TILE2D_K(double, 2, 1, 1), SSAM_TILE2D_K(double, 1, 1, 1), {}},
        {SSAM_TILE2D_K(double, 2, 2, 1), SSAM_TILE2D_K(double, 1, 2, 1), {}},
        {SSAM_TILE2D_K(double, 2, 3, 1), SSAM_TILE2D_K(double, 1, 3, 1), {}},
        {SSAM_TILE2D_K(double, 2, 4, 1), SSAM_TILE2D_K(double, 1, 4, 1), {}},
        {SSAM_TILE2D_K(double, 2, 5, 1), SSAM_TILE2D_K(double, 1, 5, 1), {}},
        {SSAM_TILE2D_K(double, 2, 6, 1), SSAM_TILE2D_K(double, 1, 6, 1), {}},
    };
    return R >= 1 && R <= 6 ? list[R - 1] : nullptr;
}

}  // namespace ssam

// Small 2D grids, many sweeps a launch (ssam_kernel2d_tile.h): fp64, boxes of radius 1 to 4.
#include "ssam_kernel2d_tile.h"

namespace ssam {

template <>
const Tile2DKernel* tile2d_kernels<double, false>(int R)
{
    static const Tile2DKernel list[][3] = {
        {SSAM_TILE2D_K(double, 2, 1, 2), SSAM_TILE2D_K(double, 1, 1, 2), {}},
        {SSAM_TILE2D_K(double, 2, 2, 2), SSAM_TILE2D_K(double, 1, 2, 2), {}},
        {SSAM_TILE2D_K(double, 2, 3, 2), SSAM_TILE2D_K(double, 1, 3, 2), {}},
        {SSAM_TILE2D_K(double, 2, 4, 2), SSAM_TILE2D_K(double, 1, 4, 2), {}},
    };
    return R >= 1 && R <= 4 ? list[R - 1] : nullptr;
}

}  // namespace ssam

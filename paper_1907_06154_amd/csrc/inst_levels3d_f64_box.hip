// Several sweeps of a radius-1 3D stencil a launch (ssam_kernel3d_levels.h): fp64, 27-point box.
#include "ssam_kernel3d_levels.h"

namespace ssam {
SSAM_LEVELS_KERNELS(double, 3)
}  // namespace ssam

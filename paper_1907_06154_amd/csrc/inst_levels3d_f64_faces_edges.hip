// Several sweeps of a radius-1 3D stencil a launch (ssam_kernel3d_levels.h): fp64, 19-point faces and edges.
#include "ssam_kernel3d_levels.h"

namespace ssam {
SSAM_LEVELS_KERNELS(double, 2)
}  // namespace ssam

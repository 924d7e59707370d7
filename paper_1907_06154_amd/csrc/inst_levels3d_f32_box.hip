// Several sweeps of a radius-1 3D stencil a launch (ssam_kernel3d_levels.h): fp32, 27-point box.
#include "ssam_kernel3d_levels.h"

namespace ssam {
SSAM_LEVELS_KERNELS(float, 3)
}  // namespace ssam

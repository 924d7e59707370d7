// Instances of the dense fp32 3D filters on the bf16 matrix cores: 1 group of eight patch columns.
#include "ssam_kernel3d_split.h"

namespace ssam {
SSAM_SPLIT3D_KERNELS(1, false)
}  // namespace ssam

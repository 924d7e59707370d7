// Multi-sweep (temporally blocked) 2D stencil instances: inst_fused2d_f64_deep.hip
#include "ssam_kernel2d_fused.h"

SSAM_INSTANCE_2D_FUSED(double, SSAM_F64, 2, 4, 1, 1, 6, 2, 0);
SSAM_INSTANCE_2D_FUSED(double, SSAM_F64, 2, 4, 1, 2, 6, 2, 0);
// Memory-bound at this depth, and two rows a group leave a third wave room (us per sweep, six sweeps a launch and eight: 8192^2 zero
// 35.5 -> 28.8, clamp 37.2 -> 31.8; 3001x6007 11.4 -> 9.5 and 12.5 -> 11.8; with four rows a group clamp 36.2 on 8192^2).  Ten and
// twelve sweeps are slower (31.4 and 29.4; clamp 39), and so are two rows a group for the box (4096x8000 clamp 24.3 -> 26.0).
SSAM_INSTANCE_2D_FUSED(double, SSAM_F64, 2, 2, 1, 1, 8, 2, 0);
SSAM_INSTANCE_2D_FUSED(double, SSAM_F64, 2, 4, 1, 2, 8, 2, 0);

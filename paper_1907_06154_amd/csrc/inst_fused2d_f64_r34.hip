// Multi-sweep (temporally blocked) 2D stencil instances: inst_fused2d_f64_r34.hip
#include "ssam_kernel2d_fused.h"

SSAM_INSTANCE_2D_FUSED(double, SSAM_F64, 2, 4, 3, 1, 2, 2, 0);
SSAM_INSTANCE_2D_FUSED(double, SSAM_F64, 2, 4, 3, 1, 3, 2, 0);
// us per sweep, three sweeps a launch and four, zero padding: 1536x2048 7.1 and 7.6, 3000x3200 15.1 and 14.1, 8192^2 80.8 and 73.8;
// clamp: 4096x8000 44.0 and 48.5, 7001x8001 82.4 and 79.1, 8192^2 85.9 and 78.5 (of other rows that are a multiple of 32 up to a tenth
// more where three go in evenly, a sixth to a fourth less for four sweeps)
SSAM_INSTANCE_2D_FUSED_FROM(double, SSAM_F64, 2, 4, 3, 1, 4, 2, 0, 9, 50);
SSAM_INSTANCE_2D_FUSED(double, SSAM_F64, 2, 4, 4, 1, 2, 2, 0);
SSAM_INSTANCE_2D_FUSED(double, SSAM_F64, 2, 4, 4, 1, 3, 2, 0);

// Multi-sweep (temporally blocked) 2D stencil instances, stars of radius 5 and 6: inst_fused2d_r56.hip
#include "ssam_kernel2d_fused.h"

SSAM_INSTANCE_2D_FUSED(double, SSAM_F64, 2, 4, 5, 1, 2, 2, 0);
// us per sweep, two sweeps a launch and three, zero padding: 1536x2048 10.6 and 11.1, 3000x3200 23.1 and 21.6, 8192^2 123 and 110;
// clamp: 4096x8000 66.6 and 66.5, 7001x8001 122 and 111, 8192^2 125 and 115.  (Radius 6: 136 and 179.)
SSAM_INSTANCE_2D_FUSED_FROM(double, SSAM_F64, 2, 4, 5, 1, 3, 2, 0, 9, 50);
SSAM_INSTANCE_2D_FUSED(double, SSAM_F64, 2, 4, 6, 1, 2, 2, 0);
SSAM_INSTANCE_2D_FUSED(float, SSAM_F32, 4, 4, 5, 1, 2, 2, 0);
SSAM_INSTANCE_2D_FUSED(float, SSAM_F32, 4, 4, 6, 1, 2, 2, 0);

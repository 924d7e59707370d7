// Multi-sweep (temporally blocked) 2D stencil instances: inst_fused2d_f64_r2.hip
#include "ssam_kernel2d_fused.h"

SSAM_INSTANCE_2D_FUSED(double, SSAM_F64, 2, 4, 2, 1, 2, 2, 0);
SSAM_INSTANCE_2D_FUSED(double, SSAM_F64, 2, 4, 2, 1, 3, 2, 0);
SSAM_INSTANCE_2D_FUSED(double, SSAM_F64, 2, 4, 2, 1, 4, 2, 0);
// us per sweep, four sweeps a launch and six, zero padding: 1536x2048 4.9 and 5.5, 3000x3200 10.6 and 10.0, 4096x8000 28.9 and 27.6,
// 8192^2 56.2 and 51.9, 7001x8001 59.9 and 47.7; the clamp rule's edge tiles take longer at this depth (4096x8000 30.9 and 38.0)
SSAM_INSTANCE_2D_FUSED_FROM(double, SSAM_F64, 2, 4, 2, 1, 6, 2, 0, 9, 32767);
SSAM_INSTANCE_2D_FUSED(double, SSAM_F64, 2, 4, 2, 2, 2, 2, 0);
SSAM_INSTANCE_2D_FUSED(double, SSAM_F64, 2, 4, 2, 2, 3, 2, 0);
SSAM_INSTANCE_2D_FUSED(double, SSAM_F64, 2, 4, 2, 2, 4, 2, 0);

// hop_f32_r12.hip -- the hop kernels of hop.hip for one storage format: FP32 spinors, 12-real links.
#define WL_HOP_FORMAT P_F32, P_F32, 12
#include "hop.hip"

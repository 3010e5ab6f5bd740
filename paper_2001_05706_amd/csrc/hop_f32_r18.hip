// hop_f32_r18.hip -- the hop kernels of hop.hip for one storage format: FP32 spinors, 18-real links.
#define WL_HOP_FORMAT P_F32, P_F32, 18
#include "hop.hip"

// hop_f64_r12.hip -- the hop kernels of hop.hip for one storage format: FP64 spinors, 12-real links.
#define WL_HOP_FORMAT P_F64, P_F64, 12
#include "hop.hip"

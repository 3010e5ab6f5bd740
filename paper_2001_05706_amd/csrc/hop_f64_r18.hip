// hop_f64_r18.hip -- the hop kernels of hop.hip for one storage format: FP64 spinors, 18-real links.
#define WL_HOP_FORMAT P_F64, P_F64, 18
#include "hop.hip"

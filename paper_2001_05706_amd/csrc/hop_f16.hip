// hop_f16.hip -- the hop kernels of hop.hip for one storage format: FP16 storage, 12-real links.
#define WL_HOP_FORMAT P_F16, P_F16, 12
#include "hop.hip"

// hop_bf16.hip -- the hop kernels of hop.hip for one storage format: BF16 storage, 12-real links.
#define WL_HOP_FORMAT P_BF16, P_BF16, 12
#include "hop.hip"

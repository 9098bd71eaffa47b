// dg_rownorm_strided.hip -- the strided-lane kernels of dg_rownorm.hip, compiled beside the contiguous ones.
#define DG_ROWNORM_STRIDED
#include "dg_rownorm.hip"

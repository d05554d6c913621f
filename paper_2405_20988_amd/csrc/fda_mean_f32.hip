// Mean-state kernels: float slab.
#define FDA_TU_TYPE float
#define FDA_TU_BATCH fda::kMeanBatchF32
#define FDA_TU_NAME launch_mean_f32
#include "fda_mean.inc"

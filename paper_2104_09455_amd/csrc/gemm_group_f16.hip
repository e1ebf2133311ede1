// Launches of several independent products, f16 operands.
#define ABFT_DT abft::DT_F16
#define ABFT_GROUP_NAME launch_group_f16
#define ABFT_SHALLOW_NAME launch_shallow_f16
#include "gemm_group.inc"

// Launches of several independent products, i8 operands.
#define ABFT_DT abft::DT_I8
#define ABFT_GROUP_NAME launch_group_i8
#define ABFT_SHALLOW_NAME launch_shallow_i8
#include "gemm_group.inc"

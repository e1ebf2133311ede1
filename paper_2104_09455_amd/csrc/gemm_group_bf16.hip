// Launches of several independent products, bf16 operands.
#define ABFT_DT abft::DT_BF16
#define ABFT_GROUP_NAME launch_group_bf16
#define ABFT_SHALLOW_NAME launch_shallow_bf16
#include "gemm_group.inc"

// Products of at most sixteen rows, bf16 operands.
#define ABFT_DT abft::DT_BF16
#define ABFT_SKINNY_NAME launch_skinny_bf16
#define ABFT_SKINNY_GROUP_NAME launch_skinny_group_bf16
#include "gemm_skinny.inc"

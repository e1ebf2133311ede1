// Products of at most sixteen rows, f16 operands.
#define ABFT_DT abft::DT_F16
#define ABFT_SKINNY_NAME launch_skinny_f16
#define ABFT_SKINNY_GROUP_NAME launch_skinny_group_f16
#include "gemm_skinny.inc"

// Products of at most sixteen rows, i8 operands.
#define ABFT_DT abft::DT_I8
#define ABFT_SKINNY_NAME launch_skinny_i8
#define ABFT_SKINNY_GROUP_NAME launch_skinny_group_i8
#include "gemm_skinny.inc"

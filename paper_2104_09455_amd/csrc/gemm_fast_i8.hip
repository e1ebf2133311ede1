// Direct-to-LDS and row-streaming kernels, i8 operands.
#define ABFT_DT abft::DT_I8
#define ABFT_FAMILY 1
#define ABFT_LAUNCH_NAME launch_fast_i8
#include "gemm_launch.inc"

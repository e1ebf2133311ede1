// Generic kernels, f16 operands.
#define ABFT_DT abft::DT_F16
#define ABFT_FAMILY 3
#define ABFT_LAUNCH_NAME launch_generic_f16
#include "gemm_launch.inc"

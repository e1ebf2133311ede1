// Direct-to-LDS and row-streaming kernels, f16 operands.
#define ABFT_DT abft::DT_F16
#define ABFT_FAMILY 1
#define ABFT_LAUNCH_NAME launch_fast_f16
#include "gemm_launch.inc"

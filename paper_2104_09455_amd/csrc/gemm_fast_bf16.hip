// Direct-to-LDS and row-streaming kernels, bf16 operands.
#define ABFT_DT abft::DT_BF16
#define ABFT_FAMILY 1
#define ABFT_LAUNCH_NAME launch_fast_bf16
#include "gemm_launch.inc"

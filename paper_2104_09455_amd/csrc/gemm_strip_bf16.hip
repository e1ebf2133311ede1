// strip kernel for bf16 operands
#define ABFT_DT DT_BF16
#define ABFT_STRIP_NAME launch_strip_bf16
#include "gemm_strip.inc"

// strip kernel for f16 operands
#define ABFT_DT DT_F16
#define ABFT_STRIP_NAME launch_strip_f16
#include "gemm_strip.inc"

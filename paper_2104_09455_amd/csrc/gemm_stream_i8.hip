// Streaming kernels, i8 operands.
#define ABFT_DT abft::DT_I8
#define ABFT_FAMILY 2
#define ABFT_LAUNCH_NAME launch_stream_i8
#include "gemm_launch.inc"

// The pipelined plain products with BF16 operands (run_gemm_lds), a
// translation unit of their own: they take minutes to compile.
#define MDNN_PIPE_UNIT
#include "gemm_launch.h"

namespace mdnn {
MDNN_RUN_GEMM_LDS(, BF16)
}  // namespace mdnn

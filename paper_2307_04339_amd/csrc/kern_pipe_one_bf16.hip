// Kernel table of the register-tile pipelined contraction for bf16 operands, one tap
// (a translation unit of its own keeps the build parallel).
#include "gemm_pipe.h"

namespace miriam {
int pipe_kernels_one_bf16(int cfg, const void *out[3], int *lds) { return pipe_table_cfg<bf16_t, false>(cfg, out, lds); }
}  // namespace miriam

// Kernel table of the register-tile pipelined contraction for bf16 operands, right operand stored [k][n].
#include "gemm_pipe.h"

namespace miriam {
int pipe_kernels_nb_bf16(int cfg, const void *out[3], int *lds) { return pipe_nb_table_cfg<bf16_t>(cfg, out, lds); }
}  // namespace miriam

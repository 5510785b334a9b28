// Kernel table of the register-tile pipelined contraction for f16 operands, right operand stored [k][n].
#include "gemm_pipe.h"

namespace miriam {
int pipe_kernels_nb_f16(int cfg, const void *out[3], int *lds) { return pipe_nb_table_cfg<half_t>(cfg, out, lds); }
}  // namespace miriam

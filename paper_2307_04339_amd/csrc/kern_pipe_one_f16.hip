// Kernel table of the register-tile pipelined contraction for f16 operands, one tap
// (a translation unit of its own keeps the build parallel).
#include "gemm_pipe.h"

namespace miriam {
int pipe_kernels_one_f16(int cfg, const void *out[3], int *lds) { return pipe_table_cfg<half_t, false>(cfg, out, lds); }
}  // namespace miriam

// Kernel table of the register-tile pipelined contraction for f16 operands, filters of several taps
// (a translation unit of its own keeps the build parallel).
#include "gemm_pipe.h"

namespace miriam {
int pipe_kernels_taps_f16(int cfg, const void *out[3], int *lds) { return pipe_table_cfg<half_t, true>(cfg, out, lds); }
}  // namespace miriam

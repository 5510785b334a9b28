// Kernel tables of the 3x3 stride-1 patch convolution for f16 operands.
#include "conv_patch.h"

namespace miriam {
int patch_kernels_f16(int cfg, const void *out[3], int *lds) {
    return patch_table_cfg<half_t>(cfg, out, lds);
}
}  // namespace miriam

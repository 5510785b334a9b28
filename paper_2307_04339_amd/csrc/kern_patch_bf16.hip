// Kernel tables of the 3x3 stride-1 patch convolution for bf16 operands.
#include "conv_patch.h"

namespace miriam {
int patch_kernels_bf16(int cfg, const void *out[3], int *lds) {
    return patch_table_cfg<bf16_t>(cfg, out, lds);
}
}  // namespace miriam

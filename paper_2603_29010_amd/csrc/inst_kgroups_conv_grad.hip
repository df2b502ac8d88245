// conv2d_dgrad, gathered operands, two K groups.
#include "ucl_launch.h"

namespace ucl {
static const VariantDesc kTable[] = {
    describe<KernelCfg<64, 64, 64, 4, 0, 3, kIm2col, kNDirect, 0, 0, 2>>(),
    describe<KernelCfg<64, 64, 64, 4, 1, 3, kIm2col, kNDirect, 0, 0, 2>>(),
};
VariantList variants_kgroups_conv_grad() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }
}  // namespace ucl

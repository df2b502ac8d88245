// conv2d_fprop, per-tap gather, two K groups.
#include "ucl_launch.h"

namespace ucl {
static const VariantDesc kTable[] = {
    describe<KernelCfg<64, 64, 64, 4, 0, 2, kIm2col, kKContig, 0, 0, 2>>(),
    describe<KernelCfg<128, 64, 64, 3, 0, 2, kIm2col, kKContig, 0, 0, 2>>(),
    describe<KernelCfg<128, 128, 64, 2, 0, 2, kIm2col, kKContig, 0, 0, 2>>(),
    describe<KernelCfg<64, 64, 64, 4, 1, 2, kIm2col, kKContig, 0, 0, 2>>(),
    describe<KernelCfg<128, 64, 64, 3, 1, 2, kIm2col, kKContig, 0, 0, 2>>(),
    describe<KernelCfg<128, 128, 64, 2, 1, 2, kIm2col, kKContig, 0, 0, 2>>(),
};
VariantList variants_kgroups_conv() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }
}  // namespace ucl

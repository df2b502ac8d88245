// gemm / batched_gemm with operands contiguous along M / N, two K groups.
#include "ucl_launch.h"

namespace ucl {
static const VariantDesc kTable[] = {
    describe<KernelCfg<64, 64, 64, 4, 0, 0, kKContig, kNDirect, 0, 0, 2>>(),
    describe<KernelCfg<64, 64, 64, 4, 1, 0, kKContig, kNDirect, 0, 0, 2>>(),
    describe<KernelCfg<64, 64, 64, 4, 0, 0, kMDirect, kNDirect, 0, 0, 2>>(),
    describe<KernelCfg<128, 128, 32, 4, 0, 0, kMDirect, kNDirect, 0, 0, 2>>(),
    describe<KernelCfg<64, 64, 64, 4, 1, 0, kMDirect, kNDirect, 0, 0, 2>>(),
    describe<KernelCfg<128, 128, 32, 4, 1, 0, kMDirect, kNDirect, 0, 0, 2>>(),
};
VariantList variants_kgroups_mn() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }
}  // namespace ucl

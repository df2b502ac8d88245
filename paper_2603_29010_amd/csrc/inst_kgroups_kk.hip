// gemm / batched_gemm, both operands contiguous along K, two K groups (problems of fewer tiles than CU slots).
#include "ucl_launch.h"

namespace ucl {
static const VariantDesc kTable[] = {
    describe<KernelCfg<64, 64, 64, 4, 0, 0, kKContig, kKContig, 0, 0, 2>>(),
    describe<KernelCfg<64, 64, 64, 4, 1, 0, kKContig, kKContig, 0, 0, 2>>(),
    describe<KernelCfg<64, 64, 64, 4, 2, 0, kKContig, kKContig, 0, 0, 2>>(),
    describe<KernelCfg<64, 64, 64, 4, 3, 0, kKContig, kKContig, 0, 0, 2>>(),
};
VariantList variants_kgroups_kk() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }
}  // namespace ucl

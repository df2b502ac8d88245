// gemm / batched_gemm / grouped_gemm of few rows.
#include "ucl_skinny.h"

namespace ucl {
static const VariantDesc kTable[] = {
    describe_skinny<SkinnyCfg<1, 1, 8, 4, 0, 0>>(),
    describe_skinny<SkinnyCfg<1, 2, 8, 4, 0, 0>>(),
    describe_skinny<SkinnyCfg<1, 4, 4, 4, 0, 0>>(),
    describe_skinny<SkinnyCfg<2, 1, 8, 4, 0, 0>>(),
    describe_skinny<SkinnyCfg<2, 2, 8, 4, 0, 0>>(),
    describe_skinny<SkinnyCfg<4, 1, 8, 4, 0, 0>>(),
    describe_skinny<SkinnyCfg<4, 2, 4, 4, 0, 0>>(),
    describe_skinny<SkinnyCfg<1, 1, 8, 4, 2, 0>>(),
    describe_skinny<SkinnyCfg<2, 2, 4, 4, 2, 0>>(),
    describe_skinny<SkinnyCfg<1, 4, 4, 2, 2, 1>>(),
    describe_skinny<SkinnyCfg<2, 1, 4, 4, 2, 1>>(),
    describe_skinny<SkinnyCfg<2, 2, 4, 4, 2, 1>>(),
    describe_skinny<SkinnyCfg<2, 4, 4, 2, 2, 1>>(),
    describe_skinny<SkinnyCfg<2, 2, 8, 4, 2, 1>>(),
};
VariantList variants_skinny() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }
}  // namespace ucl

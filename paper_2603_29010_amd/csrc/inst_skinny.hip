// gemm / batched_gemm / grouped_gemm and small forward convolutions: problems of few rows or few tiles.
#include "ucl_skinny.h"

namespace ucl {
static const VariantDesc kTable[] = {
    describe_skinny_pair<1, 1, 4, 0, 0>(),
    describe_skinny_pair<1, 2, 4, 0, 0>(),
    describe_skinny_pair<2, 2, 4, 0, 0>(),
    describe_skinny_pair<2, 4, 3, 0, 0>(),
    describe_skinny_pair<1, 1, 4, 1, 0>(),
    describe_skinny_pair<1, 2, 4, 1, 0>(),
    describe_skinny_pair<2, 2, 4, 1, 0>(),
    describe_skinny_pair<2, 4, 3, 1, 0>(),
    describe_skinny_pair<1, 1, 4, 2, 0>(),
    describe_skinny_pair<1, 2, 4, 2, 0>(),
    describe_skinny_pair<2, 2, 4, 2, 0>(),
    describe_skinny_pair<2, 4, 3, 2, 0>(),
    describe_skinny_pair<1, 1, 4, 3, 0>(),
    describe_skinny_pair<1, 2, 4, 3, 0>(),
    describe_skinny_pair<2, 2, 4, 3, 0>(),
    describe_skinny_pair<2, 4, 3, 3, 0>(),
    describe_skinny<SkinnyCfg<4, 4, 8, 1, 0, 0>>(),
    describe_skinny<SkinnyCfg<4, 4, 8, 1, 1, 0>>(),
    describe_skinny<SkinnyCfg<2, 2, 4, 2, 0, 1>>(),
    describe_one_buffer<SkinnyCfg<2, 2, 4, 1, 0, 1>>(),
    describe_one_buffer<SkinnyCfg<2, 4, 4, 1, 0, 1>>(),
    describe_skinny<SkinnyCfg<2, 2, 4, 2, 1, 1>>(),
    describe_one_buffer<SkinnyCfg<2, 2, 4, 1, 1, 1>>(),
    describe_one_buffer<SkinnyCfg<2, 4, 4, 1, 1, 1>>(),
    describe_skinny<SkinnyCfg<2, 2, 4, 2, 2, 1>>(),
    describe_one_buffer<SkinnyCfg<2, 2, 4, 1, 2, 1>>(),
    describe_one_buffer<SkinnyCfg<2, 4, 4, 1, 2, 1>>(),
    describe_skinny<SkinnyCfg<2, 2, 4, 2, 3, 1>>(),
    describe_one_buffer<SkinnyCfg<2, 2, 4, 1, 3, 1>>(),
    describe_one_buffer<SkinnyCfg<2, 4, 4, 1, 3, 1>>(),
    describe_skinny<SkinnyCfg<1, 2, 4, 4, 0, 2>>(),
    describe_skinny<SkinnyCfg<1, 2, 4, 4, 1, 2>>(),
};
VariantList variants_skinny() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }
}  // namespace ucl

// conv2d_wgrad of 3x3 filters, all taps of a pixel in one workgroup.
#include "ucl_wgrad_taps.h"

namespace ucl {
static const VariantDesc kTable[] = {
    VariantDesc{64, 288, 128, 4, 0, 4, 5, 4, kLdsBytesPerCU, 0, 1, 2, 0, &launch_wgrad_taps<0>, nullptr},
    VariantDesc{64, 288, 128, 4, 1, 4, 5, 4, kLdsBytesPerCU, 0, 1, 2, 0, &launch_wgrad_taps<1>, nullptr},
};
VariantList variants_wgrad_taps() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }
}  // namespace ucl

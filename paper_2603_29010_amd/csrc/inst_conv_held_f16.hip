// 3x3 convolutions and data gradients with the filter in registers, f16.
#include "ucl_conv_held.h"

namespace ucl {
static hipError_t launch_held(int mode, const HeldPlan &h, const KParams &p, hipStream_t stream) {
    if (mode == 3) return p.fused.has_res ? launch_conv_held_mode<1, 3, true>(h, p, stream) : launch_conv_held_mode<1, 3, false>(h, p, stream);
    if (h.stride == 2) return p.fused.has_res ? launch_conv_held_mode<1, 2, true, 2>(h, p, stream) : launch_conv_held_mode<1, 2, false, 2>(h, p, stream);
    return p.fused.has_res ? launch_conv_held_mode<1, 2, true>(h, p, stream) : launch_conv_held_mode<1, 2, false>(h, p, stream);
}
static const VariantDesc kTable[] = {
    VariantDesc{0, 0, 64, 1, 1, 2, 3, 0, kLdsBytesPerCU, 0, 1, 1, 0, nullptr, nullptr, &launch_held},
};
VariantList variants_conv_held_f16() { return {kTable, (int)(sizeof(kTable) / sizeof(kTable[0]))}; }
}  // namespace ucl

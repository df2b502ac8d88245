// Registry of the built kernel variants: every instantiation unit contributes a table of these.
#pragma once
#include "ucl_device.h"

namespace ucl {

// 3x3 convolutions with the filter in registers (conv_held_kernel): how a launch is cut up.  Not among the variants that a tile names.
struct HeldPlan {
    int stride = 1;
    int kg = 0, ng = 0;            // wave groups over channels (64 each) and filters (32 each) of a workgroup; 0: not served
    int R = 0;                     // padded output rows per workgroup
    int strip_split = 1;           // of the waves that kg and ng leave, as many share out strips, the others rows
    int pair = 1, pitch = 0, strips = 0, rows = 0, bands = 0, tiles_n = 0, passes = 1, keep_bytes = 0;
    double seconds = 0;
};
constexpr int kHeldMaxKG = 4;
// LDS of a workgroup: one tap of its filters (KG x NG x 4 KB), several on their way; where KG > 1 its waves' sums of four output rows meet in their
// place; 1 KB for the bias.  The rest is its pixels' (0: wave groups that no kernel is built for).
constexpr int held_slots(int kg, int ng) { return kg * ng == 8 ? 3 : kg * ng == 4 ? 4 : 9; }
constexpr int held_filter_bytes(int kg, int ng) {
    const int filter = held_slots(kg, ng) * kg * ng * 4096, meet = kg == 1 ? 0 : 4 * 8 * 2048;
    return filter > meet ? filter : meet;
}
constexpr int held_patch_capacity(int kg, int ng) {
    return kg * ng <= 8 && (kg == 2 || ng == 2 || kg * ng == 4) ? kLdsBytesPerCU - held_filter_bytes(kg, ng) - 1024 : 0;
}
// ... which are, for R output rows at a pitch: the image rows their taps reach and eight zeros behind them, per plane of 64 channels
constexpr int64_t held_plane_bytes(int64_t stride, int64_t R, int64_t pitch) { return ((stride * R + 3 - stride) * stride * pitch + 8) * 128; }
// Rows of one of `groups` waves that share R: in pairs, and a last single one where the registers hold its own body
constexpr int held_rows_of_wave(int R, int groups, int kg, bool multi) {
    const int rows = (R + groups - 1) / groups;
    return kg == 1 || multi ? (rows + 1) & ~1 : rows;
}

struct VariantDesc {
    int tile_m, tile_n, tile_k, stages;
    int dt;             // inputs: 0 bf16, 1 fp16, 2 fp8 e4m3, 3 fp8 e5m2 (8-bit inputs are handled as pairs: K, strides in 16-bit units)
    int mode;           // 0 gemm / batched, 1 grouped, 2 conv2d fprop, 3 conv2d dgrad, 4 conv2d wgrad
    int la, lb;         // 0: operand contiguous along K, 1: contiguous along M / N (register transpose); A only: 2 im2col gather,
                        // 3 resident patch; 4 (B) / 5 (A): contiguous along N / M, copied directly and read through the LDS transpose read
    int lds_bytes;
    int persistent;     // tile scheduler the kernel is built for: 0 one workgroup per tile, 1 persistent (grid = CU slots, workgroups
                        // walk the tile order), 2 stream-K (grid = CU slots, workgroups take equal runs of (tile, k range) iterations)
    int wgs_per_cu;     // workgroups of the kernel a CU is meant to hold (register budget it was built with)
    int k_groups;       // wave groups of a workgroup that share a tile, each taking a part of K (1: none)
    int patch_c;        // resident-patch kernels: channels per pixel of the tensor the patch holds (64 or 128), else 0
    hipError_t (*launch)(const KParams &p, const GroupTable *gt, int grid, hipStream_t stream);
    int (*resident)();          // workgroups one CU holds at a time (queried from the runtime)
    hipError_t (*launch_held)(int mode, const HeldPlan &h, const KParams &p, hipStream_t stream);      // variants_conv_held_* only
};

// Few-row kernels of four waves: with more tiles than this, one per CU, those with one stage buffer per wave serve (gemm and batched calls: the
// launch takes them, up to kOneBufferMaxK; grouped calls: variants of their own).
constexpr int kOneBufferAbove = 256, kOneBufferMaxK = 4096;
inline bool takes_one_buffer(int64_t tiles, int64_t K) { return tiles > kOneBufferAbove && K <= kOneBufferMaxK; }

// (few-row kernels: stages 1, and 4 for those with one buffer for each of their waves)
inline bool is_few_row(const VariantDesc &v) { return v.stages == 1 || v.tile_m < 64; }

struct VariantList {
    const VariantDesc *v;
    int n;
};

// one per instantiation unit
VariantList variants_gemm_kk_bf16_a();
VariantList variants_gemm_kk_bf16_b();
VariantList variants_gemm_kk_bf16_c();
VariantList variants_gemm_kk_bf16_d();
VariantList variants_gemm_kk_f16_a();
VariantList variants_gemm_kk_f16_b();
VariantList variants_gemm_mn_bf16();
VariantList variants_gemm_mn_f16();
VariantList variants_grouped_a();
VariantList variants_grouped_b();
VariantList variants_conv_a();
VariantList variants_conv_b();
VariantList variants_conv_f16();
VariantList variants_conv_halo();
VariantList variants_gemm_kn_bf16();
VariantList variants_gemm_kn_f16();
VariantList variants_gemm_mx_bf16();
VariantList variants_gemm_mx_f16();
VariantList variants_grouped_kn();
VariantList variants_persistent();
VariantList variants_streamk();
VariantList variants_grouped_fp8_e4m3();
VariantList variants_grouped_fp8_e5m2();
VariantList variants_gemm_kk_fp8();
VariantList variants_conv_dgrad();
VariantList variants_conv_dgrad_halo();
VariantList variants_conv_wgrad();
VariantList variants_skinny();
VariantList variants_kgroups_kk();
VariantList variants_kgroups_mn();
VariantList variants_kgroups_conv();
VariantList variants_kgroups_conv_grad();

// conv2d_wgrad with all taps of a pixel in one workgroup, by input type (not among the variants that a tile names; split_k and k_per_slice of
// its arguments are slices and padded pixels per slice)
VariantList variants_wgrad_taps();

// 3x3 convolutions and data gradients with the filter in registers, by input type (chosen only, by their launch_held)
VariantList variants_conv_held_bf16();
VariantList variants_conv_held_f16();

}  // namespace ucl

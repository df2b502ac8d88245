// Host side of the C ABI declared in include/ucl.h: argument validation with explanatory
// errors, the per-problem tile / stage selection table, the launch, and the SOL analysis.
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <vector>

#include <mutex>

#include "ucl_kernel.h"      // the epilogue's element-wise arithmetic (the split-K reduction kernel finishes simple chains itself)
#include "ucl_variants.h"
#include "ucl_costs.h"

// Split-K workspace of ucl_gemm_static_workspace: counters followed by partial tiles, held by every
// GPU the library runs on until the process ends.  Host code never uses this name as an address: it
// asks the runtime for the array's device address once per device (static_workspace() below).
static __device__ __align__(256) unsigned char scratch[UCL_STATIC_WORKSPACE_BYTES];

namespace ucl {
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
// the transform stage lives in its own unit
ucl_status transpose_run(int64_t batch, int64_t rows, int64_t cols, const void *src, int32_t dt_src, void *dst, int32_t dt_dst,
                         void *stream);
const char *transpose_last_error();

namespace {

thread_local char g_err[512] = "";

ucl_status fail(ucl_status st, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return st;
}

const std::vector<VariantDesc> &all_variants() {
    static const std::vector<VariantDesc> v = [] {
        std::vector<VariantDesc> out;
        for (VariantList l : {variants_gemm_kk_bf16_a(), variants_gemm_kk_bf16_b(), variants_gemm_kk_bf16_c(), variants_gemm_kk_bf16_d(), variants_gemm_kk_f16_a(), variants_gemm_kk_f16_b(), variants_gemm_mn_bf16(), variants_gemm_mn_f16(), variants_grouped_a(), variants_grouped_b(), variants_conv_a(), variants_conv_b(), variants_conv_f16(), variants_conv_halo(), variants_gemm_kn_bf16(), variants_gemm_kn_f16(), variants_gemm_mx_bf16(), variants_gemm_mx_f16(), variants_grouped_kn(), variants_conv_dgrad(), variants_conv_dgrad_halo(), variants_conv_wgrad(), variants_gemm_kk_fp8(), variants_persistent(), variants_grouped_fp8_e4m3(), variants_grouped_fp8_e5m2(), variants_streamk(), variants_kgroups_kk(), variants_kgroups_mn(), variants_kgroups_conv(), variants_kgroups_conv_grad(), variants_skinny()})
            for (int i = 0; i < l.n; ++i) out.push_back(l.v[i]);
        return out;
    }();
    return v;
}

// The cost row of every variant, in the same order (kernels of another tile scheduler take the row of their tile).  Kernels
// without one -- those that transpose operands in registers, for matrices beyond the reach of 32-bit offsets -- are priced
// by the tile alone, far above the others.
const std::vector<CostRow> &all_costs() {
    static const std::vector<CostRow> c = [] {
        std::vector<CostRow> out;
        for (const VariantDesc &v : all_variants()) {
            const float slow = (int64_t)v.tile_m * v.tile_n >= 128 * 128 ? 20.f : 14.f;
            CostRow row = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 2, 8.f, 4.f, slow, 2.f, 1.5f, 1.f, 0.f, 1.f};
            for (const CostRow &r : kCostRows)
                if (r.mode == v.mode && r.la == v.la && r.lb == v.lb && r.eight_bit == (v.dt >= 2) && r.tile_m == v.tile_m && r.tile_n == v.tile_n &&
                    r.tile_k == v.tile_k && r.stages == v.stages && r.k_groups == v.k_groups && r.patch_c == (v.la == 3 ? v.patch_c : 0))
                    row = r;
            out.push_back(row);
        }
        return out;
    }();
    return c;
}

// The rows of the few-row kernels for more tiles than CUs, in the same order (one_buffer() says which have one).
const std::vector<CostRow> &many_tiles_costs() {
    static const std::vector<CostRow> c = [] {
        std::vector<CostRow> out;
        for (const VariantDesc &v : all_variants()) {
            CostRow row = {};
            for (const CostRow &r : kManyTilesRows)
                if (r.mode == v.mode && r.la == v.la && r.lb == v.lb && r.eight_bit == (v.dt >= 2) && r.tile_m == v.tile_m && r.tile_n == v.tile_n &&
                    v.stages == 1 && r.k_groups == v.k_groups)
                    row = r;
            out.push_back(row);
        }
        return out;
    }();
    return c;
}

// Where the variants of one operation and input type stand in all_variants(): every call walks these 4 to 49 instead of all.
const std::vector<int> &variants_of(int mode, int dt) {
    static const std::vector<std::vector<int>> lists = [] {
        std::vector<std::vector<int>> out(5 * 4);
        for (size_t i = 0; i < all_variants().size(); ++i) out[all_variants()[i].mode * 4 + all_variants()[i].dt].push_back((int)i);
        return out;
    }();
    return lists[mode * 4 + dt];
}

bool is8(int dt) { return dt == UCL_FP8_E4M3 || dt == UCL_FP8_E5M2; }
int elem_size(int dt) { return dt == UCL_F32 ? 4 : is8(dt) ? 1 : 2; }
bool is16(int dt) { return dt == UCL_F16 || dt == UCL_BF16; }
bool valid_dtype(int dt) { return dt == UCL_F32 || dt == UCL_F16 || dt == UCL_BF16; }     // outputs and epilogue tensors
const char *dtype_name(int dt) {
    return dt == UCL_F32 ? "fp32" : dt == UCL_F16 ? "fp16" : dt == UCL_BF16 ? "bf16" : dt == UCL_FP8_E4M3 ? "fp8_e4m3"
           : dt == UCL_FP8_E5M2 ? "fp8_e5m2" : "?";
}
// input type code of the kernel variants
int dt_code(int dt) { return dt == UCL_F16 ? 1 : dt == UCL_FP8_E4M3 ? 2 : dt == UCL_FP8_E5M2 ? 3 : 0; }
bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

bool op_has_tensor(int op) {
    switch (op) {
    case UCL_EPI_BIAS: case UCL_EPI_AUX_LOAD: case UCL_EPI_PER_ROW_SCALE: case UCL_EPI_PER_COL_SCALE:
    case UCL_EPI_ROW_BROADCAST: case UCL_EPI_COL_BROADCAST: case UCL_EPI_AUX_STORE:
        return true;
    default:
        return false;
    }
}
bool op_is_matrix(int op) { return op == UCL_EPI_AUX_LOAD || op == UCL_EPI_AUX_STORE; }

// ---- generic description of one launch, filled by the four entry points -------------------------
struct Launch {
    int mode = 0;                 // 0 gemm / batched, 1 grouped, 2 conv fprop, 3 conv dgrad, 4 conv wgrad
    int64_t batch = 1, M = 0, N = 0, K = 0;
    int la = 0, lb = 0;           // operand layouts
    int64_t lda = 0, ldb = 0;     // leading strides (0 where only sizes are known)
    int dt = 0;                   // input type code of the kernels: 0 bf16, 1 fp16, 2 fp8 e4m3, 3 fp8 e5m2
    int dtD = 0;
    int groups = 0;
    const int64_t *M_g = nullptr;
    int64_t sum_Mg = 0;
    int patch_c = 0;              // conv: the problem fits the resident-patch kernels built for pixels of this many channels (0: none)
    bool f32_results = false;     // the output or a stored epilogue tensor is fp32: the sums' rounding shows in it
    int64_t cN = 0, cH = 0, cW = 0, str_h = 1, str_w = 1;    // conv dgrad: images, extents of the activations, strides
    int taps_stride = 0;          // conv wgrad: stride of a problem that wgrad_taps_kernel serves (0: it does not)
    int64_t cP = 0, cQ = 0, cC = 0;
    int held_stride = 0;          // conv fprop / dgrad: stride of a problem that conv_held_kernel serves (cN, cP, cQ, cC set; 0: it does not)
    int64_t gathered = 0;         // ... and bytes of the pixels it gathers
    bool ndirect_ok = false;      // B contiguous along N and small enough for 32-bit byte offsets: direct-copy kernels apply
    bool mdirect_ok = false;      // the same for A contiguous along M
};

// The resident-patch conv kernels hold pixels of 64 or 128 channels and address the taps of a 3x3 filter at unit
// stride / dilation with one pad pixel, the image row (plus one pixel) on either side of a tile in LDS.  fprop: the
// pixels are those of the activations (C channels); data gradient: those of the output gradient (Kout channels;
// P = H and Q = W follow from the geometry), taps mirrored.  Returns the channel count, 0 if the kernels do not apply.
int conv_patch_channels(int64_t W, int64_t channels, int64_t R, int64_t S, int64_t pad_h, int64_t pad_w, int64_t str_h,
                        int64_t str_w, int64_t dil_h, int64_t dil_w) {
    const bool ok = (channels == 64 || channels == 128) && R == 3 && S == 3 && pad_h == 1 && pad_w == 1 && str_h == 1 &&
                    str_w == 1 && dil_h == 1 && dil_w == 1 && W + 1 <= 59;
    return ok ? (int)channels : 0;
}

// Filter gradients that wgrad_taps_kernel serves: 3x3 filters at pad 1, unit dilation and a stride of 1 or 2 whose rows are narrow enough for
// the ring of its x pixels (four k-tiles, of which the taps may reach over one) and which have fewer than 2^20 rows: the kernel finds the row of a
// slot's first pixel by an fp32 product, exact for twice as many (its relative error of 2^-22.5 over up to 2 (P + 1) + 64 rows has to stay below half a
// row in P + 1; 4210560 rows come out one off).  (Up to 32 filters, half of a workgroup's, the choice and the workspace of the tile kernel stay.)
void taps_launch(Launch &L, int64_t N, int64_t H, int64_t W, int64_t C, int64_t P, int64_t Q, int64_t R, int64_t S, int64_t pad_h, int64_t pad_w,
                 int64_t str_h, int64_t str_w, int64_t dil_h, int64_t dil_w) {
    L.cN = N; L.cH = H; L.cW = W; L.cP = P; L.cQ = Q; L.cC = C;
    const bool ok = R == 3 && S == 3 && pad_h == 1 && pad_w == 1 && str_h == str_w && (str_h == 1 || str_h == 2) && dil_h == 1 && dil_w == 1 &&
                    Q <= 62 && P < (1 << 20) && L.M > 32 && L.dt < variants_wgrad_taps().n && N * (P + 1) * (Q + 1) < (1ll << 30) && N * P * Q * L.M * 2 < (1ll << 30) && N * H * W * C * 2 < (1ll << 30);
    L.taps_stride = ok ? (int)str_h : 0;
}

// Convolutions that conv_held_kernel serves: 3x3 with pad 1 and unit dilation, as a forward pass at stride 1 or 2 and up to the channels of one pass (further
// ones gain nothing there: 0.7 of the tile kernels' speed), as a data gradient at stride 1 and of any channels.  n images of P x Q output pixels, C channels to multiply, L.N to write; the limits are
// those of 32-bit offsets and of divisions by reciprocals.
void held_launch(Launch &L, int64_t n_img, int64_t H, int64_t W, int64_t P, int64_t Q, int64_t C, int64_t R, int64_t S, int64_t pad_h, int64_t pad_w, int64_t str_h,
                 int64_t str_w, int64_t dil_h, int64_t dil_w) {
    L.cN = n_img; L.cP = P; L.cQ = Q; L.cC = C;
    // (rows whose offsets a launch works out: also those of a missing partner of the last image of up to seven columns, and those that the last band and its
    // waves have beyond the images, fewer than 64 padded ones.  With 2 GiB or more of them the offset of a row and the one that keeps a lane from
    // storing could add up to an address inside the result.)
    const int64_t named_rows = (n_img + (Q <= 7)) * P + 128;
    const bool ok = R == 3 && S == 3 && pad_h == 1 && pad_w == 1 && str_h == str_w && (str_h == 1 || (str_h == 2 && L.mode == 2)) && dil_h == 1 && dil_w == 1 && L.dt < 2 &&
                    (L.dt == 0 ? variants_conv_held_bf16() : variants_conv_held_f16()).n > 0 &&
                    (L.mode == 3 || C <= 64 * kHeldMaxKG) && L.N % 8 == 0 && Q <= 1024 && P < (1 << 20) && n_img * (P + 1) * ((L.N + 31) / 32) < (1ll << 20) &&
                    named_rows * Q * L.N < (1ll << 30) && n_img * H * W * C < (1ll << 30) && C * 9 * L.N < (1ll << 30);
    L.held_stride = ok ? (int)str_h : 0;
    L.gathered = n_img * H * W * C * 2;
}

// Per-problem selection: of the variants built for this (mode, input type, operand layouts) the one with the smallest
// estimated launch time (estimate_seconds, constants in ucl_costs.h).
int64_t count_tiles(const Launch &L, int tm, int tn) {
    const int64_t tiles_n = (L.N + tn - 1) / tn;
    if (L.mode == 1) {
        int64_t t = 0;
        for (int g = 0; g < L.groups; ++g) t += (L.M_g[g] + tm - 1) / tm * tiles_n;
        return t;
    }
    // (stride 1: the same as the general form)
    if (L.mode == 3) return dgrad_tile_rows(L.cN, L.cH, L.cW, L.str_h, L.str_w, tm) * tiles_n;
    return L.batch * ((L.M + tm - 1) / tm) * tiles_n;
}

// Launch description of a data gradient: extents for the tile count, and the mean depth over the residue classes of a
// strided convolution (every tap meets one class in stride_h * stride_w).  Extents, pads and dilated filters are below 2^24: every
// stride from kWidestStride on has one output row and pairs it with the same pixels, so wider ones (the kernels count in
// 32 bits) are taken as that.
constexpr int64_t kWidestStride = 1ll << 26;
void dgrad_launch(Launch &L, int64_t N, int64_t H, int64_t W, int64_t stride_h, int64_t stride_w) {
    if (stride_h > kWidestStride) stride_h = kWidestStride;
    if (stride_w > kWidestStride) stride_w = kWidestStride;
    L.cN = N; L.cH = H; L.cW = W; L.str_h = stride_h; L.str_w = stride_w;
    if (stride_h * stride_w > 1) L.K = (L.K + stride_h * stride_w - 1) / (stride_h * stride_w);
}

// The wide epilogue path addresses a wave's row panel (up to 128 rows) with 32-bit byte offsets.
constexpr int64_t kMaxWideLd = 1ll << 21;

// Workgroups of a variant that fit on one CU: 512 registers per lane and SIMD (the kernels are built
// with a budget by tile area), 160 KB of LDS.
int workgroups_per_cu(const VariantDesc &v) {
    const int64_t area = (int64_t)v.tile_m * v.tile_n;
    const int by_regs = area >= 256 * 256 ? 1 : area >= 256 * 128 ? 2 : area >= 128 * 128 ? 3 : 4;
    const int by_lds = v.lds_bytes > 0 ? kLdsBytesPerCU / v.lds_bytes : 8;
    return by_regs < by_lds ? by_regs : by_lds;
}

// Launch time of a variant:  fixed + round * rounds + loop (+) output, where
//   rounds = turns of resident workgroups the tiles make over the chip,
//   loop   = what bounds it: the bytes the busiest CU copies, its multiplications, the chain of a workgroup's k-tiles, or
//            the operands' trip from memory (5.3 TB/s), added as fourth powers (the largest, somewhat more where two are close),
//   output = the output's bytes, part of it hidden under the loop in the same sense.
double fourth_power_sum(double a, double b, double c = 0, double d = 0) {
    a *= a; b *= b; c *= c; d *= d;
    return sqrt(sqrt(a * a + b * b + c * c + d * d));
}
// Few-row kernels with one stage buffer per wave: gemm and batched launches take them under the named tile's tuple, with a cost row of its own
// (kManyTilesRows); grouped ones are variants of their own.  Their workgroups are short and follow one another on a CU without rounds.
bool one_buffer(const VariantDesc &v, const Launch &L, int64_t tiles) {
    if (L.mode == 1) return is_few_row(v) && v.stages != 1;
    return L.mode == 0 && v.stages == 1 && v.k_groups == 4 && takes_one_buffer(tiles, L.K);
}
// (row, many: the variant's rows of all_costs() and many_tiles_costs(); *one: whether it runs with one stage buffer per wave)
double estimate_seconds(const VariantDesc &v, const CostRow &row, const CostRow &many, const Launch &L, bool *one) {
    const int64_t tiles_n = (L.N + v.tile_n - 1) / v.tile_n;
    const int64_t tiles = count_tiles(L, v.tile_m, v.tile_n);
    *one = one_buffer(v, L, tiles);
    const CostRow &r = L.mode == 0 && *one ? many : row;
    const int64_t slots = 256 * (int64_t)r.resident, rounds = (tiles + slots - 1) / slots;
    const double on_cu = tiles <= slots || *one ? (double)((tiles + 255) / 256) : (double)(rounds * r.resident);
    // (8-bit inputs: K counts pairs of elements, 2 bytes)
    double rows = (double)L.M, all_rows = (double)L.batch * L.M, panels = (double)L.batch;
    if (L.mode == 1) {
        rows = tiles > 0 ? (double)L.sum_Mg * tiles_n / tiles : 0;             // mean rows of a tile
        all_rows = (double)L.sum_Mg;
        panels = L.groups;
    }
    const double tile_rows = (rows < v.tile_m ? rows : v.tile_m) + (double)(L.N < v.tile_n ? L.N : v.tile_n);
    const double K = (double)L.K;
    const double copies = on_cu * tile_rows * K * 2.0 / (r.gbs * 1e3);
    const double math = on_cu * 2.0 * v.tile_m * v.tile_n * K / (r.tflops * 1e6);
    const int64_t step_k = (v.stages == 1 ? 64 : v.tile_k) * (int64_t)v.k_groups;
    const double chain = (double)rounds * (double)((L.K + step_k - 1) / step_k) * r.step;
    const double memory = (all_rows + panels * L.N) * K * 2.0 / 5.3e6;
    const double loop = fourth_power_sum(copies, math, chain, memory);
    const double out = all_rows * L.N * (L.dtD == UCL_F32 ? 4.0 : 2.0) / 4.6e6 * r.out;
    return 1e-6 * r.factor * (r.fixed + r.round * (double)rounds + fourth_power_sum(loop, out * r.hidden) + out * (1.0 - r.hidden));
}

constexpr int kNumCUs = 256;

// Slices a split-K launch of `total_tiles` tiles gets: as asked for, or (0) enough to give every CU a workgroup
// while each keeps at least 4 x 64 of K; slices are whole multiples of 64 along K.
// The weight gradient in parallel mode gets two workgroups per CU where the variant fits twice: its gathered operand
// leaves a lone workgroup waiting (measured 36.7 -> 32.6 us on 32x56x56x64 -> 128), and the streaming reduction
// kernel takes the extra partial tiles in its stride; the GEMMs measured best with one (256x256x16384: 15.0 us with
// 16 slices, 16.9 with 32).
int split_fill(const Launch &L, const VariantDesc &v, const ucl_tuning *tune) {
    return L.mode == 4 && tune->split_k_mode == UCL_SPLIT_K_PARALLEL && workgroups_per_cu(v) >= 2 ? 2 * kNumCUs : kNumCUs;
}
void split_slices(const Launch &L, int64_t want, int64_t total_tiles, int fill, int &slices, int &k_per_slice) {
    const int64_t kt = (L.K + 63) / 64;
    if (want == 0) {
        want = total_tiles >= fill ? 1 : (fill + total_tiles - 1) / total_tiles;
        if (want > kt / 4) want = kt / 4;
        if (want < 1) want = 1;
    }
    if (want > kt) want = kt;
    const int64_t per = (kt + want - 1) / want;
    k_per_slice = (int)(per * 64);
    slices = (int)((kt + per - 1) / per);
}

// Rate of a CU that is busy with variant v (gemm, batched gemm and weight gradient), relative to the best variant.
double relative_rate(const VariantDesc &v) {
    const int64_t area = (int64_t)v.tile_m * v.tile_n;
    const bool two_buf = v.stages == 2 && v.tile_k == 64 && v.lb != 1 && v.la != 1;
    if (v.la == 1 || v.lb == 1) return area >= 128 * 128 ? 0.30 : 0.20;     // register-transposed operands
    const double nd = (v.lb == 4 ? 0.95 : 1.0) * (v.la == 5 ? 0.9 : 1.0);   // two LDS reads per fragment of a directly copied operand
    if (area >= 256 * 256) return nd * (two_buf ? 1.00 : v.stages >= 5 ? 0.92 : 0.90);
    if (area >= 256 * 128) return nd * (two_buf ? 0.81 : v.stages == 3 ? 0.80 : 0.73);
    // (with a directly copied operand the two-buffer loop of this size measured below the 4-stage one)
    if (area >= 128 * 128) return nd * (two_buf ? (nd < 1.0 ? 0.62 : 0.86) : v.tile_k == 32 ? (v.stages >= 4 ? 0.67 : 0.65) : 0.58);
    return nd * (v.tile_k == 64 ? 0.49 : v.stages == 3 ? 0.41 : 0.37);
}

// Launch time of variant v without a split, in the terms of the split model below, for the comparison of the two:
//     tiles of the busiest CU * ( tile FLOPs / rate + fixed cost of a tile, exposed as far as no co-resident workgroup hides it )
// (estimate_seconds is fitted to other measurements: a split in one model against no split in the other takes slices where whole
// tiles are sooner done, bf16 4096 x 512 x 16384 among them, and none where they pay.)
double estimate_whole_seconds(const VariantDesc &v, const Launch &L) {
    const double kCuRate = 1.38e15 / 256;            // FLOP/s of one CU at the best variant's measured rate
    const double kCuStore = 4.6e12 / 256;            // B/s of output one CU gets when all CUs store
    const int wg = workgroups_per_cu(v);
    const int64_t tiles = count_tiles(L, v.tile_m, v.tile_n);
    const int64_t slots = 256 * (int64_t)wg;
    // tiles the busiest CU works through: they run wg at a time, a new set starting when slots free up
    const double per_cu = tiles <= slots ? (double)((tiles + 255) / 256) : (double)((tiles + slots - 1) / slots * wg);
    // the chip is power-limited: CUs run faster when fewer of them are busy (measured ~1.5x at 144 of 256)
    const double active = tiles / per_cu < 256.0 ? tiles / per_cu : 256.0;
    double boost = pow(256.0 / (active < 1.0 ? 1.0 : active), 0.7);
    if (boost > 1.5) boost = 1.5;
    const double tile_flops = 2.0 * v.tile_m * v.tile_n * (double)L.K;
    const double out_bytes = (double)v.tile_m * v.tile_n * (L.dtD == UCL_F32 ? 4.0 : 2.0);
    const double fixed = 2.0e-6 + out_bytes / kCuStore;
    // co-resident workgroups hide about half of what perfect overlap of one's fixed cost with the
    // others' MFMA time would; a CU with a single tile has nothing to overlap with
    const double exposed = per_cu > 1.0 ? 0.5 * (1.0 + 1.0 / wg) : 1.0;
    // a variant built to share its CU runs below its rate when it has the CU to itself (one wave per SIMD
    // with the register budget of two: measured 0.7x for 256x128 tiles)
    const double alone = (wg >= 2 && per_cu < 2.0) ? 0.7 : 1.0;
    return per_cu * (tile_flops / (relative_rate(v) * alone * kCuRate * boost) + fixed * exposed);
}

// Launch time of variant v under split-K, for the choice among the variants when the caller names no tile.
// What counts differs from the unsplit case.  Every CU has a workgroup, so the mainloop is bound by one of: the
// operand bytes all workgroups together copy into LDS (measured ~10 TB/s over the chip when they stream from
// HBM, ~16 TB/s when the operands stay in the L2s), the MFMA rate, or a workgroup's own chain of copies (stages-1
// k-tiles in flight, a round trip of ~1.5 us from HBM, ~0.8 us from L2).  The partial tiles then cross memory:
// in parallel mode through a streaming reduction kernel and two more launches (measured: 6 us plus 1 us per MB
// of partial tiles; chains the reduction kernel finishes itself need one launch less, which is the same for every
// tile and is left out of the comparison), in serial mode through the last workgroup of each tile, which reads all slices alone
// (measured 15-28 GB/s per workgroup).
double estimate_split_seconds(const VariantDesc &v, const Launch &L, const ucl_tuning *tune) {
    const int64_t tiles = count_tiles(L, v.tile_m, v.tile_n);
    int slices = 1, kps = 0;
    split_slices(L, tune->split_k_slices, tiles, split_fill(L, v, tune), slices, kps);
    if (slices <= 1) return estimate_whole_seconds(v, L);
    const double wgs = (double)tiles * slices;
    const double rounds = ceil(wgs / (256.0 * workgroups_per_cu(v)));
    const double busy = wgs < 256.0 ? wgs / 256.0 : 1.0;
    const bool resident = (double)L.batch * (L.M + L.N) * (double)L.K * 2.0 <= 32.0e6;
    const double copy_bytes = wgs * kps * (double)(v.tile_m + v.tile_n) * 2.0;
    const double flops = 2.0 * wgs * kps * (double)v.tile_m * v.tile_n;
    double main = copy_bytes / ((resident ? 16.0e12 : 10.0e12) * busy);
    const double mfma = flops / (relative_rate(v) * 1.38e15 * busy);
    if (mfma > main) main = mfma;
    const double chain = rounds * (kps / (double)v.tile_k) * (resident ? 0.8e-6 : 1.5e-6) / (v.stages > 1 ? v.stages - 1 : 1);
    if (chain > main) main = chain;
    const double tile_bytes = (double)v.tile_m * v.tile_n * 4.0;
    if (tune->split_k_mode == UCL_SPLIT_K_PARALLEL) return main + 6.0e-6 + wgs * tile_bytes / 1.0e12;
    return main + 3.0e-6 + slices * tile_bytes / (v.tile_m * v.tile_n >= 128 * 128 ? 15.0e9 : 28.0e9);
}

// Weight gradient: kernel and slices of a parallel split-K call that leaves the slices to the library, chosen together.
// Its K (output pixels) is deep, its output small: what decides is how many k-tiles a workgroup chains (0.37 us each of the
// 64x64x32 kernel, whose four workgroups per CU hide the gathered operand best) against the bytes of partial tiles.
// Measured against one or two workgroups per CU of the tile the general split model likes: 120 drawn layers 1.26 times faster in the
// geometric mean (128 <- 1152 over 25088 pixels 47.0 -> 26.7 us), 40 that the general rule does not split 1.40 times.
// Parallel split-K with up to this many slices lets the last launch of the tile kernel add them up itself.
constexpr int kReduceInTileKernel = 2;

struct SplitChoice {
    const VariantDesc *v = nullptr;
    int slices = 1, k_per_slice = 0;
};
double estimate_wgrad_seconds(const VariantDesc &v, const CostRow &r, const Launch &L, int slices, int64_t k_per_slice) {
    const int64_t wgs = L.batch * ((L.M + v.tile_m - 1) / v.tile_m) * ((L.N + v.tile_n - 1) / v.tile_n) * slices;
    const int64_t slots = 256 * (int64_t)r.resident, rounds = (wgs + slots - 1) / slots;
    const double on_cu = wgs <= slots ? (double)((wgs + 255) / 256) : (double)(rounds * r.resident);
    const double tile_rows = (double)(L.M < v.tile_m ? L.M : v.tile_m) + (double)(L.N < v.tile_n ? L.N : v.tile_n), K = (double)k_per_slice;
    const double loop = fourth_power_sum(on_cu * tile_rows * K * 2.0 / (r.gbs * 1e3), on_cu * 2.0 * v.tile_m * v.tile_n * K / (r.tflops * 1e6),
                                         (double)rounds * (double)((k_per_slice + v.tile_k - 1) / v.tile_k) * r.step);
    double t = r.fixed + r.round * (double)rounds + loop;
    if (slices > 1) {
        SplitCostRow s = {0, 0, 0, 0, 2.f, 2.4f};
        for (const SplitCostRow &c : kWgradSplitRows)
            if (c.tile_m == v.tile_m && c.tile_n == v.tile_n && c.tile_k == v.tile_k && c.stages == v.stages) s = c;
        t += s.fixed + (double)wgs * v.tile_m * v.tile_n * 4.0 / (s.tbs * 1e6) + 0.02 * slices;
        // (two slices are not added up by the reduction kernel but by another launch of the tile kernel: 5 us more than three, 361 to 2916 pixels)
        if (slices <= kReduceInTileKernel) t += 5.0;
    }
    return 1e-6 * t;
}
// Operand panels are addressed with 32-bit byte offsets inside range-checked buffer resources.
bool panel_fits(int64_t rows, int64_t ld, int64_t K) { return (rows * ld + K) * 2 < (1ll << 31); }
bool panels_fit(const VariantDesc &v, const Launch &L) {
    return (v.la != 0 || panel_fits(v.tile_m, L.lda, L.K)) && (v.lb != 0 || panel_fits(v.tile_n, L.ldb, L.K));
}

bool names_tile(const ucl_tuning *tune);
const VariantDesc *select_variant(const Launch &L, const ucl_tuning *tune);
SplitChoice general_split(const Launch &L, const ucl_tuning *tune);

// GEMM, both 16-bit operands contiguous along K: the same, for the two kernels that were the fastest or next to it in 310 problems
// (32..768 rows and columns, K 2048..65536; tiles of 64x64 nearly always, of 128x128 where there are 20 and more).  Constants
// fitted to every power of two of slices: launches, GB/s copied per CU, us per k-tile of a chain, TB/s of partial tiles and
// of operands, us that each slice adds to the reduction's chain of loads.
struct GemmSplitRow {
    int tile;
    double fixed, gbs, tflops, step, partial_tbs, operand_tbs, slice;
};
constexpr GemmSplitRow kGemmSplitRows[] = {{64, 10.46, 90.7, 20.0, 0.207, 2.24, 5.10, 0.022}, {128, 13.24, 81.4, 20.0, 0.640, 3.07, 5.63, 0.017}};
bool has_gemm_split_row(const VariantDesc &v) {
    return v.mode == 0 && v.la == 0 && v.lb == 0 && v.k_groups == 1 && v.tile_k == 64 &&
           ((v.tile_m == 64 && v.tile_n == 64 && v.stages == 4) || (v.tile_m == 128 && v.tile_n == 128 && v.stages == 2));
}
double estimate_gemm_split_seconds(const VariantDesc &v, const Launch &L, int slices, int64_t k_per_slice) {
    const GemmSplitRow &r = kGemmSplitRows[v.tile_m == 64 ? 0 : 1];
    const int64_t wgs = count_tiles(L, v.tile_m, v.tile_n) * slices, resident = 2;
    const int64_t slots = 256 * resident, rounds = (wgs + slots - 1) / slots;
    const double on_cu = wgs <= slots ? (double)((wgs + 255) / 256) : (double)(rounds * resident);
    const double tile_rows = (double)(L.M < v.tile_m ? L.M : v.tile_m) + (double)(L.N < v.tile_n ? L.N : v.tile_n), K = (double)k_per_slice;
    const double loop = fourth_power_sum(on_cu * tile_rows * K * 2.0 / (r.gbs * 1e3), on_cu * 2.0 * v.tile_m * v.tile_n * K / (r.tflops * 1e6),
                                         (double)rounds * (double)((k_per_slice + 63) / 64) * r.step,
                                         (double)(L.M + L.N) * (double)L.K * 2.0 / (r.operand_tbs * 1e6));
    return 1e-6 * (r.fixed + loop + (double)wgs * v.tile_m * v.tile_n * 4.0 / (r.partial_tbs * 1e6) + r.slice * slices);
}

// Parallel split-K calls whose slices the library chooses together with the kernel
bool split_left_open(const Launch &L, const ucl_tuning *tune) {
    if (!tune || tune->split_k_mode != UCL_SPLIT_K_PARALLEL || tune->split_k_slices != 0 || tune->scheduler != UCL_SCHED_DEFAULT) return false;
    if (L.mode == 4) return true;
    // (fp32 results keep the slices of the general rule: the sums' rounding shows in them, and longer slices round more, 2.2e-7 to
    // 4.4e-7 on 464 x 393 x 19848; a 16-bit output's error is the same to six digits either way)
    // (K as far as the rows were fitted: 936 x 472 x 103648 took 157 us by them, 128 us by the general rule)
    return L.mode == 0 && L.K <= 65536 && !L.f32_results && L.batch == 1 && L.la == 0 && L.lb == 0 && (L.dt == 0 || L.dt == 1) && !names_tile(tune);
}
SplitChoice choose_split(const Launch &L, const ucl_tuning *tune) {
    const bool named = names_tile(tune);
    const int64_t kt = (L.K + 63) / 64;
    SplitChoice best;
    double best_t = 0;
    SplitChoice general;
    if (L.f32_results) general = general_split(L, tune);
    // The filter gradient in fp32: the same slices as the general rule's or shorter ones, as longer ones would round more (fp16 32 x 28 x 28
    // x 512 -> 256, 3x3 at stride 2: with 3 slices instead of 8 2.9e-7 instead of 1.9e-7 off the exact sums).
    const int64_t longest = general.v && general.slices > 1 ? general.k_per_slice : kt * 64;
    for (int i : variants_of(L.mode, L.dt)) {
        const VariantDesc &v = all_variants()[i];
        if (v.persistent) continue;
        if (L.mode == 0 && !(has_gemm_split_row(v) && panels_fit(v, L))) continue;
        // Over many pixels the two k-tiles that 64x64x32 has in flight, 4 KB of each operand, don't cover the trips to memory: 64 <- 576 columns over
        // 100352 pixels 32.8 us, 64x64x64 26.0 us; 128 <- 576 over as many 53.7 us, 128x128x32 33.9 us.  Below, its four workgroups per CU
        // do (128 <- 1152 over 6272: 17.0 against 17.0 us, 256 <- 2304 over 1568: 19.4 against 24 us).  Between, 54 layers of 20000 to 49152 pixels: with
        // more than 32 filters it is mostly behind (184 <- 216 over 36000: 21.2 against 18.5 us, 264 <- 1512 over 33300: 97 against 76 us), with up to
        // 32 mostly ahead (24 <- 2952 over 25200: 36.6 against 41.0 us, 16 <- 1584 over 31360: 28.5 against 32.8 us).
        if (L.mode == 4 && !named && v.tile_m == 64 && v.tile_k == 32 && L.K > (L.M <= 32 ? 49152 : 24576)) continue;
        if (named && (v.tile_m != tune->tile_m || v.tile_n != tune->tile_n || v.tile_k != tune->tile_k || v.stages != tune->stages)) continue;
        const int64_t tiles = count_tiles(L, v.tile_m, v.tile_n);
        // A GEMM whose tiles fill the chip without a split gains nothing from one, and larger outputs than that were not fitted (fp16 2254 x 2456
        // x 13408, 360 tiles of 128x128: 204 us whole, 224 us in 4 slices; bf16 3081 x 1795 x 34392, 375 tiles: 566 and 631 us).
        if (L.mode == 0 && tiles >= kNumCUs) continue;
        // no split, a few slices, and what fills the chip with one to eight workgroups per CU
        const int64_t fills[] = {1, 2 * tiles, 4 * tiles, 256, 512, 768, 1024, 1536, 2048, general.slices * tiles};
        for (int64_t fill : fills) {
            int64_t want = (fill + tiles - 1) / tiles;
            if (want > kt / 2) want = kt / 2;
            if (want < 1) want = 1;
            // (more slices than 64 were not measured for a GEMM)
            if (L.mode == 0 && want > 64) want = 64;
            int slices = 1, kps = 0;
            split_slices(L, want, tiles, 0, slices, kps);
            if (L.mode == 0 && slices == 1) continue;       // (a GEMM that is not split has more kernels: below)
            if (kps > longest || (slices > 1 && tiles > UCL_SPLIT_K_MAX_TILES)) continue;
            const double t = L.mode == 0 ? estimate_gemm_split_seconds(v, L, slices, kps)
                                         : estimate_wgrad_seconds(v, all_costs()[i], L, slices, slices > 1 ? kps : L.K);
            if (!best.v || t < best_t) {
                best_t = t;
                best.v = &v;
                best.slices = slices;
                best.k_per_slice = kps;
            }
        }
    }
    // The few-row kernels and K groups often need less time for the whole of K than the launches of a split take: 1.4 to 1.8 times
    // less at K = 4096 to 5000 (88 x 159 x 4200: 7.1 against 12.1 us), 1.2 times at 8192 and up to 16 tiles.  Beyond that K their
    // workgroups have to be enough to draw on the memory, and their rows, fitted up to K = 16384, are trusted less: 1 x 1508 x 9560 8.9
    // against 18.9 us, 8 x 6072 x 11888 38.4 against 53.0 us, but split 1664 x 16 x 31144 takes 45.4 us instead of 61.2, 16 x 2039 x 29328
    // 39.6 instead of 57.5 us (priced at 0.86 and 0.83 of the split).  Over 110 problems with a side above 768 and K of 8192 to 65536 1.09 times less time
    // than always split, none slower.
    if (L.mode == 0) {
        const VariantDesc *v = select_variant(L, nullptr);
        bool one = false;
        if (!best.v || (v && (L.K <= 8192 || count_tiles(L, v->tile_m, v->tile_n) >= 64) &&
                        estimate_seconds(*v, all_costs()[v - all_variants().data()], many_tiles_costs()[v - all_variants().data()], L, &one) < (L.K <= 8192 ? 0.9 : 0.8) * best_t)) {
            best.v = v;
            best.slices = 1;
        }
    }
    return best;
}
int64_t split_bytes(const Launch &L, const SplitChoice &c) {
    if (!c.v || c.slices <= 1) return 0;
    return UCL_WORKSPACE_COUNTER_BYTES + (int64_t)c.slices * count_tiles(L, c.v->tile_m, c.v->tile_n) * c.v->tile_m * c.v->tile_n * 4;
}

// Filter gradients whose slices are left to the library: wgrad_taps_kernel and its slices (0: the kernel and slices chosen above).
// The constants of its launch time were fitted to 16670 launches of 3992 of 17441 timed geometries (1 to 64 images, 3 to 62 pixels a side, 8 to 512
// channels and filters, up to ten choices of slices each; 5 % off in the mean near the best choice): microseconds of a launch, of a round of
// workgroups and of a k-tile in it, of the second launch, TB/s of partial sums, what a slice and a MB of the gradient add.
struct TapsRow {
    double fixed, round, ktile, second, partial_tbs, slice, out;
};
constexpr TapsRow kTapsRows[2] = {{3.78, 2.48, 0.679, 2.88, 2.97, 0.025, 0.244}, {3.75, 2.56, 0.534, 2.86, 3.16, 0.023, 0.180}};
struct TapsChoice {
    int slices = 0, px_per_slice = 0;
};
TapsChoice choose_taps(const Launch &L, const VariantDesc &v, const SplitChoice &other) {
    TapsChoice best;
    const TapsRow &r = kTapsRows[L.taps_stride - 1];
    const int64_t kt = L.taps_stride == 1 ? 128 : 64, nk = (L.cN * (L.cP + 1) * (L.cQ + 1) + kt - 1) / kt;
    const int64_t tiles = ((L.M + 63) / 64) * ((L.cC + 31) / 32);
    const double out_mb = (double)L.M * L.N * 4e-6;
    // What the tile kernel is expected to take.  Both models are off by some 5 %: a tie stays with it.
    double best_t = 0.94e6 * estimate_wgrad_seconds(v, all_costs()[&v - all_variants().data()], L, other.slices, other.slices > 1 ? other.k_per_slice : L.K);
    // An accumulator's roundings: one per MFMA (32 pixels) of its chain and one per slice; their squares weigh about alike in the error of the sum.
    // fp32 results take no choice with more of them than the tile kernel's.  (16-bit ones may: their own rounding is hundreds of times a sum's error.)
    const int64_t roundings = (other.slices > 1 ? other.k_per_slice : L.K) / 32 + other.slices;
    // no split, and what gives 1/4 to all of the CUs a workgroup, or two
    const int fills[] = {1, 64, 96, 128, 160, 192, 224, 256, 384, 512};
    for (int fill : fills) {
        int64_t want = fill / tiles;
        if (want > nk) want = nk;
        if (want < 1) want = 1;
        const int64_t per = (nk + want - 1) / want, slices = (nk + per - 1) / per;
        if (L.f32_results && per * kt / 64 + slices > roundings) continue;
        const int64_t rounds = (tiles * slices + kNumCUs - 1) / kNumCUs;
        const double t = r.fixed + (double)rounds * (r.round + r.ktile * (double)per) + out_mb * r.out +
                         (slices > 1 ? r.second + (double)slices * (out_mb / r.partial_tbs + r.slice) : 0.0);
        if (t < best_t) {
            best_t = t;
            best.slices = (int)slices;
            best.px_per_slice = (int)(per * kt);
        }
    }
    return best;
}
bool takes_taps(const Launch &L, const ucl_tuning *tune) { return L.taps_stride > 0 && split_left_open(L, tune) && !names_tile(tune); }
bool serves_taps(const Launch &L, const KParams &kp, const ucl_tuning *tune) {
    return L.mode == 4 && takes_taps(L, tune) && kp.fused.enabled && !kp.fused.has_bias && !kp.fused.has_res && !kp.fused.act;
}
int64_t taps_bytes(const Launch &L, const TapsChoice &c) { return c.slices > 1 ? UCL_WORKSPACE_COUNTER_BYTES + (int64_t)c.slices * L.M * L.N * 4 : 0; }

// Kernels that the general rule chooses among.  Split-K has kernels without K groups only.  And the slices an open call gets are what
// fills the chip with the chosen tile, so a larger tile makes longer slices, and their fp32 sums round more: fp16 calls stay with the
// tiles whose slices their results have always had (with all that bf16 has, fp16 -> fp32 512 x 512 x 8192 has 4 slices
// instead of 16 and is 2.9e-7 off the exact sums instead of 1.7e-7, A^T B 4096 x 256 x 16384 none instead of 16, 8.1e-7 instead of 2.2e-7).
bool in_general_rule(const VariantDesc &v) {
    if (v.k_groups > 1) return false;
    if (v.dt != 1 || v.la == 1 || v.lb == 1) return true;
    if (v.tile_m * v.tile_n == 64 * 64) return v.tile_k == 32 && v.stages == 3;
    if (v.mode == 4) return v.tile_k == 32;
    if (v.la == 5) return v.tile_m * v.tile_n == 256 * 256;
    return v.lb != 4 || v.tile_m * v.tile_n != 256 * 128;
}

// Does a variant of L's operation and input type serve its layouts, and the scheduler and iterator that the call names?
bool serves(const VariantDesc &v, const Launch &L, const ucl_tuning *tune) {
    const int want_persistent = !tune ? 0 : tune->scheduler == UCL_SCHED_PERSISTENT ? 1 : tune->scheduler == UCL_SCHED_STREAM_K ? 2 : 0;
    if (v.persistent != want_persistent) return false;
    if (v.lb == 4 ? !(L.lb == 1 && L.ndirect_ok) : v.lb != L.lb) return false;
    if (L.mode == 2 || L.mode == 3) {
        // conv: the iterator knob picks between the per-tap gather (la 2) and the resident patch (la 3)
        const int it = tune ? tune->iterator : 0;
        return v.la == 3 ? (L.patch_c == v.patch_c && it != UCL_ITER_ANALYTIC) : (v.la == 2 && it != UCL_ITER_FIXED_STRIDE_DILATION);
    }
    return v.la == 5 ? (L.la == 1 && L.mdirect_ok) : v.la == L.la;
}
bool names_tile(const ucl_tuning *tune) { return tune && (tune->tile_m || tune->tile_n || tune->tile_k || tune->stages); }

// Is a few-row kernel a candidate where no tile is named?  (L.K counts pairs for 8-bit inputs.)
// GEMM: from the second 64-wide step of a wave's row on; measured over 104 problems of up to 600 rows and K of 72 to 640 they are 4 to 32 %
// ahead of the tile kernels wherever the cost rows choose them, none behind.  16-bit inputs at K up to 256, where that is 4 to 20 %, stay
// with the tile kernels that ucl_select_tuning has always reported for them.
// Grouped: with a tile for each CU at most they are ahead from K = 256 on (6 groups of 896 columns, e4m3, K = 960: 4.5 against 5.7 us; 7 of 832
// columns bf16 4.8 against 6.1 us).  With more tiles, those with one buffer per wave from K = 512 on, the least that was fitted (64 experts of 0 ..
// 32 rows, 2048 columns, K = 1024, e4m3 27 us, tile kernel 32 us; 128 of 4096 columns, K = 512 54 and 70 us; 49 of 30 rows, 2400 columns, K = 576 bf16
// 32.4 and 37.5 us; below, 39 groups of 51 rows, 2312 columns, K = 256 bf16 21.8 and 17.2 us), and those with several where K is deep (38 of 2100
// columns, K = 1536: 45 us against 58 us for the tile kernels).  Convolutions: five steps, as their row was fitted.
bool few_rows_apply(const VariantDesc &v, const Launch &L) {
    if (L.mode == 1) {
        const bool many = count_tiles(L, v.tile_m, v.tile_n) > kOneBufferAbove;
        if (v.stages != 1) return many && L.K >= (L.dt >= 2 ? 256 : 512);
        return L.K >= 1408 || (!many && L.K >= (L.dt >= 2 ? 128 : 256));
    }
    // (64 rows: for half of them at least, which is what its row was fitted to; 26 x 12360 x 7680 bf16 46.0 us, 16x32 tiles 41.4 us; and for half of
    // the CUs: with fewer tiles each wave's one buffer keeps too little of B's way from memory in flight, 35 x 7304 x 8016 bf16 51.9 us, 32x64 tiles
    // 40.3 us; over 3600 problems it is 1.04 to 1.7 times behind below 128 tiles, level from there on)
    if (L.mode == 0) return L.K > (L.dt >= 2 ? 64 : 256) && (v.tile_m < 64 || (L.M > 32 && count_tiles(L, v.tile_m, v.tile_n) >= kNumCUs / 2));
    return L.K >= 320;
}

// Microseconds that the CUs take for a conv_held_kernel launch (constants in ucl_costs.h): the workgroups of a round have `pairs` pairs of rows per
// wave to multiply and `pixels` bytes of pixels and their filters to copy, whose rate falls with the CUs that copy.
double held_microseconds(const HeldPlan &h, double pairs, int64_t pixels) {
    const HeldCosts &c = kHeldCosts;
    const int k = h.kg == 1 ? 0 : h.kg == 2 ? 1 : 2, mg = 8 / (h.kg * h.ng), m = mg == 1 ? 0 : mg == 2 ? 1 : 2;
    const double filter = h.kg * h.ng * 36.864e3, fixed = c.pass[k] + c.sharing[m] + c.pair[k] * pairs;
    auto round = [&](double busy) { return h.passes * (fixed + filter * (c.filter * busy + c.filter_alone) + (double)pixels * (c.pixels * busy + c.pixels_alone)) + c.next_pass * (h.passes - 1); };
    const int wgs = h.bands * h.tiles_n, full = wgs / kNumCUs, rest = wgs % kNumCUs;
    return c.launch + (double)full * round(1.0) + (rest ? round((double)rest / kNumCUs) : 0.0);
}

// How conv_held_kernel would cut up a problem: of the plans whose pixels fit into LDS, with as many rows per workgroup as one to four rounds
// of workgroups take, or as LDS holds where that is fewer, the one with the shortest estimate.  (Every call that may be served asks: 32-bit
// numbers, what all plans move left to the end, and no strips shared out among more waves than there are strips.)
HeldPlan choose_held(const Launch &L, bool residual) {
    HeldPlan best;
    if (!L.held_stride) return best;
    HeldPlan h;
    h.stride = L.held_stride;
    h.kg = L.cC <= 64 ? 1 : L.cC <= 128 ? 2 : kHeldMaxKG;
    h.passes = (int)((L.cC + 64 * h.kg - 1) / (64 * h.kg));
    h.pair = L.cQ <= 7 ? 2 : 1;
    h.pitch = (int)(L.cQ + 16) / 16 * 16;
    h.strips = h.pair == 2 ? 1 : (int)(L.cQ + 15) / 16;
    h.rows = (int)((L.cN + h.pair - 1) / h.pair * (L.cP + 1));
    double best_us = 0;
    for (h.ng = 4; h.ng >= 1; h.ng /= 2) {
        const int capacity = held_patch_capacity(h.kg, h.ng);
        if (capacity == 0) continue;
        h.tiles_n = ((int)L.N + 32 * h.ng - 1) / (32 * h.ng);
        const int mg = 8 / (h.kg * h.ng);
        for (h.strip_split = 1; h.strip_split <= mg && (h.strip_split == 1 || h.strip_split / 2 < h.strips); h.strip_split *= 2) {
            const int groups = mg / h.strip_split, strips = (h.strips + h.strip_split - 1) / h.strip_split;
            auto per_of = [&](int R) { return held_rows_of_wave(R, groups, h.kg, h.passes > 1); };
            // (sums of earlier passes: one more pair, what the first pair's MFMAs find to finish)
            auto keep_of = [&](int R) { return h.passes > 1 ? (per_of(R) * strips + 2) * 512 * (8 / h.kg) * 4 : 0; };
            int most = ((capacity / h.kg / 128 - 8) / (h.stride * h.pitch) - 3 + h.stride) / h.stride;
            while (most > 0 && held_plane_bytes(h.stride, most, h.pitch) * h.kg + keep_of(most) > capacity) --most;
            for (int rounds = 1, tried = 0; rounds <= 4 && most > 0; ++rounds) {
                const int bands = kNumCUs * rounds / h.tiles_n;
                h.R = bands > 0 ? (h.rows + bands - 1) / bands : most + 1;
                if (h.R > most) {
                    if (rounds < 4) continue;
                    h.R = most;
                }
                if (h.R == tried) continue;
                tried = h.R;
                // (rows are multiplied in pairs and strips 16 columns at a time: what is read beyond the band's pixels has to be in LDS, too)
                const int per = per_of(h.R), last = (h.R - 1) / per * per + per;
                const int64_t plane = held_plane_bytes(h.stride, h.R, h.pitch);
                if (plane * (h.kg - 1) + ((int64_t)(h.stride * (last - 1) + 3) * h.stride * h.pitch + 16 * h.strip_split + 32) * 128 > kLdsBytesPerCU) continue;
                h.bands = (h.rows + h.R - 1) / h.R;
                h.keep_bytes = keep_of(h.R);
                const double us = held_microseconds(h, (per / 2 + (per & 1 ? 0.55 : 0.0)) * strips, plane * h.kg);
                if (best.R == 0 || us < best_us) { best = h; best_us = us; }
                if (h.R == most || h.R == 1) break;
            }
        }
    }
    const HeldCosts &c = kHeldCosts;
    const double moved = (double)L.gathered + (double)(L.cN * L.cP * L.cQ) * (double)(L.N * (residual ? 2 : 1)) * 2.0;
    best.seconds = 1e-6 * fourth_power_sum(best_us, c.memory + c.moved * moved + c.weights * (double)(9 * L.cC * L.N) * 2.0);
    return best;
}

// Seconds of the tile kernel that a 3x3 convolution would get instead (kConvRows), 0 for one without a row.
double tile_kernel_seconds(const VariantDesc &v, const Launch &L, bool residual) {
    for (const ConvRow &r : kConvRows) {
        if (r.mode != v.mode || r.tile_m != v.tile_m || r.tile_n != v.tile_n || r.tile_k != v.tile_k || r.stages != v.stages || r.k_groups != v.k_groups || r.patch_c != v.patch_c) continue;
        const int64_t tiles_n = (L.N + v.tile_n - 1) / v.tile_n, tiles = count_tiles(L, v.tile_m, v.tile_n), slots = kNumCUs * r.resident, rounds = (tiles + slots - 1) / slots;
        const double on_cu = tiles <= slots ? (double)((tiles + kNumCUs - 1) / kNumCUs) : (double)(rounds * r.resident), K = (double)L.K, N = (double)L.N;
        const double lines = (double)((L.cC + 63) / 64 * 64) / (double)L.cC - 1.0;
        const double rows = v.tile_m * (1.0 + r.lines * lines + (L.held_stride == 2 ? r.stride2 : 0.0) + (L.cC % 64 ? r.odd_c : 0.0));
        const double columns = (L.N < v.tile_n ? N : v.tile_n) + (L.N < 64 ? r.few_n * (64.0 - N) : 0.0);
        const double copies = on_cu * (rows + columns) * K * 2.0 / (r.gbs * 1e3);
        const double math = on_cu * 2.0 * v.tile_m * v.tile_n * K / (r.tflops * 1e6);
        const int64_t step_k = (is_few_row(v) ? 64 : v.tile_k) * v.k_groups;
        const double chain = (double)(rounds * ((L.K + step_k - 1) / step_k)) * r.step, memory = ((double)L.gathered + N * K * 2.0) / 5.3e6 * r.memory;
        const double out = (double)L.M * N * 2.0 / 4.6e6 * (r.out + (residual ? r.residual : 0.0)) *
                           (1.0 + (L.N % v.tile_n ? r.part / (double)tiles_n : 0.0) + (L.N % 64 ? r.half_line : 0.0));
        return 1e-6 * (r.fixed + r.round * (double)rounds + fourth_power_sum(fourth_power_sum(copies, math, chain, memory), out * r.hidden) + out * (1.0 - r.hidden));
    }
    return 0;
}

// The plan of a convolution that runs on conv_held_kernel, R = 0 for one that does not: calls that name nothing, with the chains of the usual layers (scale,
// bias, residual, ReLU) and outputs of the inputs' type, where the estimate is shorter than that of the kernel `v` the call would get.
HeldPlan plan_held(const Launch &L, const KParams &kp, const ucl_tuning *tune, const VariantDesc &v) {
    if (!L.held_stride || (tune && (names_tile(tune) || tune->raster || tune->iterator || tune->scheduler || tune->split_k_mode))) return HeldPlan();
    const int type = L.dt == 1 ? UCL_F16 : UCL_BF16;
    const FusedEpi &f = kp.fused;
    if (!f.enabled || (f.act && f.act != UCL_EPI_RELU) || L.dtD != type || !kp.d_vec || (f.has_res && (f.res_dt != (type | 0x100) || f.res_ld != L.N))) return HeldPlan();
    const double tile_seconds = tile_kernel_seconds(v, L, f.has_res != 0);
    const HeldPlan h = choose_held(L, f.has_res != 0);
    return h.R > 0 && h.seconds < tile_seconds ? h : HeldPlan();
}

const VariantDesc *select_variant(const Launch &L, const ucl_tuning *tune) {
    const auto &vs = all_variants();
    const auto &costs = all_costs(), &many = many_tiles_costs();
    const VariantDesc *best = nullptr;
    double best_t = 0;
    bool best_fits = false;
    for (int i : variants_of(L.mode, L.dt)) {
        const VariantDesc &v = vs[i];
        if (!serves(v, L, tune)) continue;
        if (names_tile(tune)) {
            if (v.tile_m != tune->tile_m || v.tile_n != tune->tile_n || v.stages != tune->stages || v.tile_k != tune->tile_k)
                continue;
            if (v.k_groups > 1 && tune->split_k_mode != UCL_SPLIT_K_NONE) continue;     // (split-K has kernels without K groups only)
            // of several kernels with the named shape: the resident-patch one, else one with the K groups named, else one without,
            // else a direct-copy one, else the first
            if (v.la == 3) return &v;
            if (best && best->k_groups != v.k_groups) {
                if (best->k_groups != tune->k_groups && (v.k_groups == tune->k_groups || v.k_groups < best->k_groups)) best = &v;
                continue;
            }
            const bool direct = v.la == 5 || v.lb == 4;
            if (!best || (direct && !(best->la == 5 || best->lb == 4))) best = &v;
            continue;
        }
        if (is_few_row(v) && !few_rows_apply(v, L)) continue;
        // A^T B of one row or column of up to 64 64x64 tiles: the fitted rows price the 128x128 kernel with K groups, whose copies bound
        // every problem it was fitted on, without its chain, and the 64x64 one without them below the one with (8 x 8 x 2048 fp32:
        // 15.4, 9.2 and 8.6 us; 8 x 24 x 7168 36.4, 23.2 and 19.3 us; 64 x 4096 x 2048 12.5 us without, 12.2 with).
        if (L.mode == 0 && v.la == 5 && v.lb == 4 && (L.M <= 64 || L.N <= 64) && count_tiles(L, 64, 64) <= 64 &&
            (v.tile_m == 128 ? v.k_groups > 1 : v.tile_m == 64 && v.tile_k == 64 && v.k_groups == 1 && L.K >= 2048))
            continue;
        // K groups of the data gradient: with fewer than three k-tiles for each of the two there is nothing to share out (24 <- 32 at 3x3, 9 x 5 x 5:
        // 9.7 against 8.3 us, 24 <- 24 over 3 x 24 x 24 9.7 against 8.6 us).
        if (L.mode == 3 && v.k_groups > 1 && L.K < 320) continue;
        bool one = false;
        double t = L.mode == 4 ? estimate_wgrad_seconds(v, costs[i], L, 1, L.K) : estimate_seconds(v, costs[i], many[i], L, &one);
        // Above 300 rows, and where K gives a wave a single step, the tile kernels are the few-row ones' rivals and both rows are 10 to 15 % off: what is no
        // clear win stays with the tile kernel.  (Slower than the choice among tile kernels by more than 4 %: 6.4 -> 3.8 % of 2700 16-bit problems of
        // 301 to 3000 rows, the timing's own share, and 7 -> 2 % of 3900 8-bit ones of K = 144 to 512, which are still 1.07 to 1.14x in the mean.)
        if (L.mode == 0 && one && (L.K <= 256 || L.M > 300)) t *= L.K <= 256 ? 1.3 : 1.2;
        // (a large tile must not make a call fail that a smaller one serves)
        const bool fits = panels_fit(v, L);
        if (!best || (fits && !best_fits) || (fits == best_fits && t < best_t)) { best_t = t; best = &v; best_fits = fits; }
    }
    return best;
}

// Kernel and slices of a split-K call by the general rule: a named tile with the slices of split_slices, else the kernel that the
// split model likes best with its slices.  Where that is no split at all the call runs as it would without a tuning.
SplitChoice general_split(const Launch &L, const ucl_tuning *tune) {
    SplitChoice c;
    if (names_tile(tune)) {
        c.v = select_variant(L, tune);
        if (c.v) split_slices(L, tune->split_k_slices, count_tiles(L, c.v->tile_m, c.v->tile_n), split_fill(L, *c.v, tune), c.slices, c.k_per_slice);
        return c;
    }
    double best_t = 0;
    for (int i : variants_of(L.mode, L.dt)) {
        const VariantDesc &v = all_variants()[i];
        if (!serves(v, L, tune) || !in_general_rule(v)) continue;
        const double t = estimate_split_seconds(v, L, tune);
        if (!c.v || t < best_t) { best_t = t; c.v = &v; }
    }
    if (!c.v) return c;
    split_slices(L, tune->split_k_slices, count_tiles(L, c.v->tile_m, c.v->tile_n), split_fill(L, *c.v, tune), c.slices, c.k_per_slice);
    if (c.slices <= 1) c.v = select_variant(L, nullptr);
    return c;
}

// The kernel of a call, and under split-K the slices chosen with it.  A call without a workspace, or with one that the partial tiles of
// chosen slices don't fit into, is served by the general rule: it may need less, or none at all.  `sizing`: no call yet,
// any workspace can be had.
const VariantDesc *select_with_split(const Launch &L, const ucl_tuning *tune, SplitChoice &choice, bool sizing = false) {
    const bool split = tune && tune->split_k_mode != UCL_SPLIT_K_NONE && tune->split_k_slices >= 0 && (L.mode == 0 || L.mode == 4) &&
                       tune->scheduler == UCL_SCHED_DEFAULT;
    if (!split) return select_variant(L, tune);
    if (split_left_open(L, tune)) {
        choice = choose_split(L, tune);
        const int64_t bytes = split_bytes(L, choice);
        if (!sizing && bytes > 0 && (!tune->workspace || !aligned16(tune->workspace) || bytes > tune->workspace_bytes)) choice = SplitChoice();
    }
    if (!choice.v) choice = general_split(L, tune);
    return choice.v;
}

// A 1x1 convolution at unit stride without padding IS a GEMM over the pixels: its forward pass (pixels x channels times filter
// rows) and its data gradient (output gradient times the filter, contiguous along N) run on the GEMM kernels, which copy rows
// instead of gathering taps and come in more tiles.  A named tile is the GEMM kernel's where one is built (what ucl_select_tuning
// answers names the same kernel again), else the convolution kernel's; with an iterator named, or another
// scheduler, it is the convolution kernel's.
bool is_plain_gemm(int64_t R, int64_t S, int64_t pad_h, int64_t pad_w, int64_t stride_h, int64_t stride_w) {
    return R == 1 && S == 1 && pad_h == 0 && pad_w == 0 && stride_h == 1 && stride_w == 1;
}
Launch gemm_of_conv(const Launch &conv) {
    Launch g;
    g.M = conv.M; g.N = conv.N; g.K = conv.K;
    g.la = 0;
    g.lb = conv.mode == 3 ? 1 : 0;
    g.ndirect_ok = conv.mode == 3;             // (the filter is below 2 GiB)
    g.dt = conv.dt; g.dtD = conv.dtD;
    return g;
}
// (Measured over 60 drawn layers: data gradients 1.41x, forward passes 1.11x.  Forward with one 64-wide k-tile is all output
// and residual: the convolution kernels' choice is 10 % ahead there, 22.5 against 25.1 us on 36 x 60 x 60 x 64 -> 128.)
bool takes_gemm(const Launch &conv, const Launch &gemm, const ucl_tuning *tune) {
    if (conv.mode == 2 && conv.K < 128 && !names_tile(tune)) return false;
    if (!tune) return true;
    if (tune->split_k_mode != UCL_SPLIT_K_NONE || tune->split_k_slices != 0 || tune->scheduler != UCL_SCHED_DEFAULT || tune->iterator != UCL_ITER_DEFAULT) return false;
    return select_variant(gemm, tune) != nullptr;
}

int default_raster(const VariantDesc &v, const Launch &L) {
    // bands of ~1024 rows: an XCD's run of 32 consecutive tiles then covers a near-square block.  Tiles of 64 rows: even bands of up to ten tiles, for the
    // same reason (2500 problems, against bands of 16: 11 to 16 rows of tiles 0.97 to 0.98 of the time, more 0.95 to 0.99; bands of eight tiles and
    // a rest cost 1.02 to 1.03 where there are nine or ten rows of tiles, 610 x 2024 x 5408 fp16 42.7 instead of 33.3 us).  With k-tiles of 32 four
    // workgroups share a CU, and bands of eight do as well as any from 17 rows of tiles on (0.99, even ones 1.01).  A group's rows stay in one band.
    if (v.tile_m == 64 && L.mode == 0) {
        const int64_t rows = (L.M + 63) / 64, bands = (rows + 9) / 10;
        return v.tile_k == 32 && rows > 16 ? 8 : (int)((rows + bands - 1) / bands);
    }
    int gm = 1024 / v.tile_m;
    return gm < 1 ? 1 : gm;
}

ucl_status check_epilogue(const ucl_epilogue *epi, const Launch &L, KParams &kp) {
    kp.n_steps = 0;
    memset(&kp.fused, 0, sizeof(kp.fused));
    kp.fused.enabled = 1;             // the empty chain is the trivial fused form
    if (!epi) return UCL_OK;
    if (epi->n_steps < 0 || epi->n_steps > UCL_MAX_EPI_STEPS)
        return fail(UCL_ERR_INVALID_ARG, "epilogue has %d steps; the chain holds 0..%d", epi->n_steps, UCL_MAX_EPI_STEPS);
    for (int i = 0; i < epi->n_steps; ++i) {
        const ucl_epi_step &s = epi->steps[i];
        if (s.op < UCL_EPI_SCALE || s.op > UCL_EPI_AUX_STORE)
            return fail(UCL_ERR_INVALID_ARG, "epilogue step %d: unknown op code %d", i, s.op);
        EpiStepDev &d = kp.steps[i];
        d.op = s.op; d.dtype = s.dtype; d.p0 = s.p0; d.p1 = s.p1; d.ptr = s.ptr; d.ld = s.ld; d.bs = s.bs;
        if (op_has_tensor(s.op)) {
            if (!s.ptr) return fail(UCL_ERR_INVALID_ARG, "epilogue step %d needs a tensor operand but ptr is NULL", i);
            if (!valid_dtype(s.dtype)) return fail(UCL_ERR_INVALID_ARG, "epilogue step %d: bad tensor dtype %d", i, s.dtype);
            // 128-bit accesses of 8 (16-bit) or 4 (fp32) elements need 16-byte aligned rows
            const int per16 = 16 / elem_size(s.dtype);
            bool vec = true;
            if (L.mode != 1) vec = aligned16(s.ptr);
            // (grouped: the per-group pointers live on the device and are required to be 16-byte aligned)
            if (op_is_matrix(s.op)) {
                if (s.ld < L.N) return fail(UCL_ERR_INVALID_ARG, "epilogue step %d: ld=%lld is smaller than N=%lld", i, (long long)s.ld, (long long)L.N);
                vec = vec && (s.ld % per16 == 0) && (s.bs % per16 == 0) && s.ld <= kMaxWideLd;
            }
            if (vec) d.dtype |= 0x100;
        }
        if (s.op == UCL_EPI_CLAMP && !(s.p0 <= s.p1))
            return fail(UCL_ERR_INVALID_ARG, "epilogue step %d: clamp(min=%g, max=%g) has min > max", i, s.p0, s.p1);
    }
    kp.n_steps = epi->n_steps;
    // Recognise  [scale] [bias | row_broadcast] [aux_load] [one activation]  in that order.
    FusedEpi f;
    memset(&f, 0, sizeof(f));
    int i = 0;
    const int n = epi->n_steps;
    if (i < n && kp.steps[i].op == UCL_EPI_SCALE) { f.has_scale = 1; f.alpha = kp.steps[i].p0; ++i; }
    if (i < n && (kp.steps[i].op == UCL_EPI_BIAS || kp.steps[i].op == UCL_EPI_ROW_BROADCAST)) {
        f.has_bias = 1; f.bias = kp.steps[i].ptr; f.bias_dt = kp.steps[i].dtype; ++i;
    }
    if (i < n && kp.steps[i].op == UCL_EPI_AUX_LOAD) {
        f.has_res = 1; f.res = kp.steps[i].ptr; f.res_dt = kp.steps[i].dtype; f.beta = kp.steps[i].p0;
        f.res_ld = kp.steps[i].ld; f.res_bs = kp.steps[i].bs; ++i;
    }
    if (i < n) {
        switch (kp.steps[i].op) {
        case UCL_EPI_RELU: case UCL_EPI_GELU_TANH: case UCL_EPI_GELU_ERF: case UCL_EPI_SILU: case UCL_EPI_SIGMOID:
        case UCL_EPI_TANH: case UCL_EPI_MISH: case UCL_EPI_HARDSWISH: case UCL_EPI_LEAKY_RELU: case UCL_EPI_ELU:
        case UCL_EPI_CLAMP:
            f.act = kp.steps[i].op; f.act_p0 = kp.steps[i].p0; f.act_p1 = kp.steps[i].p1; ++i;
            break;
        default:
            break;
        }
    }
    f.enabled = (i == n);
    kp.fused = f;
    return UCL_OK;
}

// Layout of a 16-bit operand from its two strides: *layout = 0 (contiguous along K) or 1
// (contiguous along its M / N extent), *ld = stride of the other dimension.
ucl_status classify(const char *name, const void *ptr, int64_t k_stride, int64_t mn_stride, int64_t mn_extent,
                    int64_t K, int *layout, int64_t *ld) {
    if (!aligned16(ptr))
        return fail(UCL_ERR_UNSUPPORTED, "%s base pointer %p is not 16-byte aligned; 128-bit loads need (alignment * element_size) %% 16 == 0", name, ptr);
    if (k_stride != 1 && mn_stride != 1)
        return fail(UCL_ERR_UNSUPPORTED, "%s has strides (%lld, %lld): one of them must be 1 (RowMajor or ColumnMajor)", name,
                    (long long)mn_stride, (long long)k_stride);
    if (k_stride == 1 && mn_stride == 1 && mn_extent > 1 && K > 1)
        return fail(UCL_ERR_INVALID_ARG, "%s has both strides 1 with both extents > 1: elements would overlap", name);
    if (k_stride == 1 && (mn_stride != 1 || K % 8 == 0)) {
        if (K % 8 != 0)
            return fail(UCL_ERR_UNSUPPORTED, "%s is contiguous along K but K=%lld is not a multiple of 8 (alignment 8 x 2 bytes = 16)", name, (long long)K);
        if (mn_extent > 1) {
            if (mn_stride % 8 != 0)
                return fail(UCL_ERR_UNSUPPORTED, "%s leading stride %lld is not a multiple of 8 elements", name, (long long)mn_stride);
            if (mn_stride < K)
                return fail(UCL_ERR_INVALID_ARG, "%s leading stride %lld is smaller than its contiguous extent K=%lld", name, (long long)mn_stride, (long long)K);
        }
        *layout = 0;
        *ld = mn_extent > 1 ? mn_stride : K;
        return UCL_OK;
    }
    if (mn_extent % 8 != 0)
        return fail(UCL_ERR_UNSUPPORTED, "%s is contiguous along its M/N extent %lld, which is not a multiple of 8", name, (long long)mn_extent);
    if (K > 1) {
        if (k_stride % 8 != 0)
            return fail(UCL_ERR_UNSUPPORTED, "%s leading stride %lld is not a multiple of 8 elements", name, (long long)k_stride);
        if (k_stride < mn_extent)
            return fail(UCL_ERR_INVALID_ARG, "%s leading stride %lld is smaller than its contiguous extent %lld", name, (long long)k_stride, (long long)mn_extent);
    }
    *layout = 1;
    *ld = K > 1 ? k_stride : mn_extent;
    return UCL_OK;
}

ucl_status check_common(int64_t M, int64_t N, int64_t K, int dtA, int dtB, int dtD, const void *A, const void *B,
                        const void *D, bool fp8_ok = false) {
    if (M <= 0 || N <= 0 || K <= 0)
        return fail(UCL_ERR_INVALID_ARG, "extents must be positive, got M=%lld N=%lld K=%lld", (long long)M, (long long)N, (long long)K);
    if (M >= (1ll << 31) || N >= (1ll << 31) || K >= (1ll << 31))
        return fail(UCL_ERR_UNSUPPORTED, "extents must be below 2^31");
    if (!A || !B || !D) return fail(UCL_ERR_INVALID_ARG, "A, B and D must be non-NULL device pointers");
    if (is8(dtA) && dtA == dtB && !fp8_ok)
        return fail(UCL_ERR_UNSUPPORTED, "fp8 inputs are built for gemm, batched_gemm and grouped_gemm");
    if (!(is16(dtA) || is8(dtA)) || dtA != dtB)
        return fail(UCL_ERR_UNSUPPORTED, "inputs must both be bf16, both fp16 or both the same fp8 type (got %s, %s); accumulation is fp32", dtype_name(dtA), dtype_name(dtB));
    if (!valid_dtype(dtD)) return fail(UCL_ERR_INVALID_ARG, "bad output dtype %d", dtD);
    return UCL_OK;
}


// Fill kernel for the counter area of a split-K workspace (a kernel, not a memset node: the call may
// be captured into a HIP graph).  One 128-bit store per thread.
__global__ void zero_words_kernel(uint32_t *w) {
    ((u32x4 *)w)[blockIdx.x * blockDim.x + threadIdx.x] = u32x4{0u, 0u, 0u, 0u};
}

// Parallel split-K, between the two launches of the tile kernel: adds the slices of every partial tile up into
// slice 0, slice 0 first (the same order, starting from +0, as the tile kernel's own loop: the results are
// bit-identical).  A tile kernel that did this itself would have one workgroup per tile read all slices of its
// tile; here every 16 bytes of a tile are a thread's work, so that the whole chip streams the partial tiles.
typedef float f32x4 __attribute__((ext_vector_type(4)));
// (sixteen, then eight slices' loads in flight per thread: what the kernel moves per microsecond is what it has in
// flight; the additions stay in slice order.  V = f32x4, or float where 16-byte words would make too few workgroups
// to occupy the chip: the same additions per element either way.)
template <int U, class V>
__device__ inline void sum_slices(const V *src, int64_t stride, int slices, int &s, V &acc) {
    for (; s + U <= slices; s += U) {
        V v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(src + (s + u) * stride);
#pragma unroll
        for (int u = 0; u < U; ++u) acc += v[u];
    }
}
template <class V>
__device__ inline V sum_slices(const V *src, int64_t stride, int slices) {
    V acc = V();                     // +0 in every element
    int s = 0;
    sum_slices<16>(src, stride, slices, s, acc);
    sum_slices<8>(src, stride, slices, s, acc);
    sum_slices<4>(src, stride, slices, s, acc);      // (left to single loads, 31 slices cost 2 us more than 24)
    sum_slices<2>(src, stride, slices, s, acc);
    sum_slices<1>(src, stride, slices, s, acc);
    return acc;
}
// `slice_stride` = floats per slice, `n` = elements of type V per slice
template <class V>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(float *partials, int64_t slice_stride, int slices, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    constexpr int kPer = sizeof(V) / 4;
    ((V *)partials)[i] = sum_slices((const V *)partials + i, slice_stride / kPer, slices);
}
// Words of 16 bytes per slice below which the reduction runs one float per thread (fewer than two workgroups per CU otherwise).
constexpr int64_t kReduceScalarBelow = 2 * 256 * 256;

// The same reduction for launches whose chain has the form act(alpha * acc + bias[n] + beta * R[m, n]) (any part may be
// missing, the empty chain included): the
// reduction kernel runs the chain on the sums, with the tile kernel's own element-wise functions and in its order of
// operations (so the bits are the same), and stores D; the finishing launch of the tile kernel is not needed.
// A 16-byte word of a partial tile is accumulator (mi, ni) of one lane: four consecutive columns of one row (the
// layout the tile kernel stores: word = (mi * NI + ni) * 256 + thread; thread = wave * 64 + lane, wave = (row half,
// column half) of the tile; row = mi * 16 + lane % 16, column = ni * 16 + 4 * (lane / 16) inside the wave's quarter).
struct ReduceStore {
    float *partials;
    void *D;
    const void *bias, *res;
    int64_t slice_stride, n4, ldd, d_bs, res_ld, res_bs;
    int32_t slices, tile_m, tile_n, M, N, tiles_m, tiles_n, tiles_per_batch, raster;
    int32_t dtD, has_bias, bias_dt, has_res, res_dt, act;
    float alpha, beta, act_p0, act_p1;
};
template <class V>
__global__ __launch_bounds__(256) void splitk_reduce_store_kernel(const ReduceStore a) {
    constexpr int kPer = sizeof(V) / 4;                // 4: a thread per 16-byte word, 1: a thread per element
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= a.n4 * (4 / kPer)) return;
    const V acc = sum_slices((const V *)a.partials + j, a.slice_stride / kPer, a.slices);
    const int64_t i = kPer == 4 ? j : j >> 2;          // the 16-byte word
    const int e0 = kPer == 4 ? 0 : (int)(j & 3);       // the thread's (first) element in it
    const int words_per_tile = a.tile_m * a.tile_n / 4, ni_count = a.tile_n / 32;
    int t = (int)(i / words_per_tile);
    const int w = (int)(i - (int64_t)t * words_per_tile);
    const int reg = w >> 8, thread = w & 255, wave = thread >> 6, lane = thread & 63;
    const int m_loc = (wave >> 1) * (a.tile_m / 2) + (reg / ni_count) * 16 + (lane & 15);
    const int n_loc = (wave & 1) * (a.tile_n / 2) + (reg % ni_count) * 16 + 4 * (lane >> 4);
    const int batch = t / a.tiles_per_batch;
    t -= batch * a.tiles_per_batch;
    int tm, tn;
    band_raster(t, a.tiles_m, a.tiles_n, a.raster, tm, tn);
    const int m = tm * a.tile_m + m_loc, n = tn * a.tile_n + n_loc + e0;
    if (m >= a.M || n >= a.N) return;
    const int nvalid = a.N - n < kPer ? a.N - n : kPer;
    float x[kPer];
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
        float b = 0.f;
        if (a.has_bias && e < nvalid)
            b = a.bias_dt == UCL_F32 ? ((const float *)a.bias)[n + e] : bits_to_f32(((const uint16_t *)a.bias)[n + e], a.bias_dt);
        float s;
        if constexpr (kPer == 4) s = acc[e]; else s = acc;
        x[e] = s * a.alpha + b;
    }
    if (a.has_res) {
        const int64_t rat = (int64_t)batch * a.res_bs + (int64_t)m * a.res_ld + n;
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
            float r = 0.f;
            if (e < nvalid)
                r = a.res_dt == UCL_F32 ? ((const float *)a.res)[rat + e] : bits_to_f32(((const uint16_t *)a.res)[rat + e], a.res_dt);
            x[e] += a.beta * r;
        }
    }
    switch (a.act) {
#define UCL_ACT_CASE(OP)                                                                                      \
    case OP:                                                                                                  \
        _Pragma("unroll") for (int e = 0; e < kPer; ++e) x[e] = act_f32<OP>(x[e], a.act_p0, a.act_p1);         \
        break;
        UCL_ACT_CASE(UCL_EPI_RELU)
        UCL_ACT_CASE(UCL_EPI_GELU_TANH)
        UCL_ACT_CASE(UCL_EPI_GELU_ERF)
        UCL_ACT_CASE(UCL_EPI_SILU)
        UCL_ACT_CASE(UCL_EPI_SIGMOID)
        UCL_ACT_CASE(UCL_EPI_TANH)
        UCL_ACT_CASE(UCL_EPI_MISH)
        UCL_ACT_CASE(UCL_EPI_HARDSWISH)
        UCL_ACT_CASE(UCL_EPI_LEAKY_RELU)
        UCL_ACT_CASE(UCL_EPI_ELU)
        UCL_ACT_CASE(UCL_EPI_CLAMP)
#undef UCL_ACT_CASE
    default: break;
    }
    const int64_t at = (int64_t)batch * a.d_bs + (int64_t)m * a.ldd + n;
    if (a.dtD == UCL_F32) {
        float *dst = (float *)a.D + at;
        if constexpr (kPer == 4) {
            if (nvalid == 4) {
                *(f32x4 *)dst = f32x4{x[0], x[1], x[2], x[3]};
                return;
            }
        }
#pragma unroll
        for (int e = 0; e < kPer; ++e)
            if (e < nvalid) dst[e] = x[e];
    } else {
        uint16_t *dst = (uint16_t *)a.D + at;
        uint32_t bits[kPer];
#pragma unroll
        for (int e = 0; e < kPer; ++e) bits[e] = f32_to_bits16(x[e], a.dtD);
        if constexpr (kPer == 4) {
            if (nvalid == 4) {
                typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                *(u32x2 *)dst = u32x2{bits[0] | (bits[1] << 16), bits[2] | (bits[3] << 16)};
                return;
            }
        }
#pragma unroll
        for (int e = 0; e < kPer; ++e)
            if (e < nvalid) dst[e] = (uint16_t)bits[e];
    }
}

// Adds up the slices of wgrad_taps_kernel, slice 0 first, and stores the gradient (the same order of elements).
template <class V>
__global__ __launch_bounds__(256) void wgrad_taps_reduce_kernel(const float *partials, void *dw, int64_t n, int slices, int32_t dtD, float alpha) {
    constexpr int kPer = sizeof(V) / 4;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n / kPer) return;
    const V acc = sum_slices((const V *)partials + i, n / kPer, slices);
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
        float x;
        if constexpr (kPer == 4) x = acc[e]; else x = acc;
        x *= alpha;
        if (dtD == UCL_F32) ((float *)dw)[i * kPer + e] = x;
        else ((uint16_t *)dw)[i * kPer + e] = (uint16_t)f32_to_bits16(x, dtD);
    }
}

// split-K plan of a launch: slices (1 = none), K extent per slice, workspace bytes.
struct SplitPlan {
    int slices = 1;
    int k_per_slice = 0;
    int64_t bytes = 0;
    // stream-K: 64-wide k steps per tile, iterations per workgroup, workgroups (0: not a stream-K launch)
    int sk_ipt = 0, sk_q = 0, sk_rounds = 0, sk_grid = 0, sk_deal = 0;
};

ucl_status plan_split(const Launch &L, const VariantDesc &v, const ucl_tuning *tune, const SplitChoice &choice, int64_t total_tiles, SplitPlan &sp) {
    sp = SplitPlan();
    if (!tune) return UCL_OK;
    if (tune->scheduler < UCL_SCHED_DEFAULT || tune->scheduler > UCL_SCHED_STREAM_K)
        return fail(UCL_ERR_INVALID_ARG, "scheduler=%d is not a ucl_tile_scheduler", tune->scheduler);
    if (tune->scheduler == UCL_SCHED_STREAM_K) {
        // every workgroup of a resident grid takes an equal run of (tile, 64-wide k range) iterations; a workgroup
        // leaves at most two parts of tiles in the workspace (two slots per workgroup behind the counters)
        if (tune->split_k_mode != UCL_SPLIT_K_NONE)
            return fail(UCL_ERR_UNSUPPORTED, "split-K and the stream_k scheduler cannot be combined");
        if (total_tiles > UCL_SPLIT_K_MAX_TILES)
            return fail(UCL_ERR_UNSUPPORTED, "the stream_k scheduler serves at most %d output tiles (this problem has %lld)", UCL_SPLIT_K_MAX_TILES, (long long)total_tiles);
        const int64_t ipt = (L.K + 63) / 64, all = total_tiles * ipt;
        if (all >= (1ll << 31)) return fail(UCL_ERR_UNSUPPORTED, "tiles x k steps exceeds 2^31");
        if (all == 0) return UCL_OK;
        // whole rounds of tiles go one tile per workgroup and round; the k steps of the tiles that are left are
        // dealt out evenly.  Fewer tiles than CU slots: no whole round, and only as many workgroups as it takes.
        const int64_t slots = (int64_t)kNumCUs * v.resident();
        int64_t grid = slots, rounds = total_tiles / slots;
        int64_t rest = (total_tiles - rounds * grid) * ipt, q = (rest + grid - 1) / grid;
        if (rounds == 0) {
            // (one workgroup per CU at most, or per tile if there are more tiles than CUs)
            if (grid > kNumCUs) grid = total_tiles > kNumCUs ? total_tiles : kNumCUs;
            if (grid > rest) grid = rest;
            q = (rest + grid - 1) / grid;
            // The workgroup that ends a tile reads the tile's other parts back one after the other, which costs it
            // about r k steps' time per part (measured: 1 for 64x64 tiles, whose parts are loaded several at a time,
            // 9 for 128x128); a run of q steps and ipt / q parts to add make q = sqrt(r ipt) the shortest path
            // through a tile.
            const double r = (int64_t)v.tile_m * v.tile_n >= 128 * 128 ? 9.0 : 1.0;
            const int64_t q_path = (int64_t)(sqrt(r * (double)ipt) + 0.5);
            if (q < q_path) q = q_path;
            if (q < 4) q = 4;
            if (q > ipt) q = ipt;
            // (a slightly longer run that divides the k steps of a tile: the runs can then be dealt k range by k range)
            for (int64_t d = q; d <= q + q / 4; ++d)
                if (ipt % d == 0) { q = d; break; }
            grid = (rest + q - 1) / q;
        }
        if (q > 0 && ipt % q == 0 && (total_tiles - rounds * grid) * (ipt / q) <= grid) sp.sk_deal = (int)(total_tiles - rounds * grid);
        sp.sk_ipt = (int)ipt;
        sp.sk_q = (int)q;
        sp.sk_rounds = (int)rounds;
        sp.sk_grid = (int)grid;
        sp.slices = q ? (int)((ipt + q - 2) / q + 1) : 1;    // parts a tile can fall into, at most
        if (sp.slices > ipt) sp.slices = (int)ipt;
        sp.bytes = UCL_WORKSPACE_COUNTER_BYTES + (int64_t)sp.sk_grid * 2 * v.tile_m * v.tile_n * 4;
        return UCL_OK;
    }
    if (tune->split_k_mode < UCL_SPLIT_K_NONE || tune->split_k_mode > UCL_SPLIT_K_PARALLEL)
        return fail(UCL_ERR_INVALID_ARG, "split_k_mode=%d is not a ucl_split_k_mode", tune->split_k_mode);
    if (tune->split_k_slices < 0) return fail(UCL_ERR_INVALID_ARG, "split_k_slices=%d must be >= 0", tune->split_k_slices);
    if (tune->split_k_mode == UCL_SPLIT_K_NONE) {
        if (tune->split_k_slices > 1)
            return fail(UCL_ERR_INVALID_ARG, "split_k_slices=%d with split_k_mode none: name serial or parallel", tune->split_k_slices);
        return UCL_OK;
    }
    if (L.mode != 0 && L.mode != 4) return fail(UCL_ERR_UNSUPPORTED, "split-K is built for gemm, batched_gemm and conv2d_wgrad");
    if (tune->scheduler == UCL_SCHED_PERSISTENT)
        return fail(UCL_ERR_UNSUPPORTED, "split-K and the persistent scheduler cannot be combined");
    sp.slices = choice.slices;
    sp.k_per_slice = choice.k_per_slice;
    if (sp.slices <= 1) { sp = SplitPlan(); return UCL_OK; }
    if (total_tiles > UCL_SPLIT_K_MAX_TILES)
        return fail(UCL_ERR_UNSUPPORTED, "split-K serves at most %d output tiles (this problem has %lld)", UCL_SPLIT_K_MAX_TILES, (long long)total_tiles);
    if (total_tiles * sp.slices >= (1ll << 31)) return fail(UCL_ERR_UNSUPPORTED, "tiles x slices exceeds the grid limit");
    sp.bytes = UCL_WORKSPACE_COUNTER_BYTES + (int64_t)sp.slices * total_tiles * v.tile_m * v.tile_n * 4;
    return UCL_OK;
}

ucl_status run_taps(const Launch &L, KParams &kp, const TapsChoice &c, void *workspace, void *stream) {
    kp.split_k = c.slices;
    kp.k_per_slice = c.px_per_slice;
    kp.ws_partials = c.slices > 1 ? (float *)((char *)workspace + UCL_WORKSPACE_COUNTER_BYTES) : nullptr;
    hipError_t e = variants_wgrad_taps().v[L.dt].launch(kp, nullptr, (int)((L.M + 63) / 64 * ((L.cC + 31) / 32) * c.slices), (hipStream_t)stream);
    if (e == hipSuccess && c.slices > 1) {
        const int64_t n = L.M * L.N, n4 = n / 4;
        const float alpha = kp.fused.has_scale ? kp.fused.alpha : 1.f;
        if (n4 < kReduceScalarBelow)
            hipLaunchKernelGGL(wgrad_taps_reduce_kernel<float>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, kp.ws_partials, kp.D, n, c.slices, kp.dtD, alpha);
        else
            hipLaunchKernelGGL(wgrad_taps_reduce_kernel<f32x4>, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, (hipStream_t)stream, kp.ws_partials, kp.D, n, c.slices, kp.dtD, alpha);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return fail(UCL_ERR_LAUNCH, "kernel launch failed: %s", hipGetErrorString(e));
    return UCL_OK;
}

ucl_status run(Launch L, KParams &kp, const ucl_tuning *tune, void *stream, bool clear_counters = false) {
    L.lda = kp.lda; L.ldb = kp.ldb;
    L.f32_results = L.dtD == UCL_F32;
    for (int i = 0; i < kp.n_steps; ++i) L.f32_results = L.f32_results || (kp.steps[i].op == UCL_EPI_AUX_STORE && (kp.steps[i].dtype & 0xff) == UCL_F32);
    if (tune && (tune->iterator < 0 || tune->iterator > UCL_ITER_FIXED_STRIDE_DILATION))
        return fail(UCL_ERR_INVALID_ARG, "iterator=%d is not a ucl_conv_iterator", tune->iterator);
    // (the GEMM entry points ignore the iterator)
    if (tune && (L.mode == 2 || L.mode == 3) && tune->iterator == UCL_ITER_FIXED_STRIDE_DILATION && !L.patch_c)
        return fail(UCL_ERR_UNSUPPORTED, "the fixed_stride_dilation iterator serves a 3x3 filter with unit stride and dilation, pad 1 and W <= 58: conv2d_fprop with 64 or 128 input channels, conv2d_dgrad with 64 or 128 output channels");
    SplitChoice choice;
    const VariantDesc *v = select_with_split(L, tune, choice);
    if (!v) {
        if (names_tile(tune)) {
            if (tune->tile_k != 32 && tune->tile_k != 64)
                return fail(UCL_ERR_UNSUPPORTED, "tile_k=%d: the built kernels stage K in steps of 32 or 64", tune->tile_k);
            const int64_t lds = (int64_t)(tune->tile_m + tune->tile_n) * tune->tile_k * 2 * tune->stages;
            if (lds > kLdsBytesPerCU)
                return fail(UCL_ERR_WORKSPACE, "tile %dx%dx%d with %d stages needs %lld bytes of LDS; a CU has %d",
                            tune->tile_m, tune->tile_n, tune->tile_k, tune->stages, (long long)lds, kLdsBytesPerCU);
            return fail(UCL_ERR_UNSUPPORTED, "no kernel built for tile %dx%dx%d, %d stages with these types/layouts; see ucl_variant()",
                        tune->tile_m, tune->tile_n, tune->tile_k, tune->stages);
        }
        if (tune && tune->scheduler == UCL_SCHED_PERSISTENT)
            return fail(UCL_ERR_UNSUPPORTED, "no kernel with the persistent tile scheduler is built for this combination of operation, input type and layouts");
        if (tune && tune->scheduler == UCL_SCHED_STREAM_K)
            return fail(UCL_ERR_UNSUPPORTED, "no kernel with the stream_k tile scheduler is built for this combination of operation, input type and layouts (gemm / batched_gemm, 16-bit inputs contiguous along K)");
        return fail(UCL_ERR_UNSUPPORTED, "no kernel built for this combination of operation, input type and layouts");
    }
    if (kp.ldd > kMaxWideLd) kp.d_vec = 0;
    int raster = tune ? tune->raster : 0;
    if (raster < 0 || raster > 64) return fail(UCL_ERR_INVALID_ARG, "raster=%d must be in 0..64", raster);
    if (raster == 0) raster = default_raster(*v, L);
    kp.raster = raster;
    kp.tiles_n = (int32_t)((L.N + v->tile_n - 1) / v->tile_n);
    GroupTable gt;
    int64_t total;
    if (L.mode == 1) {
        int64_t acc = 0;
        for (int g = 0; g < L.groups; ++g) {
            gt.m[g] = (int32_t)L.M_g[g];
            gt.tile_start[g] = (int32_t)acc;
            acc += (L.M_g[g] + v->tile_m - 1) / v->tile_m * kp.tiles_n;
        }
        for (int g = L.groups; g <= UCL_MAX_GROUPS; ++g) gt.tile_start[g] = (int32_t)acc;
        for (int g = L.groups; g < UCL_MAX_GROUPS; ++g) gt.m[g] = 0;
        total = acc;
        kp.tiles_m = 0;
        kp.tiles_per_batch = 0;
    } else {
        kp.tiles_m = (int32_t)((L.M + v->tile_m - 1) / v->tile_m);
        kp.tiles_per_batch = kp.tiles_m * kp.tiles_n;
        total = L.mode == 3 ? count_tiles(L, v->tile_m, v->tile_n) : (int64_t)kp.tiles_per_batch * L.batch;
    }
    if (total >= (1ll << 31)) return fail(UCL_ERR_UNSUPPORTED, "problem needs %lld tiles; the grid is limited to 2^31-1", (long long)total);
    SplitPlan sp;
    if (ucl_status st = plan_split(L, *v, tune, choice, total, sp)) return st;
    if (sp.sk_grid > 0) {
        if (!tune->workspace)
            return fail(UCL_ERR_WORKSPACE, "the stream_k scheduler needs a workspace of %lld bytes (ucl_workspace_size); tune->workspace is NULL", (long long)sp.bytes);
        if (!aligned16(tune->workspace)) return fail(UCL_ERR_WORKSPACE, "the workspace must be 16-byte aligned");
        if (tune->workspace_bytes < sp.bytes)
            return fail(UCL_ERR_WORKSPACE, "the stream_k scheduler with %d workgroups and tiles of %dx%d needs %lld bytes of workspace, got %lld",
                        sp.sk_grid, v->tile_m, v->tile_n, (long long)sp.bytes, (long long)tune->workspace_bytes);
        kp.sk_ipt = sp.sk_ipt;
        kp.sk_q = sp.sk_q;
        kp.sk_deal = sp.sk_deal;
        kp.sk_rounds = sp.sk_rounds;
        kp.ws_counters = (uint32_t *)tune->workspace;
        kp.ws_partials = (float *)((char *)tune->workspace + UCL_WORKSPACE_COUNTER_BYTES);
    } else if (sp.slices > 1) {
        if (!tune->workspace)
            return fail(UCL_ERR_WORKSPACE, "split-K with %d slices needs a workspace of %lld bytes (ucl_workspace_size); tune->workspace is NULL", sp.slices, (long long)sp.bytes);
        if (!aligned16(tune->workspace)) return fail(UCL_ERR_WORKSPACE, "the split-K workspace must be 16-byte aligned");
        if (tune->workspace_bytes < sp.bytes)
            return fail(UCL_ERR_WORKSPACE, "split-K with %d slices over %lld tiles of %dx%d needs %lld bytes of workspace, got %lld",
                        sp.slices, (long long)total, v->tile_m, v->tile_n, (long long)sp.bytes, (long long)tune->workspace_bytes);
        kp.split_k = sp.slices;
        kp.k_per_slice = sp.k_per_slice;
        kp.ws_counters = (uint32_t *)tune->workspace;
        kp.ws_partials = (float *)((char *)tune->workspace + UCL_WORKSPACE_COUNTER_BYTES);
    }
    if (v->la == 0 && !panel_fits(v->tile_m, kp.lda, L.K))
        return fail(UCL_ERR_UNSUPPORTED, "A leading stride %lld too large: a %d-row panel must span less than 2 GiB", (long long)kp.lda, v->tile_m);
    if (v->lb == 0 && !panel_fits(v->tile_n, kp.ldb, L.K))
        return fail(UCL_ERR_UNSUPPORTED, "B leading stride %lld too large: a %d-row panel must span less than 2 GiB", (long long)kp.ldb, v->tile_n);
    kp.total_tiles = (int32_t)total;
    if (serves_taps(L, kp, tune) && aligned16(kp.D)) {
        const TapsChoice taps = choose_taps(L, *v, choice);
        if (taps.slices == 1 || (taps.slices > 1 && tune->workspace && aligned16(tune->workspace) && taps_bytes(L, taps) <= tune->workspace_bytes))
            return run_taps(L, kp, taps, tune->workspace, stream);
    }
    if (L.held_stride) {
        const HeldPlan h = plan_held(L, kp, tune, *v);
        if (h.R > 0) {
            const hipError_t e = (L.dt == 0 ? variants_conv_held_bf16() : variants_conv_held_f16()).v->launch_held(L.mode, h, kp, (hipStream_t)stream);
            if (e != hipSuccess) return fail(UCL_ERR_LAUNCH, "kernel launch failed: %s", hipGetErrorString(e));
            return UCL_OK;
        }
    }
    if (total == 0) return UCL_OK;     // grouped with every M_g == 0: nothing to do
    const GroupTable *gtp = L.mode == 1 ? &gt : nullptr;
    hipError_t e;
    if (sp.sk_grid > 0) {
        if (clear_counters) {
            hipLaunchKernelGGL(zero_words_kernel, dim3(UCL_WORKSPACE_COUNTER_BYTES / 16 / 256), dim3(256), 0, (hipStream_t)stream,
                               (uint32_t *)tune->workspace);
            e = hipGetLastError();
            if (e != hipSuccess) return fail(UCL_ERR_LAUNCH, "kernel launch failed: %s", hipGetErrorString(e));
        }
        e = v->launch(kp, gtp, sp.sk_grid, (hipStream_t)stream);
    } else if (sp.slices > 1 && tune->split_k_mode == UCL_SPLIT_K_PARALLEL) {
        kp.split_phase = 1;
        e = v->launch(kp, gtp, (int)(total * sp.slices), (hipStream_t)stream);
        bool finished = false;
        if (e == hipSuccess && sp.slices > kReduceInTileKernel) {
            // many slices: a launch of its own adds them up with the whole chip, the last launch then finds one slice
            const int64_t slice_floats = total * v->tile_m * v->tile_n, n4 = slice_floats / 4;
            const bool simple = kp.fused.enabled && kp.d_vec && L.mode != 1;
            if (simple) {
                // ... or none: a chain of the form act(alpha * acc + bias[n] + beta * R[m, n]) is run by the reduction kernel on the sums
                ReduceStore rs;
                rs.partials = kp.ws_partials; rs.D = kp.D; rs.bias = kp.fused.bias;
                rs.dtD = kp.dtD; rs.has_bias = kp.fused.has_bias; rs.bias_dt = kp.fused.bias_dt & 0xff; rs.act = kp.fused.act;
                rs.alpha = kp.fused.has_scale ? kp.fused.alpha : 1.f; rs.act_p0 = kp.fused.act_p0; rs.act_p1 = kp.fused.act_p1;
                rs.has_res = kp.fused.has_res; rs.res = kp.fused.res; rs.res_dt = kp.fused.res_dt & 0xff; rs.beta = kp.fused.beta;
                rs.res_ld = kp.fused.res_ld; rs.res_bs = kp.fused.res_bs;
                rs.slice_stride = slice_floats; rs.n4 = n4; rs.ldd = kp.ldd; rs.d_bs = kp.d_bs;
                rs.slices = sp.slices; rs.tile_m = v->tile_m; rs.tile_n = v->tile_n; rs.M = kp.M; rs.N = kp.N;
                rs.tiles_m = kp.tiles_m; rs.tiles_n = kp.tiles_n; rs.tiles_per_batch = kp.tiles_per_batch; rs.raster = kp.raster;
                if (n4 < kReduceScalarBelow)
                    hipLaunchKernelGGL(splitk_reduce_store_kernel<float>, dim3((unsigned)((slice_floats + 255) / 256)), dim3(256), 0, (hipStream_t)stream, rs);
                else
                    hipLaunchKernelGGL(splitk_reduce_store_kernel<f32x4>, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, (hipStream_t)stream, rs);
                finished = true;
            } else if (n4 < kReduceScalarBelow) {
                hipLaunchKernelGGL(splitk_reduce_kernel<float>, dim3((unsigned)((slice_floats + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                                   kp.ws_partials, slice_floats, sp.slices, slice_floats);
            } else {
                hipLaunchKernelGGL(splitk_reduce_kernel<f32x4>, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                                   kp.ws_partials, slice_floats, sp.slices, n4);
            }
            e = hipGetLastError();
            kp.split_k = 1;
        }
        if (e == hipSuccess && !finished) {
            kp.split_phase = 2;
            e = v->launch(kp, gtp, (int)total, (hipStream_t)stream);
        }
    } else {
        if (clear_counters && sp.slices > 1) {
            // the static workspace is shared by every call on this GPU: start from zeroed counters whatever
            // an earlier call left behind (a fill kernel, so that the call can be captured into a graph)
            hipLaunchKernelGGL(zero_words_kernel, dim3(UCL_WORKSPACE_COUNTER_BYTES / 16 / 256), dim3(256), 0, (hipStream_t)stream,
                               (uint32_t *)tune->workspace);
            e = hipGetLastError();
            if (e != hipSuccess) return fail(UCL_ERR_LAUNCH, "kernel launch failed: %s", hipGetErrorString(e));
        }
        int64_t grid = total * sp.slices;
        if (v->persistent) {
            // one workgroup per CU slot; a multiple of 8 keeps each workgroup on the tile run of its XCD
            // (as many as the compiled kernel's registers and LDS let a CU hold, so that the whole grid is resident)
            const int64_t slots = (int64_t)kNumCUs * v->resident();
            if (grid > slots) grid = slots;
        }
        e = v->launch(kp, gtp, (int)grid, (hipStream_t)stream);
    }
    if (e != hipSuccess) return fail(UCL_ERR_LAUNCH, "kernel launch failed: %s", hipGetErrorString(e));
    return UCL_OK;
}

ucl_status gemm_like(int64_t batch, int64_t M, int64_t N, int64_t K,
                     const void *A, int dtA, int64_t a_rs, int64_t a_cs, int64_t a_bs,
                     const void *B, int dtB, int64_t b_rs, int64_t b_cs, int64_t b_bs,
                     void *D, int dtD, int64_t d_rs, int64_t d_cs, int64_t d_bs,
                     const ucl_epilogue *epi, const ucl_tuning *tune, void *stream, bool clear_counters = false) {
    g_err[0] = 0;
    if (batch <= 0) return fail(UCL_ERR_INVALID_ARG, "batch=%lld must be positive", (long long)batch);
    if (ucl_status st = check_common(M, N, K, dtA, dtB, dtD, A, B, D, /*fp8_ok=*/true)) return st;
    if (is8(dtA)) {
        // 8-bit inputs are handled as pairs of elements: from here on K and the strides of A and B count
        // 16-bit units, which the checks below require to be 16-byte aligned like those of 16-bit inputs
        if (a_cs != 1 || b_rs != 1)
            return fail(UCL_ERR_UNSUPPORTED, "fp8 inputs must both be contiguous along K (A row-major, B column-major)");
        if (K % 16 || (M > 1 && a_rs % 16) || (N > 1 && b_cs % 16) || (batch > 1 && (a_bs % 16 || b_bs % 16)))
            return fail(UCL_ERR_UNSUPPORTED, "fp8 inputs: K=%lld, the leading strides (%lld, %lld) and the batch strides must be multiples of 16 (alignment 16 x 1 byte = 16)",
                        (long long)K, (long long)a_rs, (long long)b_cs);
        K /= 2; a_rs /= 2; b_cs /= 2; a_bs /= 2; b_bs /= 2;
    }
    if (d_cs != 1)
        return fail(UCL_ERR_UNSUPPORTED, "D must be row-major (d_cs == 1, got %lld); for a column-major D swap the operands' roles: (A.B)^T = B^T.A^T", (long long)d_cs);
    if (d_rs < N && M > 1) return fail(UCL_ERR_INVALID_ARG, "d_rs=%lld is smaller than N=%lld", (long long)d_rs, (long long)N);
    if (batch > 1 && ((a_bs % 8) || (b_bs % 8)))
        return fail(UCL_ERR_UNSUPPORTED, "batch strides of A and B must be multiples of 8 elements (16-byte alignment of every batch)");
    Launch L;
    L.mode = 0; L.batch = batch; L.M = M; L.N = N; L.K = K; L.dt = dt_code(dtA); L.dtD = dtD;
    KParams kp;
    memset(&kp, 0, sizeof(kp));
    if (ucl_status st = classify("A", A, a_cs, a_rs, M, K, &L.la, &kp.lda)) return st;
    if (ucl_status st = classify("B", B, b_rs, b_cs, N, K, &L.lb, &kp.ldb)) return st;
    // direct copies of an N-contiguous B address it with 32-bit byte offsets from the start of a batch
    L.ndirect_ok = L.lb == 1 && ((K - 1) * kp.ldb + N) * 2 < (1ll << 31);
    L.mdirect_ok = L.la == 1 && ((K - 1) * kp.lda + M) * 2 < (1ll << 31);
    if (ucl_status st = check_epilogue(epi, L, kp)) return st;
    kp.A = A; kp.B = B; kp.D = D;
    kp.ldd = d_rs; kp.a_bs = a_bs; kp.b_bs = b_bs; kp.d_bs = d_bs;
    kp.M = (int32_t)M; kp.N = (int32_t)N; kp.K = (int32_t)K;
    kp.dtD = dtD;
    kp.d_vec = aligned16(D) && (d_rs % (16 / elem_size(dtD)) == 0) && (d_bs % (16 / elem_size(dtD)) == 0);
    return run(L, kp, tune, stream, clear_counters);
}

// ---- SOL ---------------------------------------------------------------------------------------

int64_t conv_out(int64_t in, int64_t pad, int64_t dil, int64_t ker, int64_t stride) {
    return (in + 2 * pad - dil * (ker - 1) - 1) / stride + 1;
}

ucl_status characterise(const ucl_problem *p, double *flops, double *bytes, int64_t *M_out, int64_t *N_out) {
    if (!p) return fail(UCL_ERR_INVALID_ARG, "problem is NULL");
    if (!(valid_dtype(p->dt_in) || is8(p->dt_in)) || !valid_dtype(p->dt_out)) return fail(UCL_ERR_INVALID_ARG, "bad dtype in problem");
    const double si = elem_size(p->dt_in), so = elem_size(p->dt_out);
    double rows = 0, N = 0, batch = 1;
    switch (p->op) {
    case UCL_OP_GEMM:
    case UCL_OP_BATCHED_GEMM: {
        batch = p->op == UCL_OP_GEMM ? 1 : (double)p->batch;
        if (p->M <= 0 || p->N <= 0 || p->K <= 0 || batch <= 0) return fail(UCL_ERR_INVALID_ARG, "extents must be positive");
        rows = (double)p->M; N = (double)p->N;
        *flops = 2.0 * batch * p->M * p->N * p->K;
        *bytes = batch * ((double)p->M * p->K + (double)p->K * p->N) * si + batch * (double)p->M * p->N * so;
        break;
    }
    case UCL_OP_GROUPED_GEMM: {
        if (p->groups <= 0 || !p->M_g || p->N <= 0 || p->K <= 0) return fail(UCL_ERR_INVALID_ARG, "grouped problem needs groups > 0, M_g, N, K");
        double sumM = 0;
        for (int g = 0; g < p->groups; ++g) {
            if (p->M_g[g] < 0) return fail(UCL_ERR_INVALID_ARG, "M_g[%d] is negative", g);
            sumM += (double)p->M_g[g];
        }
        rows = sumM; N = (double)p->N;
        *flops = 2.0 * sumM * p->N * p->K;
        // every group's A, B and D once
        *bytes = (sumM * p->K + (double)p->groups * p->K * p->N) * si + sumM * p->N * so;
        break;
    }
    case UCL_OP_CONV2D_FPROP:
    case UCL_OP_CONV2D_DGRAD:
    case UCL_OP_CONV2D_WGRAD: {
        if (p->cN <= 0 || p->cH <= 0 || p->cW <= 0 || p->cC <= 0 || p->cKout <= 0 || p->cR <= 0 || p->cS <= 0 ||
            p->stride_h <= 0 || p->stride_w <= 0 || p->dil_h <= 0 || p->dil_w <= 0 || p->pad_h < 0 || p->pad_w < 0)
            return fail(UCL_ERR_INVALID_ARG, "conv geometry must be positive (pads non-negative)");
        const int64_t P = conv_out(p->cH, p->pad_h, p->dil_h, p->cR, p->stride_h);
        const int64_t Q = conv_out(p->cW, p->pad_w, p->dil_w, p->cS, p->stride_w);
        if (P <= 0 || Q <= 0) return fail(UCL_ERR_INVALID_ARG, "conv output is empty");
        const double n_y = (double)p->cN * P * Q * (double)p->cKout, n_x = (double)p->cN * p->cH * p->cW * p->cC;
        const double n_w = (double)p->cKout * p->cR * p->cS * p->cC;
        // padded taps are counted, as a dense implicit GEMM executes them (the same count in all three directions)
        *flops = 2.0 * n_y * (double)(p->cR * p->cS * p->cC);
        if (p->op == UCL_OP_CONV2D_FPROP) {
            rows = (double)p->cN * P * Q; N = (double)p->cKout;
            *bytes = (n_x + n_w) * si + n_y * so;
        } else if (p->op == UCL_OP_CONV2D_DGRAD) {
            rows = (double)p->cN * p->cH * p->cW; N = (double)p->cC;
            *bytes = (n_y + n_w) * si + n_x * so;
        } else {
            rows = (double)p->cKout; N = (double)(p->cR * p->cS * p->cC);
            *bytes = (n_y + n_x) * si + n_w * so;
        }
        break;
    }
    default:
        return fail(UCL_ERR_INVALID_ARG, "unknown op kind %d", p->op);
    }
    if (p->epi) {
        if (p->epi->n_steps < 0 || p->epi->n_steps > UCL_MAX_EPI_STEPS) return fail(UCL_ERR_INVALID_ARG, "bad epilogue length");
        for (int i = 0; i < p->epi->n_steps; ++i) {
            const ucl_epi_step &s = p->epi->steps[i];
            if (!op_has_tensor(s.op)) continue;
            const double se = elem_size(s.dtype);
            const double groups = p->op == UCL_OP_GROUPED_GEMM ? p->groups : 1;
            if (op_is_matrix(s.op)) *bytes += batch * rows * N * se;
            else if (s.op == UCL_EPI_PER_ROW_SCALE || s.op == UCL_EPI_COL_BROADCAST) *bytes += rows * se;
            else *bytes += groups * N * se;
        }
    }
    if (M_out) *M_out = (int64_t)rows;
    if (N_out) *N_out = (int64_t)N;
    return UCL_OK;
}


// Device address of this GPU's copy of the static workspace, looked up once per device with that
// device current (each GPU holds its own copy at its own address).
constexpr int kMaxDevices = 64;
std::mutex g_static_mu;
void *g_static_ptr[kMaxDevices] = {};

ucl_status static_workspace(void **out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(UCL_ERR_LAUNCH, "hipGetDevice failed: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return fail(UCL_ERR_UNSUPPORTED, "device index %d outside [0, %d)", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_static_mu);
    if (!g_static_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return fail(UCL_ERR_LAUNCH, "hipGetSymbolAddress of the static workspace failed: %s", hipGetErrorString(e));
        g_static_ptr[dev] = ptr;
    }
    *out = g_static_ptr[dev];
    return UCL_OK;
}

// Launch description of a problem given as ucl_problem (packed operands), for the host-only queries.
ucl_status launch_from_problem(const ucl_problem *p, Launch &L) {
    double f, b;
    int64_t M = 0, N = 0;
    if (ucl_status st = characterise(p, &f, &b, &M, &N)) return st;
    if (!is16(p->dt_in) && !is8(p->dt_in)) return fail(UCL_ERR_UNSUPPORTED, "kernels take bf16, fp16 or fp8 inputs");
    if (is8(p->dt_in) && (p->op > UCL_OP_GROUPED_GEMM || p->a_layout != UCL_LAYOUT_K_CONTIGUOUS || p->b_layout != UCL_LAYOUT_K_CONTIGUOUS || p->K % 16))
        return fail(UCL_ERR_UNSUPPORTED, "fp8 inputs are built for gemm, batched_gemm and grouped_gemm with both operands contiguous along K, K a multiple of 16");
    L.mode = p->op == UCL_OP_GROUPED_GEMM ? 1 : p->op == UCL_OP_CONV2D_FPROP ? 2 : p->op == UCL_OP_CONV2D_DGRAD ? 3
             : p->op == UCL_OP_CONV2D_WGRAD ? 4 : 0;
    L.batch = p->op == UCL_OP_BATCHED_GEMM ? p->batch : 1;
    L.M = M; L.N = N;
    L.K = is8(p->dt_in) ? p->K / 2 : p->K;          // 8-bit inputs: the kernels count pairs
    if (L.mode >= 2) {
        const int64_t P = conv_out(p->cH, p->pad_h, p->dil_h, p->cR, p->stride_h), Q = conv_out(p->cW, p->pad_w, p->dil_w, p->cS, p->stride_w);
        L.K = L.mode == 2 ? p->cR * p->cS * p->cC : L.mode == 3 ? p->cR * p->cS * p->cKout : p->cN * P * Q;
    }
    L.groups = p->groups; L.M_g = p->M_g;
    if (L.mode == 2) {
        L.la = 2; L.lb = 0;
    } else if (L.mode == 3) {
        L.la = 2; L.lb = 1; L.ndirect_ok = true;
    } else if (L.mode == 4) {
        L.la = 1; L.lb = 1; L.ndirect_ok = L.mdirect_ok = true;
    } else {
        if ((p->a_layout != UCL_LAYOUT_K_CONTIGUOUS && p->a_layout != UCL_LAYOUT_MN_CONTIGUOUS) ||
            (p->b_layout != UCL_LAYOUT_K_CONTIGUOUS && p->b_layout != UCL_LAYOUT_MN_CONTIGUOUS))
            return fail(UCL_ERR_INVALID_ARG, "a_layout / b_layout must be ucl_operand_layout values");
        if (L.mode == 1 && p->a_layout != UCL_LAYOUT_K_CONTIGUOUS)
            return fail(UCL_ERR_UNSUPPORTED, "grouped_gemm is built for a row-major A");
        L.la = p->a_layout; L.lb = p->b_layout;
        // packed operands: the same reach test for directly copied rows as the launch path applies
        const int64_t Mmax = L.mode == 1 ? 0 : M;
        L.ndirect_ok = L.lb == 1 && ((L.K - 1) * N + N) * 2 < (1ll << 31);
        L.mdirect_ok = L.la == 1 && ((L.K - 1) * Mmax + Mmax) * 2 < (1ll << 31);
    }
    L.dt = dt_code(p->dt_in);
    L.dtD = p->dt_out;
    L.f32_results = L.dtD == UCL_F32;
    for (int i = 0; p->epi && i < p->epi->n_steps; ++i)
        L.f32_results = L.f32_results || (p->epi->steps[i].op == UCL_EPI_AUX_STORE && p->epi->steps[i].dtype == UCL_F32);
    if (L.mode == 4)
        taps_launch(L, p->cN, p->cH, p->cW, p->cC, conv_out(p->cH, p->pad_h, p->dil_h, p->cR, p->stride_h), conv_out(p->cW, p->pad_w, p->dil_w, p->cS, p->stride_w),
                    p->cR, p->cS, p->pad_h, p->pad_w, p->stride_h, p->stride_w, p->dil_h, p->dil_w);
    if (L.mode == 2)
        L.patch_c = conv_patch_channels(p->cW, p->cC, p->cR, p->cS, p->pad_h, p->pad_w, p->stride_h, p->stride_w, p->dil_h, p->dil_w);
    if (L.mode == 3) {
        L.patch_c = conv_patch_channels(p->cW, p->cKout, p->cR, p->cS, p->pad_h, p->pad_w, p->stride_h, p->stride_w, p->dil_h, p->dil_w);
        dgrad_launch(L, p->cN, p->cH, p->cW, p->stride_h, p->stride_w);
    }
    if (L.mode == 2 || L.mode == 3) {
        const int64_t P = conv_out(p->cH, p->pad_h, p->dil_h, p->cR, p->stride_h), Q = conv_out(p->cW, p->pad_w, p->dil_w, p->cS, p->stride_w);
        const bool fwd = L.mode == 2;
        held_launch(L, p->cN, fwd ? p->cH : P, fwd ? p->cW : Q, fwd ? P : p->cH, fwd ? Q : p->cW, fwd ? p->cC : p->cKout, p->cR, p->cS, p->pad_h, p->pad_w,
                    p->stride_h, p->stride_w, p->dil_h, p->dil_w);
    }
    if (L.mode == 1)
        for (int g = 0; g < L.groups; ++g) L.sum_Mg += L.M_g[g];
    return UCL_OK;
}


}  // namespace
}  // namespace ucl

using namespace ucl;

extern "C" {

ucl_status ucl_gemm(int64_t M, int64_t N, int64_t K, const void *A, int32_t dtA, int64_t a_rs, int64_t a_cs,
                    const void *B, int32_t dtB, int64_t b_rs, int64_t b_cs, void *D, int32_t dtD, int64_t d_rs,
                    int64_t d_cs, const ucl_epilogue *epi, const ucl_tuning *tune, void *stream) {
    return gemm_like(1, M, N, K, A, dtA, a_rs, a_cs, 0, B, dtB, b_rs, b_cs, 0, D, dtD, d_rs, d_cs, 0, epi, tune, stream);
}

ucl_status ucl_gemm_static_workspace(int64_t M, int64_t N, int64_t K, const void *A, int32_t dtA, int64_t a_rs, int64_t a_cs,
                                     const void *B, int32_t dtB, int64_t b_rs, int64_t b_cs, void *D, int32_t dtD, int64_t d_rs,
                                     int64_t d_cs, const ucl_epilogue *epi, const ucl_tuning *tune, void *stream) {
    g_err[0] = 0;
    if (!tune || tune->split_k_mode == UCL_SPLIT_K_NONE)
        return fail(UCL_ERR_INVALID_ARG, "ucl_gemm_static_workspace is the split-K form of ucl_gemm: tune must name split_k_mode serial or parallel");
    void *ws = nullptr;
    if (ucl_status st = static_workspace(&ws)) return st;
    ucl_tuning t = *tune;
    t.workspace = ws;                       // (the device address, never the array's name)
    t.workspace_bytes = UCL_STATIC_WORKSPACE_BYTES;
    const ucl_status st = gemm_like(1, M, N, K, A, dtA, a_rs, a_cs, 0, B, dtB, b_rs, b_cs, 0, D, dtD, d_rs, d_cs, 0, epi, &t, stream,
                                    /*clear_counters=*/t.split_k_mode == UCL_SPLIT_K_SERIAL);
    if (st == UCL_ERR_WORKSPACE) {
        // say which limit was hit: the message of the general path speaks of the caller's workspace
        char detail[384];
        snprintf(detail, sizeof(detail), "%s", g_err);
        return fail(UCL_ERR_WORKSPACE, "the static workspace holds %lld bytes: %s (use fewer slices, or ucl_gemm with a workspace of your own)",
                    (long long)UCL_STATIC_WORKSPACE_BYTES, detail);
    }
    return st;
}

ucl_status ucl_batched_gemm(int64_t batch, int64_t M, int64_t N, int64_t K, const void *A, int32_t dtA, int64_t a_rs,
                            int64_t a_cs, int64_t a_bs, const void *B, int32_t dtB, int64_t b_rs, int64_t b_cs,
                            int64_t b_bs, void *D, int32_t dtD, int64_t d_rs, int64_t d_cs, int64_t d_bs,
                            const ucl_epilogue *epi, const ucl_tuning *tune, void *stream) {
    return gemm_like(batch, M, N, K, A, dtA, a_rs, a_cs, a_bs, B, dtB, b_rs, b_cs, b_bs, D, dtD, d_rs, d_cs, d_bs, epi,
                     tune, stream);
}

ucl_status ucl_grouped_gemm(int32_t groups, const int64_t *M_g, int64_t N, int64_t K, const void *const *A_g,
                            int32_t dtA, int64_t a_rs, int64_t a_cs, const void *const *B_g, int32_t dtB, int64_t b_rs,
                            int64_t b_cs, void *const *D_g, int32_t dtD, int64_t d_rs, int64_t d_cs,
                            const ucl_epilogue *epi, const ucl_tuning *tune, void *stream) {
    g_err[0] = 0;
    if (groups <= 0 || groups > UCL_MAX_GROUPS)
        return fail(UCL_ERR_INVALID_ARG, "groups=%d must be in 1..%d", groups, UCL_MAX_GROUPS);
    if (!M_g) return fail(UCL_ERR_INVALID_ARG, "M_g (host array of group sizes) is NULL");
    Launch L;
    L.mode = 1; L.groups = groups; L.M_g = M_g; L.N = N; L.K = K; L.dt = dt_code(dtA); L.dtD = dtD;
    for (int g = 0; g < groups; ++g) {
        if (M_g[g] < 0 || M_g[g] >= (1ll << 31)) return fail(UCL_ERR_INVALID_ARG, "M_g[%d]=%lld must be in [0, 2^31)", g, (long long)M_g[g]);
        L.sum_Mg += M_g[g];
    }
    if (ucl_status st = check_common(1, N, K, dtA, dtB, dtD, A_g, B_g, D_g, /*fp8_ok=*/true)) return st;
    if (a_cs != 1 || (b_rs != 1 && b_cs != 1))
        return fail(UCL_ERR_UNSUPPORTED, "grouped_gemm is built for A row-major (a_cs == 1) and B column-major (b_rs == 1) or row-major (b_cs == 1)");
    const bool b_row = b_rs != 1;             // B[k*b_rs + n]: contiguous along N
    int64_t ldb = b_row ? b_rs : b_cs;
    if (is8(dtA)) {
        // 8-bit inputs are handled as pairs of elements (see gemm_like): K and the leading strides count 16-bit units below
        if (b_row) return fail(UCL_ERR_UNSUPPORTED, "fp8 inputs must both be contiguous along K (A row-major, B column-major)");
        if (K % 16 || a_rs % 16 || ldb % 16)
            return fail(UCL_ERR_UNSUPPORTED, "fp8 inputs: K=%lld and the leading strides (%lld, %lld) must be multiples of 16 (alignment 16 x 1 byte = 16)",
                        (long long)K, (long long)a_rs, (long long)ldb);
        K /= 2; a_rs /= 2; ldb /= 2;
        L.K = K;
    }
    if (K % 8 || a_rs % 8 || ldb % 8 || a_rs < K || ldb < (b_row ? N : K))
        return fail(UCL_ERR_UNSUPPORTED, "K=%lld and the leading strides (%lld, %lld) must be multiples of 8 and at least the contiguous extent", (long long)K, (long long)a_rs, (long long)ldb);
    if (b_row) {
        if (N % 8) return fail(UCL_ERR_UNSUPPORTED, "B is contiguous along N=%lld, which is not a multiple of 8", (long long)N);
        if (((K - 1) * ldb + N) * 2 >= (1ll << 31))
            return fail(UCL_ERR_UNSUPPORTED, "a row-major B of a group must be smaller than 2 GiB (32-bit offsets)");
        L.lb = 1;
        L.ndirect_ok = true;
    }
    if (d_cs != 1 || d_rs < N) return fail(UCL_ERR_UNSUPPORTED, "D must be row-major with d_rs >= N");
    KParams kp;
    memset(&kp, 0, sizeof(kp));
    if (ucl_status st = check_epilogue(epi, L, kp)) return st;
    kp.A_g = A_g; kp.B_g = B_g; kp.D_g = D_g;
    kp.lda = a_rs; kp.ldb = ldb; kp.ldd = d_rs;
    kp.N = (int32_t)N; kp.K = (int32_t)K; kp.groups = groups; kp.dtD = dtD;
    kp.d_vec = d_rs % (16 / elem_size(dtD)) == 0;      // group base pointers are required to be 16-byte aligned
    return run(L, kp, tune, stream);
}

ucl_status ucl_conv2d_fprop(int64_t N, int64_t H, int64_t W, int64_t C, int64_t Kout, int64_t R, int64_t S,
                            int64_t pad_h, int64_t pad_w, int64_t stride_h, int64_t stride_w, int64_t dil_h,
                            int64_t dil_w, const void *x, int32_t dtX, const void *w, int32_t dtW, void *y, int32_t dtY,
                            const ucl_epilogue *epi, const ucl_tuning *tune, void *stream) {
    g_err[0] = 0;
    if (N <= 0 || H <= 0 || W <= 0 || C <= 0 || Kout <= 0 || R <= 0 || S <= 0)
        return fail(UCL_ERR_INVALID_ARG, "conv extents must be positive");
    if (pad_h < 0 || pad_w < 0 || stride_h <= 0 || stride_w <= 0 || dil_h <= 0 || dil_w <= 0)
        return fail(UCL_ERR_INVALID_ARG, "pads must be >= 0, strides and dilations > 0");
    const int64_t P = conv_out(H, pad_h, dil_h, R, stride_h), Q = conv_out(W, pad_w, dil_w, S, stride_w);
    if (P <= 0 || Q <= 0) return fail(UCL_ERR_INVALID_ARG, "conv output is empty (P=%lld, Q=%lld)", (long long)P, (long long)Q);
    const int64_t M = N * P * Q, Kg = R * S * C;
    if (ucl_status st = check_common(M, Kout, Kg, dtX, dtW, dtY, x, w, y)) return st;
    if (C % 8) return fail(UCL_ERR_UNSUPPORTED, "C=%lld must be a multiple of 8 so that a 128-bit load never straddles a filter tap", (long long)C);
    if (!aligned16(x) || !aligned16(w)) return fail(UCL_ERR_UNSUPPORTED, "x and w must be 16-byte aligned");
    if (N * H * W * C * 2 >= (1ll << 31)) return fail(UCL_ERR_UNSUPPORTED, "activation tensor must be smaller than 2 GiB (32-bit offsets)");
    if (H >= (1 << 24) || W >= (1 << 24) || pad_h >= (1 << 24) || pad_w >= (1 << 24))
        return fail(UCL_ERR_UNSUPPORTED, "image extents / pads must be below 2^24");
    Launch L;
    L.mode = 2; L.M = M; L.N = Kout; L.K = Kg; L.la = 2; L.lb = 0; L.dt = dt_code(dtX); L.dtD = dtY;
    L.patch_c = conv_patch_channels(W, C, R, S, pad_h, pad_w, stride_h, stride_w, dil_h, dil_w);
    held_launch(L, N, H, W, P, Q, C, R, S, pad_h, pad_w, stride_h, stride_w, dil_h, dil_w);
    KParams kp;
    memset(&kp, 0, sizeof(kp));
    if (ucl_status st = check_epilogue(epi, L, kp)) return st;
    kp.A = x; kp.B = w; kp.D = y;
    kp.a_bytes = N * H * W * C * 2;
    kp.lda = 0; kp.ldb = Kg; kp.ldd = Kout;
    kp.M = (int32_t)M; kp.N = (int32_t)Kout; kp.K = (int32_t)Kg; kp.dtD = dtY;
    kp.cH = (int32_t)H; kp.cW = (int32_t)W; kp.cC = (int32_t)C; kp.cS = (int32_t)S; kp.cP = (int32_t)P; kp.cQ = (int32_t)Q;
    kp.pad_h = (int32_t)pad_h; kp.pad_w = (int32_t)pad_w; kp.str_h = (int32_t)stride_h; kp.str_w = (int32_t)stride_w;
    kp.dil_h = (int32_t)dil_h; kp.dil_w = (int32_t)dil_w;
    kp.d_vec = aligned16(y) && (Kout % (16 / elem_size(dtY)) == 0);
    if (is_plain_gemm(R, S, pad_h, pad_w, stride_h, stride_w)) {
        const Launch G = gemm_of_conv(L);
        if (takes_gemm(L, G, tune)) {
            kp.lda = C;
            return run(G, kp, tune, stream);
        }
    }
    return run(L, kp, tune, stream);
}

// Shared checks of the two gradient entry points; P, Q of the forward geometry.
static ucl_status conv_grad_common(int64_t N, int64_t H, int64_t W, int64_t C, int64_t Kout, int64_t R, int64_t S,
                                   int64_t pad_h, int64_t pad_w, int64_t stride_h, int64_t stride_w, int64_t dil_h,
                                   int64_t dil_w, int64_t *P, int64_t *Q) {
    if (N <= 0 || H <= 0 || W <= 0 || C <= 0 || Kout <= 0 || R <= 0 || S <= 0)
        return fail(UCL_ERR_INVALID_ARG, "conv extents must be positive");
    if (pad_h < 0 || pad_w < 0 || stride_h <= 0 || stride_w <= 0 || dil_h <= 0 || dil_w <= 0)
        return fail(UCL_ERR_INVALID_ARG, "pads must be >= 0, strides and dilations > 0");
    *P = conv_out(H, pad_h, dil_h, R, stride_h);
    *Q = conv_out(W, pad_w, dil_w, S, stride_w);
    if (*P <= 0 || *Q <= 0) return fail(UCL_ERR_INVALID_ARG, "conv output is empty (P=%lld, Q=%lld)", (long long)*P, (long long)*Q);
    if (C % 8 || Kout % 8)
        return fail(UCL_ERR_UNSUPPORTED, "C=%lld and Kout=%lld must be multiples of 8 so that a 128-bit load never straddles a filter tap or a pixel", (long long)C, (long long)Kout);
    if (N * H * W * C * 2 >= (1ll << 31) || N * *P * *Q * Kout * 2 >= (1ll << 31) || Kout * R * S * C * 2 >= (1ll << 31))
        return fail(UCL_ERR_UNSUPPORTED, "activations, output gradient and filter must each be smaller than 2 GiB (32-bit offsets)");
    if (H >= (1 << 24) || W >= (1 << 24) || pad_h >= (1 << 24) || pad_w >= (1 << 24) || dil_h * R >= (1 << 24) || dil_w * S >= (1 << 24))
        return fail(UCL_ERR_UNSUPPORTED, "image extents, pads and dilated filter extents must be below 2^24");
    return UCL_OK;
}

ucl_status ucl_conv2d_dgrad(int64_t N, int64_t H, int64_t W, int64_t C, int64_t Kout, int64_t R, int64_t S,
                            int64_t pad_h, int64_t pad_w, int64_t stride_h, int64_t stride_w, int64_t dil_h,
                            int64_t dil_w, const void *dy, int32_t dtDy, const void *w, int32_t dtW, void *dx, int32_t dtDx,
                            const ucl_epilogue *epi, const ucl_tuning *tune, void *stream) {
    g_err[0] = 0;
    int64_t P = 0, Q = 0;
    if (ucl_status st = conv_grad_common(N, H, W, C, Kout, R, S, pad_h, pad_w, stride_h, stride_w, dil_h, dil_w, &P, &Q)) return st;
    const int64_t M = N * H * W, Kg = R * S * Kout;
    if (ucl_status st = check_common(M, C, Kg, dtDy, dtW, dtDx, dy, w, dx)) return st;
    if (!aligned16(dy) || !aligned16(w)) return fail(UCL_ERR_UNSUPPORTED, "dy and w must be 16-byte aligned");
    Launch L;
    L.mode = 3; L.M = M; L.N = C; L.K = Kg; L.la = 2; L.lb = 1; L.ndirect_ok = true; L.dt = dt_code(dtDy); L.dtD = dtDx;
    L.patch_c = conv_patch_channels(W, Kout, R, S, pad_h, pad_w, stride_h, stride_w, dil_h, dil_w);
    dgrad_launch(L, N, H, W, stride_h, stride_w);
    held_launch(L, N, P, Q, H, W, Kout, R, S, pad_h, pad_w, stride_h, stride_w, dil_h, dil_w);
    KParams kp;
    memset(&kp, 0, sizeof(kp));
    // (the tiles that take longest start first)
    kp.dg_reverse = dgrad_taps((int)L.str_h - 1, (int)pad_h, (int)dil_h, (int)L.str_h, (int)R).count >
                    dgrad_taps(0, (int)pad_h, (int)dil_h, (int)L.str_h, (int)R).count;
    if (ucl_status st = check_epilogue(epi, L, kp)) return st;
    kp.A = dy; kp.B = w; kp.D = dx;
    kp.a_bytes = N * P * Q * Kout * 2;
    kp.b_bytes = Kout * R * S * C * 2;
    kp.lda = 0; kp.ldb = R * S * C; kp.ldd = C;
    kp.M = (int32_t)M; kp.N = (int32_t)C; kp.K = (int32_t)Kg; kp.dtD = dtDx;
    // the gathered tensor is dy: its extents take the place of the image's, the rows are input pixels
    kp.cH = (int32_t)P; kp.cW = (int32_t)Q; kp.cC = (int32_t)Kout; kp.cS = (int32_t)S; kp.cP = (int32_t)H; kp.cQ = (int32_t)W;
    kp.pad_h = (int32_t)pad_h; kp.pad_w = (int32_t)pad_w; kp.str_h = (int32_t)L.str_h; kp.str_w = (int32_t)L.str_w;
    kp.dil_h = (int32_t)dil_h; kp.dil_w = (int32_t)dil_w;
    kp.d_vec = aligned16(dx) && (C % (16 / elem_size(dtDx)) == 0);
    if (is_plain_gemm(R, S, pad_h, pad_w, stride_h, stride_w)) {
        const Launch G = gemm_of_conv(L);
        if (takes_gemm(L, G, tune)) {
            kp.lda = Kout;
            return run(G, kp, tune, stream);
        }
    }
    return run(L, kp, tune, stream);
}

ucl_status ucl_conv2d_wgrad(int64_t N, int64_t H, int64_t W, int64_t C, int64_t Kout, int64_t R, int64_t S,
                            int64_t pad_h, int64_t pad_w, int64_t stride_h, int64_t stride_w, int64_t dil_h,
                            int64_t dil_w, const void *dy, int32_t dtDy, const void *x, int32_t dtX, void *dw, int32_t dtDw,
                            const ucl_epilogue *epi, const ucl_tuning *tune, void *stream) {
    g_err[0] = 0;
    int64_t P = 0, Q = 0;
    if (ucl_status st = conv_grad_common(N, H, W, C, Kout, R, S, pad_h, pad_w, stride_h, stride_w, dil_h, dil_w, &P, &Q)) return st;
    const int64_t Ng = R * S * C, Kg = N * P * Q;
    if (ucl_status st = check_common(Kout, Ng, Kg, dtDy, dtX, dtDw, dy, x, dw)) return st;
    if (!aligned16(dy) || !aligned16(x)) return fail(UCL_ERR_UNSUPPORTED, "dy and x must be 16-byte aligned");
    Launch L;
    L.mode = 4; L.M = Kout; L.N = Ng; L.K = Kg; L.la = 1; L.lb = 1; L.ndirect_ok = L.mdirect_ok = true;
    L.dt = dt_code(dtDy); L.dtD = dtDw;
    KParams kp;
    memset(&kp, 0, sizeof(kp));
    if (ucl_status st = check_epilogue(epi, L, kp)) return st;
    kp.A = dy; kp.B = x; kp.D = dw;
    kp.b_bytes = N * H * W * C * 2;
    kp.lda = Kout; kp.ldb = 0; kp.ldd = Ng;
    kp.M = (int32_t)Kout; kp.N = (int32_t)Ng; kp.K = (int32_t)Kg; kp.dtD = dtDw;
    kp.cH = (int32_t)H; kp.cW = (int32_t)W; kp.cC = (int32_t)C; kp.cS = (int32_t)S; kp.cP = (int32_t)P; kp.cQ = (int32_t)Q;
    kp.pad_h = (int32_t)pad_h; kp.pad_w = (int32_t)pad_w; kp.str_h = (int32_t)stride_h; kp.str_w = (int32_t)stride_w;
    kp.dil_h = (int32_t)dil_h; kp.dil_w = (int32_t)dil_w;
    kp.d_vec = aligned16(dw) && (Ng % (16 / elem_size(dtDw)) == 0);
    taps_launch(L, N, H, W, C, P, Q, R, S, pad_h, pad_w, stride_h, stride_w, dil_h, dil_w);
    return run(L, kp, tune, stream);
}

ucl_status ucl_transpose(int64_t batch, int64_t rows, int64_t cols, const void *src, int32_t dt_src, void *dst,
                         int32_t dt_dst, void *stream) {
    g_err[0] = 0;
    const ucl_status st = transpose_run(batch, rows, cols, src, dt_src, dst, dt_dst, stream);
    if (st != UCL_OK) return fail(st, "%s", transpose_last_error());
    return UCL_OK;
}

ucl_status ucl_sol_bound(const ucl_problem *p, const ucl_hw *hw, ucl_sol_report *out) {
    g_err[0] = 0;
    if (!out) return fail(UCL_ERR_INVALID_ARG, "report pointer is NULL");
    double flops = 0, bytes = 0;
    if (ucl_status st = characterise(p, &flops, &bytes, nullptr, nullptr)) return st;
    // Hardware limits: published peaks, scaled linearly by the clock ratios.
    ucl_hw mi355x = {2516.6e12, 157.3e12, 8.0e12, 1.0, 1.0, 5033.2e12};
    const ucl_hw &h = hw ? *hw : mi355x;
    if (!(h.peak_bw > 0) || !(h.compute_clock_ratio > 0) || !(h.memory_clock_ratio > 0))
        return fail(UCL_ERR_INVALID_ARG, "hardware descriptor needs positive peaks and clock ratios");
    const double peak = (p->dt_in == UCL_F32 ? h.peak_flops_f32 : is8(p->dt_in) ? h.peak_flops_8bit : h.peak_flops_16bit) * h.compute_clock_ratio;
    if (!(peak > 0)) return fail(UCL_ERR_INVALID_ARG, "hardware descriptor has no compute peak for %s inputs", dtype_name(p->dt_in));
    const double bw = h.peak_bw * h.memory_clock_ratio;
    out->flops = flops;
    out->bytes = bytes;
    out->peak_flops = peak;
    out->peak_bw = bw;
    out->ai = flops / bytes;
    out->ridge = peak / bw;
    out->t_compute = flops / peak;
    out->t_mem = bytes / bw;
    out->t_sol = out->t_compute > out->t_mem ? out->t_compute : out->t_mem;
    out->compute_bound = out->ai >= out->ridge ? 1 : 0;
    out->reserved = 0;
    return UCL_OK;
}

ucl_status ucl_select_tuning(const ucl_problem *p, ucl_tuning *out) {
    g_err[0] = 0;
    if (!out) return fail(UCL_ERR_INVALID_ARG, "output pointer is NULL");
    Launch L;
    if (ucl_status st = launch_from_problem(p, L)) return st;
    if ((L.mode == 2 || L.mode == 3) && is_plain_gemm(p->cR, p->cS, p->pad_h, p->pad_w, p->stride_h, p->stride_w)) {
        const Launch G = gemm_of_conv(L);
        if (takes_gemm(L, G, nullptr)) L = G;
    }
    const VariantDesc *v = select_variant(L, nullptr);
    if (!v) return fail(UCL_ERR_UNSUPPORTED, "no kernel built for this problem");
    memset(out, 0, sizeof(*out));
    out->tile_m = v->tile_m; out->tile_n = v->tile_n; out->tile_k = v->tile_k; out->stages = v->stages;
    out->raster = default_raster(*v, L);
    out->k_groups = v->k_groups;
    out->iterator = v->la == 3 ? UCL_ITER_FIXED_STRIDE_DILATION : v->la == 2 ? UCL_ITER_ANALYTIC : UCL_ITER_DEFAULT;
    return UCL_OK;
}

ucl_status ucl_unnamed_kernel(const ucl_problem *p, const ucl_tuning *tune, int32_t *kernel) {
    g_err[0] = 0;
    if (!kernel) return fail(UCL_ERR_INVALID_ARG, "output pointer is NULL");
    *kernel = UCL_UNNAMED_NONE;
    Launch L;
    if (ucl_status st = launch_from_problem(p, L)) return st;
    if (!L.held_stride && !L.taps_stride) return UCL_OK;
    SplitChoice choice;
    const VariantDesc *v = select_with_split(L, tune, choice, /*sizing=*/true);
    if (!v) return fail(UCL_ERR_UNSUPPORTED, "no kernel built for this problem and tuning; see ucl_variant()");
    ucl_epilogue epi;
    memset(&epi, 0, sizeof(epi));
    if (p->epi) epi = *p->epi;
    for (int i = 0; i < epi.n_steps && i < UCL_MAX_EPI_STEPS; ++i) {
        if (!epi.steps[i].ptr) epi.steps[i].ptr = (const void *)(uintptr_t)16;      // (looked at for its alignment only)
        if (!epi.steps[i].ld) epi.steps[i].ld = L.N;
    }
    KParams kp;
    memset(&kp, 0, sizeof(kp));
    if (ucl_status st = check_epilogue(&epi, L, kp)) return st;
    kp.d_vec = L.N % (16 / elem_size(L.dtD)) == 0;
    if (plan_held(L, kp, tune, *v).R > 0) *kernel = UCL_UNNAMED_CONV_HELD;
    if (serves_taps(L, kp, tune) && choose_taps(L, *v, choice).slices > 0) *kernel = UCL_UNNAMED_WGRAD_TAPS;
    return UCL_OK;
}

ucl_status ucl_workspace_size(const ucl_problem *p, const ucl_tuning *tune, int64_t *bytes, int32_t *slices_out) {
    g_err[0] = 0;
    if (!bytes) return fail(UCL_ERR_INVALID_ARG, "output pointer is NULL");
    *bytes = 0;
    if (slices_out) *slices_out = 1;
    Launch L;
    if (ucl_status st = launch_from_problem(p, L)) return st;
    if (tune && (tune->iterator < 0 || tune->iterator > UCL_ITER_FIXED_STRIDE_DILATION))
        return fail(UCL_ERR_INVALID_ARG, "iterator=%d is not a ucl_conv_iterator", tune->iterator);
    SplitChoice choice;
    const VariantDesc *v = select_with_split(L, tune, choice, /*sizing=*/true);
    if (!v) return fail(UCL_ERR_UNSUPPORTED, "no kernel built for this problem and tuning; see ucl_variant()");
    SplitPlan sp;
    if (ucl_status st = plan_split(L, *v, tune, choice, count_tiles(L, v->tile_m, v->tile_n), sp)) return st;
    *bytes = sp.bytes;
    if (slices_out) *slices_out = sp.slices;
    if (split_left_open(L, tune)) {
        // (strides that the chosen kernel cannot address, or an fp32 tensor stored by a chain that p does not show, leave the
        // call to the general rule: what this answers serves that too)
        const int64_t general = split_bytes(L, general_split(L, tune));
        if (general > *bytes) *bytes = general;
        const bool plain = !p->epi || p->epi->n_steps == 0 || (p->epi->n_steps == 1 && p->epi->steps[0].op == UCL_EPI_SCALE);
        if (L.mode == 4 && takes_taps(L, tune) && plain) {
            const TapsChoice taps = choose_taps(L, *v, choice);
            if (taps.slices > 0 && slices_out) *slices_out = taps.slices;
            if (taps_bytes(L, taps) > *bytes) *bytes = taps_bytes(L, taps);
        }
    }
    return UCL_OK;
}

ucl_status ucl_workspace_init(void *workspace, int64_t workspace_bytes, void *stream) {
    g_err[0] = 0;
    if (!workspace || !aligned16(workspace)) return fail(UCL_ERR_INVALID_ARG, "workspace must be a 16-byte aligned device pointer");
    if (workspace_bytes < UCL_WORKSPACE_COUNTER_BYTES)
        return fail(UCL_ERR_WORKSPACE, "a split-K workspace holds at least its %d bytes of counters, got %lld", UCL_WORKSPACE_COUNTER_BYTES, (long long)workspace_bytes);
    hipLaunchKernelGGL(zero_words_kernel, dim3(UCL_WORKSPACE_COUNTER_BYTES / 16 / 256), dim3(256), 0, (hipStream_t)stream, (uint32_t *)workspace);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(UCL_ERR_LAUNCH, "kernel launch failed: %s", hipGetErrorString(e));
    return UCL_OK;
}

ucl_status ucl_tile_map(int32_t groups, const int32_t *tiles_m, int32_t tiles_n, int32_t raster, int32_t wg,
                        int32_t *group, int32_t *tile_m, int32_t *tile_n) {
    g_err[0] = 0;
    if (groups <= 0 || !tiles_m || tiles_n <= 0 || raster <= 0 || !group || !tile_m || !tile_n)
        return fail(UCL_ERR_INVALID_ARG, "bad arguments to ucl_tile_map");
    std::vector<int32_t> start(groups + 1, 0);
    for (int g = 0; g < groups; ++g) {
        if (tiles_m[g] < 0) return fail(UCL_ERR_INVALID_ARG, "tiles_m[%d] is negative", g);
        start[g + 1] = start[g] + tiles_m[g] * tiles_n;
    }
    const int total = start[groups];
    if (wg < 0 || wg >= total) return fail(UCL_ERR_INVALID_ARG, "wg=%d outside [0, %d)", wg, total);
    int t = xcd_remap(wg, total);
    const int g = find_group(start.data(), groups, t);
    t -= start[g];
    int tm, tn;
    band_raster(t, tiles_m[g], tiles_n, raster, tm, tn);
    *group = g; *tile_m = tm; *tile_n = tn;
    return UCL_OK;
}

// (the few-row kernels come last and are not counted)
int32_t ucl_num_variants(void) {
    const auto &vs = all_variants();
    int32_t n = (int32_t)vs.size();
    while (n > 0 && is_few_row(vs[n - 1])) --n;
    return n;
}

ucl_status ucl_variant(int32_t i, ucl_variant_info *out) {
    const auto &vs = all_variants();
    if (i < 0 || i >= (int)vs.size() || !out) return fail(UCL_ERR_INVALID_ARG, "variant index %d outside [0, %d)", i, (int)vs.size());
    const VariantDesc &v = vs[i];
    memset(out, 0, sizeof(*out));
    out->tile_m = v.tile_m; out->tile_n = v.tile_n; out->tile_k = v.tile_k; out->stages = v.stages;
    out->iterator = v.la == 3 ? UCL_ITER_FIXED_STRIDE_DILATION : v.la == 2 ? UCL_ITER_ANALYTIC : UCL_ITER_DEFAULT;
    out->op_class = v.mode;
    out->dt_in = v.dt == 1 ? UCL_F16 : v.dt == 2 ? UCL_FP8_E4M3 : v.dt == 3 ? UCL_FP8_E5M2 : UCL_BF16;
    out->a_layout = (v.la == 1 || v.la == 5) ? UCL_LAYOUT_MN_CONTIGUOUS : UCL_LAYOUT_K_CONTIGUOUS;
    out->b_layout = (v.lb == 1 || v.lb == 4) ? UCL_LAYOUT_MN_CONTIGUOUS : UCL_LAYOUT_K_CONTIGUOUS;
    out->a_path = v.la; out->b_path = v.lb;
    out->lds_bytes = v.lds_bytes;
    out->patch_channels = v.patch_c;
    out->scheduler = v.persistent == 2 ? UCL_SCHED_STREAM_K : v.persistent ? UCL_SCHED_PERSISTENT : UCL_SCHED_DEFAULT;
    return UCL_OK;
}

int32_t ucl_variant_k_groups(int32_t i) {
    const auto &vs = all_variants();
    return i < 0 || i >= (int)vs.size() ? 0 : vs[i].k_groups;
}

const char *ucl_status_string(ucl_status s) {
    switch (s) {
    case UCL_OK: return "UCL_OK";
    case UCL_ERR_INVALID_ARG: return "UCL_ERR_INVALID_ARG";
    case UCL_ERR_UNSUPPORTED: return "UCL_ERR_UNSUPPORTED";
    case UCL_ERR_WORKSPACE: return "UCL_ERR_WORKSPACE";
    case UCL_ERR_LAUNCH: return "UCL_ERR_LAUNCH";
    }
    return "UCL_ERR_?";
}

const char *ucl_last_error(void) { return g_err; }
const char *ucl_version(void) { return "ucl 0.1 (gfx950)"; }

}  // extern "C"

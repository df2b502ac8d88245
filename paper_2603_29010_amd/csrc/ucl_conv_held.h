// 3x3 convolutions with pad 1: forward pass at stride 1 or 2, data gradient at stride 1 (the same convolution of the output gradient with the
// taps mirrored).  The filter stays in registers, the pixels stay in LDS.
//
// A workgroup of eight waves owns a band of output rows and 32 NG output channels.  A wave holds nine taps x 64 channels x 32 filters
// (144 registers) for the whole launch; KG waves share out channels beyond 64, NG the filters, MG = 8 / (KG NG) the rows or columns.  The pixels
// that the band's taps reach are copied into LDS once, in planes of 64 channels (rows of 128 bytes, chunks XORed as in the
// tile kernels), image rows at a pitch that is a multiple of 16 pixels with a zero in front, and a zero row between images: a tap is a
// constant shift then and no address is tested.  A wave walks strips of 16 columns downwards: the six fragments of an input row (three
// shifts, two halves of the channels) are multiplied into the three output rows whose taps meet it, so LDS delivers a third of
// what fragments read per tap would take (it bounded the patch kernels' loop), no filter passes through LDS in the loop, and nothing
// in the loop waits for a barrier (KG = 1).  Rows are taken in pairs: 72 MFMAs without a branch, beside which the pair before is finished (its sums
// meet in LDS where KG > 1), its residual requested a pair ahead and its stores left to run.
//
// What bounds it: a wave's pair takes 1.3 us (KG = 1) to 1.5 us, 1.15 of it MFMAs; a launch 2.9 us and about 2 us until filter and pixels are there, which
// 295 KB of filters per CU stretch to 4 us where all CUs copy (15 TB/s from L2).  Measured on the steps to it, 4 images of 56 x 56 x 64 <- 64, us per
// pair: rows one by one with a branch per tap row 2.3, pairs 1.95, addresses kept and conversions packed 1.55, sums stored from the MFMA's layout 1.3.
// Stores with the non-temporal bit and residual loads without it (a wave reads half lines): 32 x 56 x 56 x 64 -> 128 22.7 -> 20.8 us.
// A last single row with half of the MFMAs (KG > 1; 0.55 of a pair) instead of a pair with one row missing: 1.03 on average over 120 drawn forward
// passes of 128 and 256 channels, up to 1.14 (12 x 11 x 11 x 256 -> 512), 1.014 with data and filter gradient together; launches of even rows as before.
// Tile kernels -> here, us in a graph: forward with bias, residual and ReLU 32 x 56 x 56 x 64 -> 128 27.8 -> 20.2, 32 x 56 x 56 x 64 -> 64 24.2 -> 12.3,
// 32 x 28 x 28 x 128 -> 128 16.3 -> 12.9, 4 x 14 x 14 x 256 -> 256 11.1 -> 7.9; data gradients 32 x 28 x 28 x 128 14.9 -> 12.6, 32 x 14 x 14 x 256
// 27.5 -> 18.9, 4 x 14 x 14 x 256 17.0 -> 8.1, 1 x 56 x 56 x 64 10.5 -> 6.3.
#pragma once
#include "ucl_skinny.h"

namespace ucl {

typedef __attribute__((__vector_size__(16))) unsigned int u32x4_b;       // (what the buffer builtins take)
typedef __attribute__((__vector_size__(8))) unsigned int u32x2_b;

struct ConvHeld {
    const void *x, *w;
    void *y;
    const void *bias, *res;
    int32_t H, W, P, Q, C, N;              // gathered pixels: H x W x C; output: P x Q x N
    int32_t n_img, pair;                   // images; images side by side in a row (2: eight columns each)
    int32_t rows, R;                       // padded output rows in all (one more than P per image or pair), per workgroup
    int32_t passes, keep_bytes;            // over the channels, 64 KG each; LDS for the sums of earlier ones
    int32_t inner, bands_inner;            // workgroups are numbered band by band and tile of filters by tile: which of them varies faster, and how many it has
    int32_t pitch, strips, strip_split;     // waves of a workgroup that share out strips (the others of MG: rows)
    uint32_t x_bytes, w_bytes, y_bytes;
    int32_t bias_dt, has_bias, has_res, relu;     // (residual and output: the inputs' type)
    float alpha, beta, rcp_inner, rcp_rows;       // 1 / inner, 1 / (P + 1)
};

template <int DT_, int MODE_ /*2 fprop, 3 dgrad*/, int KG_, int NG_, bool RES_ /*the chain adds a residual*/, bool MULTI_ = false /*several passes over the channels*/, int ST_ = 1 /*stride*/>
struct HeldCfg {
    static constexpr int DT = DT_, MODE = MODE_, KG = KG_, NG = NG_, MG = 8 / (KG_ * NG_);
    static constexpr bool RES = RES_, MULTI = MULTI_;
    static constexpr int ST = ST_;
    static_assert(ST_ == 1 || (ST_ == 2 && MODE_ == 2), "stride 2: forward");
    static_assert(!MULTI_ || KG_ > 1, "the sums of a pass are kept where they meet");
    static_assert(MG * KG * NG == 8, "eight waves");
    static constexpr int SLOT_BYTES = KG * NG * 4096, SLOT_COPIES = SLOT_BYTES / 8192, SLOTS = held_slots(KG_, NG_);
    static constexpr bool PRIVATE = MG == 1;                      // a wave copies and reads its own filters only
    static constexpr int FILTER_BYTES = held_filter_bytes(KG_, NG_);
    static constexpr int PATCH_BYTES = held_patch_capacity(KG_, NG_);
    static_assert(PATCH_BYTES > 0, "not among the wave groups that are chosen");
};

// The lane's number, worked out where it is needed: a register less to keep.
__device__ __forceinline__ int lane_again() {
    int l = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    asm volatile("" : "+v"(l));
    return l;
}

// The MFMA with its accumulator in place: left to rename accumulators where branches meet, the compiler runs out of registers.  As asm statements they
// stay in source order, and nobody counts wait states: operands come from LDS reads only, and sums_ready() stands before a sum is read.
template <int DT, bool FIRST>
__device__ __forceinline__ void mfma_held(f32x4_t &c, const u32x4_t &a, const u32x4_t &b) {
    if constexpr (FIRST) {
        if constexpr (DT == 1) asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "v"(b));
        else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "v"(b));
    } else {
        if constexpr (DT == 1) asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
        else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
    }
}
// (two numbers rounded to nearest even and packed)
template <int DT>
__device__ __forceinline__ uint32_t pack16(float lo, float hi) {
    if constexpr (DT == 0) return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{lo, hi}), bf16x2_t));
    else return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t{lo, hi}), f16x2_t));
}
__device__ __forceinline__ uint32_t lds_addr(const void *p) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char *)p; }
template <class V>
__device__ __forceinline__ __attribute__((address_space(3))) V *lds_ptr(uint32_t at) { return (__attribute__((address_space(3))) V *)(uintptr_t)at; }
__device__ __forceinline__ void sums_ready(f32x4_t (&c)[2]) { asm volatile("s_nop 15" : "+v"(c[0]), "+v"(c[1])); }

// pipeline_barrier, or for copies that one wave alone reads the waits of it only.
template <int VM, bool ALL>
__device__ __forceinline__ void wait_copies() {
    if constexpr (ALL) pipeline_barrier<VM>();
    else {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt((VM & 0xF) | ((VM >> 4) << 14) | (0x7 << 4) | (0x0 << 8));
        asm volatile("" ::: "memory");
    }
}

template <class Cfg>
__global__ __launch_bounds__(512, 2) void conv_held_kernel(const ConvHeld a) {
    constexpr int DT = Cfg::DT, MODE = Cfg::MODE, ST = Cfg::ST, KG = Cfg::KG, NG = Cfg::NG, MG = Cfg::MG, SLOTS = Cfg::SLOTS, SC = Cfg::SLOT_COPIES;
    __shared__ __attribute__((aligned(1024))) char smem[kLdsBytesPerCU];
    char *const patch = smem, *const stage = smem + Cfg::PATCH_BYTES;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ng = wave % NG, kg = wave / NG % KG, mg = wave / (NG * KG);
    const int t = xcd_remap(blockIdx.x, gridDim.x);
    // (divisions by a reciprocal: exact below 2^21)
    auto divide = [](int x, float rcp) { return __builtin_amdgcn_readfirstlane((int)(((float)x + 0.5f) * rcp)); };
    // (an XCD takes a run of these: bands of one tile of filters after the other, or tiles of one band, so that of pixels and filters the larger is read once)
    const int outer = divide(t, a.rcp_inner), inner = t - outer * a.inner;
    const int band = a.bands_inner ? inner : outer, n0 = (a.bands_inner ? outer : inner) * (32 * NG);
    const int R = a.R, pitch = a.pitch, Pp = a.P + 1, line = ST * pitch;      // (pixels of an image row in LDS)
    const int row0 = band * R;                                    // the band's first padded row
    const int plane_bytes = (int)held_plane_bytes(ST, R, pitch);

    // (asked for first, as the copies retire in order)
    float *const bias = (float *)(stage + Cfg::FILTER_BYTES);
    const Raw8 bias_raw = load8(a.bias, a.bias_dt, n0 + tid * 8, a.has_bias && tid < NG * 4 ? a.N - n0 - tid * 8 : 0);
    for (int pass = 0;;) {
    const int c0 = pass * (64 * KG);
    const int lane = Cfg::MULTI ? lane_again() : tid & 63;
    // ---- the filter, tap by tap through LDS into registers -----------------------------------------------------------
    // A block of 16 filters is a row block of the MFMA: row 4 g + i of block nb is filter 8 g + 4 nb + i of the wave's 32, so that a lane's two
    // accumulators are eight consecutive channels.
    u32x4_t wf[9][2][2];
    const rsrc_t w_rsrc = buffer_rsrc(a.w, a.w_bytes);
    uint32_t w_off[SC];
    static_for<SC>([&](auto j) {
        const int i = wave * SC + j;
        if constexpr (MODE == 2) {          // rows of filters, 64 channels each
            const int plane = i / (NG * 4), row = (i % (NG * 4)) * 8 + (lane >> 3), ch = c0 + plane * 64 + ((lane & 7) ^ lds_swz<8>(row)) * 8;
            w_off[j] = n0 + row < a.N && ch < a.C ? (uint32_t)((n0 + row) * 9 * a.C + ch) * 2 : kOobOffset;
        } else if constexpr (Cfg::PRIVATE) {    // rows of gathered channels, the wave's 32 output channels each
            const int k = c0 + kg * 64 + j * 16 + (lane >> 2), n = n0 + ng * 32 + (lane & 3) * 8;
            w_off[j] = k < a.C && n < a.N ? (uint32_t)(k * 9 * a.N + n) * 2 : kOobOffset;
        } else {                                // rows of gathered channels, 32 NG output channels each
            constexpr int PER = NG * 4, RPI = 64 / PER;
            const int k = c0 + i * RPI + lane / PER;
            const int x = NG == 4 ? (k & 3) << 2 : NG == 2 ? (k & 2) << 1 : 0;
            const int n = n0 + ((lane % PER) ^ x) * 8;
            w_off[j] = k < a.C && n < a.N ? (uint32_t)(k * 9 * a.N + n) * 2 : kOobOffset;
        }
    });
    auto copy = [&](int tap) __attribute__((always_inline)) {
        char *dst = stage + tap % SLOTS * Cfg::SLOT_BYTES + wave * (SC * 1024);
        const int at = MODE == 2 ? tap * a.C * 2 : (8 - tap) * a.N * 2;
        static_for<SC>([&](auto j) { __builtin_amdgcn_raw_ptr_buffer_load_lds(w_rsrc, UCL_LDS_PTR(dst + j * 1024), 16, w_off[j], at, 0, 0); });
    };
    static_for<SLOTS>([&](auto t_) { copy(t_); });

    // ---- copies of the pixels: local row i holds row h of an image, h = -1 and from H on standing for zero rows, eight pixels of a plane per
    // instruction.  Stride 1: entry e of a row is column e - 1.  Stride 2: columns 2 e - 1, then columns 2 e. ------------
    int pixel_copies = 0;                                         // that the wave has issued
    {
        const rsrc_t x_rsrc = buffer_rsrc(a.x, a.x_bytes);
        const int half = pitch / 8 * KG, per_row = ST * half, rows_in = ST * R + 3 - ST, period = ST * Pp;
        int b = wave, i = 0;
        int img = divide(row0, a.rcp_rows), h = ST * (row0 - img * Pp) - 1;
        while (b >= per_row) { b -= per_row; ++i; ++h; }
        while (h >= period - 1) { h -= period; ++img; }
        while (i < rows_in) {
            const int even = ST == 2 && b >= half, plane = b & (KG - 1), blk = (even ? b - half : b) / KG;
            const int col = blk * 8 + (lane >> 3);
            const int ch = c0 + plane * 64 + ((lane & 7) ^ lds_swz<8>(col)) * 8;
            int e = col, im = img * a.pair;
            if (a.pair == 2) {
                const bool second = ST == 1 ? col > 8 : col >= 8;
                im += second;
                e = second ? col - 8 : col;
            }
            const int w = ST == 1 ? e - 1 : 2 * e - 1 + even;
            const bool in = (unsigned)h < (unsigned)a.H && (unsigned)w < (unsigned)a.W && im < a.n_img && ch < a.C;
            const uint32_t off = (((uint32_t)(im * a.H + h) * (uint32_t)a.W + (uint32_t)w) * (uint32_t)a.C + (uint32_t)ch) * 2;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(x_rsrc, UCL_LDS_PTR(patch + plane * plane_bytes + (i * line + even * pitch + blk * 8) * 128), 16, in ? off : kOobOffset, 0, 0, 0);
            ++pixel_copies;
            b += 8;
            while (b >= per_row) {
                b -= per_row;
                ++i;
                if (++h == period - 1) { h = -1; ++img; }
            }
        }
        // (the zeros behind the last row: what a tap to the right of its last column reads where the pitch leaves no zero there)
        if (ST == 1 && wave < KG)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(x_rsrc, UCL_LDS_PTR(patch + wave * plane_bytes + (R + 2) * pitch * 128), 16, kOobOffset, 0, 0, 0);
    }

    {
        const int l = lane & 15, g = lane >> 4;
        static_for<9>([&](auto t_) {
            // The first SLOTS taps were requested before the pixels, which may still be on their way while these are read; of the pixels' copies
            // what is known at compile time is counted.
            constexpr int tap = decltype(t_)::value, later = (8 - tap < SLOTS - 1 ? 8 - tap : SLOTS - 1) * SC;
            if (tap >= SLOTS || pixel_copies < 8) wait_copies<later, !Cfg::PRIVATE>();
            else if (pixel_copies < 16) wait_copies<later + 8, !Cfg::PRIVATE>();
            else if (pixel_copies < 24) wait_copies<later + 16, !Cfg::PRIVATE>();
            else wait_copies<later + 24, !Cfg::PRIVATE>();
            const char *const slot = stage + tap % SLOTS * Cfg::SLOT_BYTES;
            if constexpr (MODE == 2) {
                static_for<2>([&](auto ks) {
                    static_for<2>([&](auto nb) {
                        const int row = ng * 32 + 8 * (l >> 2) + 4 * nb + (l & 3);
                        wf[tap][ks][nb] = *(const u32x4_t *)(slot + kg * (NG * 4096) + row * 128 + (((ks * 4 + g) ^ lds_swz<8>(row)) << 4));
                    });
                });
            } else {
                // transpose reads of four rows each; the other halves, blocks and k-steps: rows and bytes on, under the same XOR
                constexpr int ROW = Cfg::PRIVATE ? 64 : NG * 64;
                const int k = 8 * g + (l >> 2), x = Cfg::PRIVATE ? 0 : NG == 4 ? (k & 3) << 2 : NG == 2 ? (k & 2) << 1 : 0;
                const int from_wave = Cfg::PRIVATE ? wave * 4096 + ((l & 3) << 4) : kg * (64 * ROW) + (((ng * 4 + (l & 3)) ^ x) << 4);
                const uint32_t from = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char *)(slot + from_wave + k * ROW);
                u32x2_t h[8];
                asm volatile("ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %8 offset:%9\n\tds_read_b64_tr_b16 %2, %8 offset:8\n\tds_read_b64_tr_b16 %3, %8 offset:%9+8\n\t"
                             "ds_read_b64_tr_b16 %4, %8 offset:%10\n\tds_read_b64_tr_b16 %5, %8 offset:%9+%10\n\tds_read_b64_tr_b16 %6, %8 offset:%10+8\n\t"
                             "ds_read_b64_tr_b16 %7, %8 offset:%9+%10+8\n\ts_waitcnt lgkmcnt(0)"
                             : "=&v"(h[0]), "=&v"(h[1]), "=&v"(h[2]), "=&v"(h[3]), "=&v"(h[4]), "=&v"(h[5]), "=&v"(h[6]), "=&v"(h[7])
                             : "v"(from), "n"(4 * ROW), "n"(32 * ROW));
                static_for<4>([&](auto i) { wf[tap][i >> 1][i & 1] = u32x4_t{h[2 * i][0], h[2 * i][1], h[2 * i + 1][0], h[2 * i + 1][1]}; });
            }
            if constexpr (tap + SLOTS < 9) {
                wait_copies<63, !Cfg::PRIVATE>();              // the slot has been read
                copy(tap + SLOTS);
            }
        });
        if (pass == 0 && tid < NG * 4) {
            float b8[8];
            decode8(bias_raw, a.bias_dt, b8);
            *(f32x4_t *)(bias + tid * 8) = f32x4_t{b8[0], b8[1], b8[2], b8[3]};
            *(f32x4_t *)(bias + tid * 8 + 4) = f32x4_t{b8[4], b8[5], b8[6], b8[7]};
        }
        pipeline_barrier<0>();                   // (the sums meet where the filter passed)
    }
    float *const meet = (float *)stage;

    // ---- the wave's part of the band: strips of 16 columns, two output rows at a time -----------------------------------
    const int sgroups = a.strip_split, rgroups = MG / sgroups;
    const int ms = mg & (sgroups - 1), mr = mg / sgroups;
    const int per = held_rows_of_wave(R, rgroups, KG, Cfg::MULTI), first = mr * per;    // output rows of the wave, and where they start
    if (KG == 1 && first >= R) return;
    const int img0 = divide(row0 + first, a.rcp_rows), p0 = row0 + first - img0 * Pp;
    const int own_rows = R - first < per ? R - first : per;
    const int rows_left = own_rows < a.rows - row0 - first ? own_rows : a.rows - row0 - first;
    const int strip_rounds = (a.strips + sgroups - 1) / sgroups;
    const int own = lane_again(), l = own & 15, g = own >> 4;
    // fragment addresses: shift s, chunk g (the other half of the channels: ^ 64)
    uint32_t at[3];
    static_for<3>([&](auto s_) {
        constexpr int s = decltype(s_)::value;
        const int e = l + (ST == 1 ? s : s >> 1);
        at[s] = lds_addr(patch + kg * plane_bytes + ((first < R ? first : 0) * ST * line + ms * 16 + (ST == 2 && s == 1 ? pitch : 0) + e) * 128) + (uint32_t)((g ^ lds_swz<8>(e)) << 4);
    });
    u32x4_t fr[6];
    auto fetch = [&](auto f_) __attribute__((always_inline)) {
        constexpr int f = decltype(f_)::value;
        fr[f] = *lds_ptr<u32x4_t>(at[f >> 1] ^ ((f & 1) << 6));
    };
    f32x4_t acc[2][2];
    // A finished block's 16 pixels x 32 channels meet in LDS and are dealt to its KG waves: EPL channels per lane.
    constexpr int EPL = 8 / KG, HALVES = KG == 1 ? 2 : 1, VW = EPL / HALVES;
    typedef __attribute__((ext_vector_type(VW))) float vec_t;
    uint32_t res[2][2][EPL / 2];                                  // of two pairs of rows
    const uint32_t row_bytes = (uint32_t)(a.Q * a.N) * 2;
    const rsrc_t y_rsrc = buffer_rsrc(a.y, a.y_bytes), res_rsrc = buffer_rsrc(a.res, a.has_res ? a.y_bytes : 0u);
    vec_t sum[HALVES], b4[HALVES];
    uint32_t out[EPL / 2];
    // where the wave's sums go (block 1: chunk ^ 1), and where its part of a block comes from (second half: chunk ^ 1; another wave's: a kilobyte
    // multiple on): LDS addresses, worked out once
    const uint32_t put_at = lds_addr(meet + wave * 512 + l * 32) + (uint32_t)(((2 * g) ^ lds_swz<8>(l)) << 4);
    const int e_px = KG == 1 ? l : kg * (16 / KG) + own / (4 * KG), e_ch = KG == 1 ? 8 * g : own % (4 * KG) * EPL;
    const uint32_t get_at = lds_addr(meet + (mg * KG * NG + ng) * 512 + e_px * 32 + (e_ch & 3)) + (uint32_t)(((e_ch >> 2) ^ lds_swz<8>(e_px)) << 4);
    const uint32_t bias_at = lds_addr(bias + ng * 32 + e_ch);
    const float floor = a.relu ? 0.f : __builtin_nanf("");       // (the larger of a number and NaN is the number)
    // several passes: what the earlier ones have added up of the lane's channels, block by block
    uint32_t keep_at = Cfg::MULTI ? lds_addr(patch + Cfg::PATCH_BYTES - a.keep_bytes) + (uint32_t)(wave * 64 + own) * (EPL * 4) : 0u;
    const bool last_pass = pass + 1 == a.passes;
    // (par: of two consecutive pairs of rows, which)
    auto put = [&](auto par_, auto o_) __attribute__((always_inline)) {
        constexpr int o = decltype(o_)::value, par = decltype(par_)::value;
        static_for<2>([&](auto nb) { *lds_ptr<f32x4_t>((put_at ^ (nb << 4)) + (par * 2 + o) * (8 * 2048)) = acc[o][nb]; });
        asm volatile("" ::: "memory");
    };
    auto get = [&](auto par_, auto o_) __attribute__((always_inline)) {
        constexpr int o = decltype(o_)::value, par = decltype(par_)::value;
        static_for<HALVES>([&](auto h_) {
            constexpr int h = decltype(h_)::value;
            b4[h] = *lds_ptr<vec_t>(bias_at + h * 16);
            static_for<KG>([&](auto k) {
                const vec_t x = *lds_ptr<vec_t>((get_at ^ (h << 4)) + (par * 2 + o) * (8 * 2048) + k * (NG * 2048));
                if constexpr (decltype(k)::value == 0) sum[h] = x; else sum[h] += x;
            });
        });
        if constexpr (Cfg::MULTI) {
            const vec_t before = *lds_ptr<vec_t>(keep_at);
            sum[0] = pass ? sum[0] + before : sum[0];
            *lds_ptr<vec_t>(keep_at) = sum[0];
            keep_at += 512 * EPL * 4;
        }
    };
    auto chain = [&](auto par_, auto o_) __attribute__((always_inline)) {
        constexpr int o = decltype(o_)::value, par = decltype(par_)::value, T = DT == 1 ? UCL_F16 : UCL_BF16;
        static_for<HALVES>([&](auto h_) {
            constexpr int h = decltype(h_)::value;
            float v[VW];
#pragma unroll
            for (int e = 0; e < VW; ++e) {
                if constexpr (KG == 1) v[e] = acc[o][h][e] * a.alpha + b4[h][e];
                else v[e] = sum[h][e] * a.alpha + b4[h][e];
                if constexpr (Cfg::RES) v[e] += a.beta * bits_to_f32(res[par][o][h * 2 + (e >> 1)] >> (e & 1) * 16 & 0xffffu, T);
                v[e] = fmaxf(v[e], floor);
            }
#pragma unroll
            for (int e = 0; e < VW / 2; ++e) out[2 * h + e] = pack16<DT>(v[2 * e], v[2 * e + 1]);
        });
    };
    auto store = [&](uint32_t off, uint32_t row) __attribute__((always_inline)) {
        if constexpr (EPL == 8) {
            const u32x4_t v{out[0], out[1], out[2], out[3]};
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_b, v), y_rsrc, off, row, kAuxStream);
            // A store of more than 64 bits may still be reading its data when the next instruction issues, also with its offset in a scalar
            // register, where the compiler expects no hazard: overwritten at once, the first words of every fourth pixel were wrong now and then.
            asm volatile("s_nop 1" ::"v"(v));
        } else if constexpr (EPL == 4) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_b, u32x2_t{out[0], out[1]}), y_rsrc, off, row, kAuxStream);
        else __builtin_amdgcn_raw_buffer_store_b32(out[0], y_rsrc, off, row, kAuxStream);
    };
    auto load = [&](auto par_, auto o_, uint32_t off, uint32_t row) __attribute__((always_inline)) {
        uint32_t(&r)[EPL / 2] = res[decltype(par_)::value][decltype(o_)::value];
        if constexpr (EPL == 8) {
            const u32x4_t v = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(res_rsrc, off, row, 0));
            static_for<4>([&](auto i) { r[i] = v[decltype(i)::value]; });
        } else if constexpr (EPL == 4) {
            const u32x2_t v = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(res_rsrc, off, row, 0));
            static_for<2>([&](auto i) { r[i] = v[decltype(i)::value]; });
        } else r[0] = __builtin_amdgcn_raw_buffer_load_b32(res_rsrc, off, row, 0);
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    // a pair of rows is finished beside the first MFMAs of the next one: where it goes
    uint32_t late_off[2] = {kOobOffset, kOobOffset}, late_row[2] = {0, 0};
    static_for<2>([&](auto o) { static_for<2>([&](auto nb) { acc[o][nb] = f32x4_t{0.f, 0.f, 0.f, 0.f}; }); });
    static_for<6>([&](auto f) { fetch(f); });
    // (of the last pair of images the second may be missing)
    const int e_last = a.pair == 2 && e_px >= 8 ? a.n_img / 2 : a.n_img;
    uint32_t e_off = 0;                                            // the lane's pixel of a strip's finished blocks: bytes from the row's first pixel
    int o = 0, sr = 0, img = img0, p = p0;
    auto strip_start = [&]() __attribute__((always_inline)) {
        const int e_n = n0 + ng * 32 + e_ch;
        int q = (sr * sgroups + ms) * 16 + e_px;
        e_off = 0;
        if (a.pair == 2) {
            q &= 7;
            e_off = e_px >= 8 ? (uint32_t)a.P * row_bytes : 0u;
        }
        e_off = e_n < a.N && q < a.Q ? e_off + (uint32_t)(q * a.N + e_n) * 2 : kOobOffset;
        img = img0;
        p = p0;
    };
    // Input rows ST o .. ST o + 2 meet output row o, ST rows on those of row o + 1.  Loads of the residual and stores
    // are issued for every row, out of range where there is nothing to do: waits then count them.
    // (ONE: the pair's second row is not the wave's: half of the MFMAs.  Where KG = 1 the body's own finishing does not fit into the registers,
    // nor with several passes: those count their rows in pairs.)
    auto rows = [&](auto par_, auto one_) __attribute__((always_inline)) {
        constexpr bool ONE = decltype(one_)::value;
        using Par = std::integral_constant<int, decltype(par_)::value>;
        using Other = std::integral_constant<int, 1 - decltype(par_)::value>;
        uint32_t off[2], row[2];
        static_for<2>([&](auto k) {
            off[k] = p < a.P && o + (int)k < rows_left && img < e_last && (!Cfg::MULTI || last_pass) ? e_off : kOobOffset;
            row[k] = (uint32_t)(img * a.pair * a.P + p) * row_bytes;
            if (++p == Pp) { p = 0; ++img; }
            if constexpr (Cfg::RES) load(Par{}, k, off[k], row[k]);
        });
        // the first row after this pair (stride 1: one up from its last, stride 2: its last again), or the wave's next strip
        const int back = o + 2 < per ? (ONE ? 2 * ST - 2 : ST - 2) * line * 128 : sr + 1 < strip_rounds ? (sgroups * 16 - (ST * (ONE ? o : per - 1) + 2) * line) * 128 : 0;
        constexpr int ROWS = ONE ? 3 : ST + 3;
        static_for<ROWS>([&](auto j_) {
            constexpr int j = decltype(j_)::value;
            static_for<3>([&](auto s) { at[s] += j == ROWS - 1 ? back : line * 128; });
            static_for<6>([&](auto f_) {
                constexpr int f = decltype(f_)::value, s = f >> 1, ks = f & 1;
                if constexpr (j <= 2) static_for<2>([&](auto nb) { mfma_held<DT, j == 0 && f == 0>(acc[0][nb], wf[j * 3 + s][ks][nb], fr[f]); });
                if constexpr (j >= ST && !ONE) static_for<2>([&](auto nb) { mfma_held<DT, j == ST && f == 0>(acc[1][nb], wf[(j - ST) * 3 + s][ks][nb], fr[f]); });
                fetch(f_);
                // (four MFMAs have been issued since the last one of the sums that are read here)
                if constexpr (KG == 1) {
                    if constexpr (j == 0 && f == 2) chain(Other{}, I1{});
                    if constexpr (j == 0 && f == 4) store(late_off[1], late_row[1]);
                    if constexpr (j == 3 && f == 2) chain(Par{}, I0{});
                    if constexpr (j == 3 && f == 4) store(off[0], row[0]);
                } else {
                    if constexpr (j == 0 && f == 1) put(Other{}, I1{});
                    if constexpr (j == 0 && f == 2) {
                        pipeline_barrier<63>();
                        get(Other{}, I0{});
                    }
                    if constexpr (j == 0 && f == 5) chain(Other{}, I0{});
                    if constexpr (j == 1 && f == 0) {
                        store(late_off[0], late_row[0]);
                        get(Other{}, I1{});
                    }
                    if constexpr (j == 1 && f == 2) chain(Other{}, I1{});
                    if constexpr (j == 1 && f == 3) store(late_off[1], late_row[1]);
                    if constexpr (j == 3 && f == 2) put(Par{}, I0{});
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        if constexpr (ONE) {
            sums_ready(acc[0]);
            put(Par{}, I0{});
        }
        static_for<2>([&](auto k) {
            late_off[k] = off[k];
            late_row[k] = row[k];
        });
    };
    // true behind the last pair
    auto step = [&](auto par) __attribute__((always_inline)) {
        if constexpr (KG > 1 && !Cfg::MULTI) {
            if (o + 1 < own_rows) rows(par, std::false_type{});
            else rows(par, std::true_type{});
        } else rows(par, std::false_type{});
        o += 2;
        if (o >= per) {
            o = 0;
            if (++sr < strip_rounds) strip_start();
        }
        return sr == strip_rounds;
    };
    auto finish = [&](auto par) __attribute__((always_inline)) {
        sums_ready(acc[1]);
        if constexpr (KG > 1) {
            put(par, I1{});
            pipeline_barrier<63>();
            get(par, I0{});
            chain(par, I0{});
            store(late_off[0], late_row[0]);
            get(par, I1{});
        }
        chain(par, I1{});
        store(late_off[1], late_row[1]);
    };
    if constexpr (KG == 1) static_for<2>([&](auto h) { b4[decltype(h)::value] = *lds_ptr<vec_t>(bias_at + h * 16); });
    strip_start();
    for (;;) {
        if (step(I0{})) {
            finish(I0{});
            break;
        }
        if (step(I1{})) {
            finish(I1{});
            break;
        }
    }
    if (!Cfg::MULTI || ++pass == a.passes) return;
    pipeline_barrier<63>();                      // (the next pass's copies go where sums and pixels were read)
    }
}

template <class Cfg>
hipError_t launch_conv_held_cfg(const ConvHeld &a, int grid, hipStream_t stream) {
    hipLaunchKernelGGL(conv_held_kernel<Cfg>, dim3((unsigned)grid), dim3(512), 0, stream, a);
    return hipGetLastError();
}

template <int DT, int MODE, bool RES, int ST = 1>
hipError_t launch_conv_held_mode(const HeldPlan &h, const KParams &p, hipStream_t stream) {
    ConvHeld a;
    a.x = p.A; a.w = p.B; a.y = p.D; a.bias = p.fused.bias; a.res = p.fused.res;
    a.H = p.cH; a.W = p.cW; a.P = p.cP; a.Q = p.cQ; a.C = p.cC; a.N = p.N;
    a.n_img = p.M / (p.cP * p.cQ); a.pair = h.pair;
    a.rows = h.rows; a.R = h.R; a.passes = h.passes; a.keep_bytes = h.keep_bytes; a.pitch = h.pitch; a.strips = h.strips; a.strip_split = h.strip_split;
    a.x_bytes = (uint32_t)p.a_bytes; a.w_bytes = (uint32_t)((int64_t)p.cC * 9 * p.N * 2);
    a.y_bytes = (uint32_t)((int64_t)p.M * p.N * 2);
    a.bias_dt = p.fused.bias_dt & 0xff;
    a.has_bias = p.fused.has_bias; a.has_res = p.fused.has_res; a.relu = p.fused.act == UCL_EPI_RELU;
    a.alpha = p.fused.has_scale ? p.fused.alpha : 1.f; a.beta = p.fused.beta;
    a.bands_inner = a.w_bytes > a.x_bytes; a.inner = a.bands_inner ? h.bands : h.tiles_n;
    a.rcp_inner = 1.f / (float)a.inner; a.rcp_rows = 1.f / (float)(p.cP + 1);
    const int grid = h.bands * h.tiles_n;
    if constexpr (MODE == 3) {
        if (h.passes > 1 && h.ng == 2) return launch_conv_held_cfg<HeldCfg<DT, MODE, kHeldMaxKG, 2, RES, true>>(a, grid, stream);
        if (h.passes > 1) return launch_conv_held_cfg<HeldCfg<DT, MODE, kHeldMaxKG, 1, RES, true>>(a, grid, stream);
    }
    switch (h.kg * 8 + h.ng) {
    case 8 + 4: return launch_conv_held_cfg<HeldCfg<DT, MODE, 1, 4, RES, false, ST>>(a, grid, stream);
    case 8 + 2: return launch_conv_held_cfg<HeldCfg<DT, MODE, 1, 2, RES, false, ST>>(a, grid, stream);
    case 16 + 4: return launch_conv_held_cfg<HeldCfg<DT, MODE, 2, 4, RES, false, ST>>(a, grid, stream);
    case 16 + 2: return launch_conv_held_cfg<HeldCfg<DT, MODE, 2, 2, RES, false, ST>>(a, grid, stream);
    case 16 + 1: return launch_conv_held_cfg<HeldCfg<DT, MODE, 2, 1, RES, false, ST>>(a, grid, stream);
    case 32 + 2: return launch_conv_held_cfg<HeldCfg<DT, MODE, 4, 2, RES, false, ST>>(a, grid, stream);
    case 32 + 1: return launch_conv_held_cfg<HeldCfg<DT, MODE, 4, 1, RES, false, ST>>(a, grid, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace ucl

// Filter gradient of 3x3 convolutions with pad 1 at stride 1 or 2: one workgroup multiplies all nine taps of its pixels.
//
//   dw[ko, r, s, c] = sum over output pixels of dy[pixel, ko] * x[pixel of tap (r, s), c]
//
// The tile kernel sees this as a GEMM with 9 C columns and gathers x once per tap: 350 MB from L2 for 32 x 28 x 28 x 128 -> 128, at the
// 14 TB/s that the gathers reach.  Here a workgroup owns 64 filters and 32 channels and copies every pixel's row of x once.
// Pixels are numbered with a zero column behind every row and a zero row behind every image, s = (n (P+1) + p) (Q+1) + q: in that
// numbering a tap is a constant shift, and what it reads outside the image is one of those zeros, so no
// fragment address has a border test.  Stride 2: x is kept as four planes by the parity of its row and column, each in the numbering of
// the output pixels; a tap is one plane and a shift.
// The pixels pass through LDS in k-tiles of KT: dy in four stage buffers, x in a ring of four k-tiles (a k-tile's taps reach into its
// neighbours).  Eight waves: two groups take half of each k-tile's pixels, in a group four waves hold 32 filters x 16 channels x
// 9 taps each; the groups' sums meet in LDS.  Slices of the pixels go to different workgroups; their sums are added up by a second launch.
// The loop is bound by the MFMAs and, with VALU work for copies only, close to them: 0.67 us per 128 pixels (0.5 at full rate; 1.06 with ring addresses worked
// out for every read and one set of fragments, 0.91 with two sets).  But it is 5 of 17.8 us for 32 x 28 x 28 x 128 -> 128, whose MFMAs take 15 %
// of the launch's clocks: the rest is 6.9 us of launch, first copies and meeting, and a second launch of some 3 us and the partial sums at 3 TB/s
// (4.5 us here), which is why 64 x 32 and not more.  Gathering tile kernel -> here, both launches in a graph, fp32 gradient:
// 32 x 28 x 28 x 128 -> 128 26.0 -> 17.8 us, 32 x 14 x 14 x 256 -> 256 31.4 -> 20.9 us, 32 x 7 x 7 x 512 -> 512 41.8 -> 19.4 us,
// 32 x 56 x 56 x 64 -> 64 25.6 -> 20.5 us, 32 x 56 x 56 x 128 -> 128 at stride 2 25.5 -> 21.8 us.
#pragma once
#include "ucl_kernel.h"
#include "ucl_variants.h"

namespace ucl {

struct WgradTaps {
    const void *dy, *x;
    void *dw;                       // one slice: the gradient
    float *partials;                // several: [slice][Kout][9 C] sums
    int32_t n_img, P, Q, H, W, C, Kout;
    int32_t tiles_k, tiles_c, slices, px_per_slice, px;       // px: padded pixels in all
    int32_t step_q, step_p, step_n;                           // a k-tile of pixels in (q, p, n)
    int32_t dtD;
    float alpha, rcp_q, rcp_p;                                // 1 / (Q + 1), 1 / (P + 1)
    uint32_t dy_bytes, x_bytes;
};

// mfma16 with the accumulator in an ordinary register: with two waves per SIMD a kernel has 256 of those, but only 128 beside accumulation registers.
template <int DT>
__device__ __forceinline__ void mfma16_v(f32x4_t &c, const u32x4_t &a, const u32x4_t &b) {
    if constexpr (DT == 1) asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
    else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}

template <int ST>
struct TapsLds {
    static constexpr int KT = ST == 1 ? 128 : 64, BLOCKS = 4, PLANES = ST * ST, STAGES = 4;
    static constexpr int BLOCK_BYTES = KT * 64, PLANE_BYTES = (BLOCKS + 1) * BLOCK_BYTES, X_BYTES = PLANES * PLANE_BYTES, DY_BYTES = KT * 128;
    static constexpr int LD = 292;                                // floats per filter where the sums meet (9 x 32, and padding against bank conflicts)
    static constexpr int MEET_BYTES = 2 * 64 * LD * 4, END_BYTES = MEET_BYTES + 32;      // (and whether each wave has a NaN)
    static constexpr int BYTES = X_BYTES + STAGES * DY_BYTES > END_BYTES ? X_BYTES + STAGES * DY_BYTES : END_BYTES;
    static_assert(BYTES <= kLdsBytesPerCU, "LDS");
};

// Stores the workgroup's sums; true where they hold a NaN and PADDING_OUT is false.
// Padded pixels have dy = 0, but their taps read real pixels of x, and an infinity or NaN there times 0 would be a NaN in the sums of taps that it
// does not belong to.  Testing every fragment would cost VALU time beside the MFMAs.  But such a product always leaves a NaN: a workgroup that
// finds one starts again (PADDING_OUT) and takes what padded pixels multiply out of the x fragments, one k-step after the other.  Finite inputs pay
// 0.1 us at most for it (both gradients of 32 x 28 x 28 x 128, 32.7 us, 0.3 % apart); with a NaN in x the filter gradient takes 43 us instead of 23.
template <int DT, int ST, bool PADDING_OUT>
__device__ __forceinline__ bool wgrad_taps_pass(const WgradTaps &a, char *smem) {
    constexpr int KT = TapsLds<ST>::KT, BLOCKS = TapsLds<ST>::BLOCKS, PLANES = TapsLds<ST>::PLANES;
    constexpr int DY_SLOTS = KT / 64, X_SLOTS = KT * PLANES / 128, COPIES = DY_SLOTS + X_SLOTS;
    constexpr int BLOCK_BYTES = TapsLds<ST>::BLOCK_BYTES, PLANE_BYTES = TapsLds<ST>::PLANE_BYTES, X_BYTES = TapsLds<ST>::X_BYTES, DY_BYTES = TapsLds<ST>::DY_BYTES;
    constexpr int LD = TapsLds<ST>::LD, MEET_BYTES = TapsLds<ST>::MEET_BYTES;
    int tid = threadIdx.x;
    if constexpr (PADDING_OUT) asm volatile("" : "+v"(tid));       // (nothing that follows from it stays in registers over the first pass)
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;
    const int tiles = a.tiles_k * a.tiles_c;
    int t = xcd_remap(blockIdx.x, tiles * a.slices);
    const int slice = t / tiles;
    t -= slice * tiles;
    const int tk = t / a.tiles_c, k0 = tk * 64, c0 = (t - tk * a.tiles_c) * 32;
    const int Pp = a.P + 1, Qp = a.Q + 1, img = Pp * Qp;
    const int s0 = slice * a.px_per_slice;
    const int mine = a.px - s0 < a.px_per_slice ? a.px - s0 : a.px_per_slice;
    const int KTn = (mine + KT - 1) / KT;
    const int halo = Qp + 1;                                      // x: pixels kept before the k-tile's own (and at stride 1 behind them)

    // ---- copies --------------------------------------------------------------------------------------------------
    // (what lies before the first or behind the last image is out of the resources' range and lands as zeros, as do a slot's
    // filters or channels past the end, whose offsets start beyond it)
    const rsrc_t x_rsrc = buffer_rsrc(a.x, a.x_bytes);
    const uint32_t ey = (uint32_t)a.Kout * 2, ex = (uint32_t)a.C * 2;
    const int kn = a.step_n, kp = a.step_p, kq = a.step_q;
    // the slice's first pixel; a slot's pixel is at most a k-tile and a halo from it, near enough for divisions in fp32 (taps_launch bounds P and Q for that)
    const int n0 = s0 / img, p0 = (s0 - n0 * img) / Qp, q0 = s0 - n0 * img - p0 * Qp;
    const uint32_t dyq = ey, dyp = a.Q * ey, dyn = a.P * a.Q * ey;
    const uint32_t xq = ST * ex, xp = ST * a.W * ex, xn = a.H * a.W * ex;
    int q[COPIES], p[COPIES];
    uint32_t off[COPIES];
    int plane_h[X_SLOTS], plane_w[X_SLOTS];
    static_for<COPIES>([&](auto i_) {
        constexpr int i = decltype(i_)::value;
        const int d = i < DY_SLOTS ? (i * 8 + wave) * 8 + (lane >> 3) : (ST == 1 ? wave * 16 : (wave & 3) * 16) + (lane >> 2) - halo;
        const int vq = q0 + d + 2 * Qp, wq = (int)(((float)vq + 0.5f) * a.rcp_q);
        const int vp = p0 + wq - 2 + Pp, wp = (int)(((float)vp + 0.5f) * a.rcp_p);
        q[i] = vq - wq * Qp;
        p[i] = vp - wp * Pp;
        const uint32_t n = (uint32_t)(n0 + wp - 1);
        if constexpr (i < DY_SLOTS) {
            const int row = (i * 8 + wave) * 8 + (lane >> 3), k = k0 + ((lane & 7) ^ ((row & 3) << 1)) * 8;
            off[i] = k < a.Kout ? n * dyn + (uint32_t)p[i] * dyp + (uint32_t)q[i] * dyq + (uint32_t)k * 2 : kOobOffset;
        } else {
            constexpr int j = i - DY_SLOTS;
            const int plane = ST == 1 ? 0 : (j * 8 + wave) >> 2;
            plane_h[j] = plane >> 1;
            plane_w[j] = plane & 1;
            const int c = c0 + ((lane & 3) ^ (((lane >> 5) & 1) << 1)) * 8;         // (row of the block >> 3) & 1 = bit 5 of the lane
            off[i] = c < a.C ? n * xn + (uint32_t)p[i] * xp + (uint32_t)q[i] * xq + (uint32_t)((plane_h[j] * a.W + plane_w[j]) * a.C + c) * 2 : kOobOffset;
        }
    });
    // slot i of stage kt (k-tile kt's dy, and block kt + 1 of x: the taps reach into it), then the slot steps on by one k-tile
    auto copy = [&](auto i_, int buf, int kt) __attribute__((always_inline)) {
        constexpr int i = decltype(i_)::value;
        constexpr bool Y = i < DY_SLOTS;
        bool ok = (q[i] < a.Q) & (p[i] < a.P);
        if constexpr (!Y && ST == 2) ok = ok & (ST * p[i] + plane_h[i - DY_SLOTS] < a.H) & (ST * q[i] + plane_w[i - DY_SLOTS] < a.W);
        uint32_t at = kOobOffset;
        if (ok) at = off[i];
        if constexpr (Y) {
            const rsrc_t r = buffer_rsrc(a.dy, kt < KTn ? a.dy_bytes : 0u);        // (past the slice: zeros)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r, UCL_LDS_PTR(smem + X_BYTES + buf * DY_BYTES + (i * 8 + wave) * 1024), 16, at, 0, 0, 0);
        } else {
            const int idx = (i - DY_SLOTS) * 8 + wave, plane = ST == 1 ? 0 : idx >> 2, part = ST == 1 ? idx : idx & 3;
            const int block = (buf + 1) % BLOCKS;
            char *dst = smem + plane * PLANE_BYTES + block * BLOCK_BYTES + part * 1024;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(x_rsrc, UCL_LDS_PTR(dst), 16, at, 0, 0, 0);
            // (block 0 stands behind block 3 once more, so that nobody's addresses wrap)
            if (block == 0) __builtin_amdgcn_raw_ptr_buffer_load_lds(x_rsrc, UCL_LDS_PTR(dst + BLOCKS * BLOCK_BYTES), 16, at, 0, 0, 0);
        }
        const uint32_t eq = Y ? dyq : xq, ep = Y ? dyp : xp, en = Y ? dyn : xn;
        q[i] += kq;
        off[i] += (uint32_t)kq * eq + (uint32_t)kp * ep + (uint32_t)kn * en;
        const bool cq = q[i] >= Qp;
        q[i] -= cq ? Qp : 0;
        p[i] += cq ? kp + 1 : kp;
        off[i] += cq ? ep - (uint32_t)Qp * eq : 0u;
        const bool cp = p[i] >= Pp;
        p[i] -= cp ? Pp : 0;
        off[i] += cp ? en - (uint32_t)Pp * ep : 0u;
    };

    // ---- fragments -----------------------------------------------------------------------------------------------
    const int l = lane & 15, g = lane >> 4;
    const int px0 = kg * (KT / 2) + 8 * g + (l >> 2);             // the lane's pixel of the group's first k-step (its second: 4 on)
    const int a_addr0 = X_BYTES + px0 * 128 + (((wm * 4 + ((l & 3) >> 1)) ^ ((l >> 2) << 1)) << 4) + (l & 1) * 8;
    // the same for tap's fragment halves, from the ring's first block on: what a k-tile and a k-step add, multiples of 32 pixels that leave the
    // chunk's XOR as it is, goes into the reads' immediate offsets (the loop is unrolled over the four blocks)
    uint32_t b_addr[9][2];
    static_for<9>([&](auto tap_) {
        constexpr int r = decltype(tap_)::value / 3, s = decltype(tap_)::value % 3;
        constexpr int plane = ST == 1 ? 0 : (r != 1 ? 2 : 0) + (s != 1 ? 1 : 0);
        const int shift = ST == 1 ? (r - 1) * Qp + s - 1 : (r == 0 ? -Qp : 0) + (s == 0 ? -1 : 0);
        static_for<2>([&](auto h) {
            const int pos = halo + px0 + shift + 4 * h;
            b_addr[tap_][h] = (uint32_t)(plane * PLANE_BYTES + pos * 64 + (((wn * 2 + ((l & 3) >> 1)) ^ (((pos >> 3) & 1) << 1)) << 4) + (l & 1) * 8);
        });
    });
    f32x4_t acc[2][9];
    static_for<2>([&](auto mi) { static_for<9>([&](auto tap) { acc[mi][tap] = f32x4_t{0.f, 0.f, 0.f, 0.f}; asm volatile("" : "+v"(acc[mi][tap])); }); });
    // Fragments of two k-steps: while one is multiplied the next one's are read.  The transpose reads are asm, which the compiler counts no
    // waits for: a phase ends with all of them back.
    u32x4_t af[2][2], bf[2][9];
    const uint32_t a_addr[2] = {(uint32_t)a_addr0, (uint32_t)a_addr0 ^ 32u};
    auto read = [&](auto set_, auto f_, auto buf_, auto ks_, int block) __attribute__((always_inline)) {
        constexpr int set = decltype(set_)::value, f = decltype(f_)::value, buf = decltype(buf_)::value, ks = decltype(ks_)::value;
        u32x2_t lo, hi;
        if constexpr (f < 2) {
            constexpr int at = buf * DY_BYTES + ks * 32 * 128;
            asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%3\n\tds_read_b64_tr_b16 %1, %2 offset:%4" : "=&v"(lo), "=&v"(hi) : "v"(a_addr[f] + block * DY_BYTES), "n"(at), "n"(at + 512));
            af[set][f] = u32x4_t{lo[0], lo[1], hi[0], hi[1]};
        } else {
            constexpr int tap = f - 2, at = buf * BLOCK_BYTES + ks * 32 * 64;
            asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%4\n\tds_read_b64_tr_b16 %1, %3 offset:%4" : "=&v"(lo), "=&v"(hi) : "v"(b_addr[tap][0] + block * BLOCK_BYTES), "v"(b_addr[tap][1] + block * BLOCK_BYTES), "n"(at));
            bf[set][tap] = u32x4_t{lo[0], lo[1], hi[0], hi[1]};
        }
    };
    auto landed = [&](auto set_) __attribute__((always_inline)) {
        constexpr int set = decltype(set_)::value;
        __builtin_amdgcn_s_waitcnt((0xF) | (0x3 << 14) | (0x7 << 4) | (0x0 << 8));   // lgkmcnt(0)
        static_for<2>([&](auto m) { keep_alive(af[set][m]); });
        static_for<9>([&](auto tap) { keep_alive(bf[set][tap]); });
    };
    // Multiplies set `set`; beside the first MFMAs the other set is read (k-step ks of the k-tile in buffer buf), beside the last ones, in a
    // phase behind a barrier, stage kt_load is requested into buffer fill.
    auto phase = [&](auto set_, auto buf_, auto ks_, auto fill_, int kt_load) __attribute__((always_inline)) {
        constexpr int set = decltype(set_)::value, fill = decltype(fill_)::value;
        static_for<18>([&](auto i_) {
            constexpr int i = decltype(i_)::value;
            mfma16_v<DT>(acc[i & 1][i >> 1], bf[set][i >> 1], af[set][i & 1]);
            if constexpr (i < 11) read(std::integral_constant<int, 1 - set>{}, i_, buf_, ks_, 0);
            else if constexpr (fill >= 0 && i - 11 < COPIES) copy(std::integral_constant<int, i - 11>{}, fill, kt_load);
        });
        landed(std::integral_constant<int, 1 - set>{});
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    // copies of the stage in buffer b: block 0 of x is written twice
    constexpr auto copies_of = [](int b) { return COPIES + ((b + 1) % BLOCKS == 0 ? X_SLOTS : 0); };

    // x block 0 (as the last slots of a stage -1), then stages 0, 1, 2
    static_for<X_SLOTS>([&](auto j) { copy(std::integral_constant<int, DY_SLOTS + decltype(j)::value>{}, BLOCKS - 1, -1); });
    static_for<3>([&](auto st) { static_for<COPIES>([&](auto i) { copy(i, st, decltype(st)::value); }); });
    // k-tile kt in buffer u, its first k-step's fragments in registers
    auto tile = [&](auto u_, int kt) __attribute__((always_inline)) {
        constexpr int u = decltype(u_)::value, nxt = (u + 1) % 4;
        if constexpr (ST == 1) phase(I0{}, u_, I1{}, std::integral_constant<int, -1>{}, 0);
        // stage kt + 1 is there, kt + 2 on its way; every wave is past k-tile kt - 1, whose buffers stage kt + 3 takes
        pipeline_barrier<copies_of((u + 2) % 4)>();
        phase(std::integral_constant<int, ST == 1 ? 1 : u & 1>{}, std::integral_constant<int, nxt>{}, I0{}, std::integral_constant<int, (u + 3) % 4>{}, kt + 3);
    };
    // k-tile kt with what padded pixels multiply taken out: pixels in rows of Qp, rows in images of Pp
    auto careful = [&](int kt) __attribute__((always_inline)) {
        pipeline_barrier<0>();
        static_for<KT / 64>([&](auto ks) {
            static_for<11>([&](auto f) { read(I0{}, f, I0{}, ks, kt % 4); });
            landed(I0{});
            const int first = s0 + kt * KT + kg * (KT / 2) + (int)ks * 32 + 8 * g, rows = first / Qp;        // the lane's eight pixels
            int fq = first - rows * Qp, fp = rows % Pp;
            uint32_t real = 0;
#pragma clang loop unroll(disable)
            for (int e = 0; e < 8; ++e) {
                if (fq < a.Q && fp < a.P && first + e < a.px) real |= 1u << e;
                const bool end = ++fq == Qp;
                fq = end ? 0 : fq;
                fp = end ? (fp + 1 == Pp ? 0 : fp + 1) : fp;
            }
            u32x4_t mask;
#pragma unroll
            for (int j = 0; j < 4; ++j) mask[j] = (real >> (2 * j) & 1) * 0xffffu | (real >> (2 * j + 1) & 1) * 0xffff0000u;
            static_for<9>([&](auto tap) { bf[0][tap] &= mask; keep_alive(bf[0][tap]); });
            asm volatile("s_nop 3");                              // (the MFMAs are asm too: nobody else counts the wait states behind the ANDs)
            static_for<18>([&](auto i) { mfma16_v<DT>(acc[i & 1][i >> 1], bf[0][i >> 1], af[0][i & 1]); });
        });
        pipeline_barrier<0>();                                    // (stage kt + 3's block of x takes the place of k-tile kt's)
        static_for<COPIES>([&](auto i) { copy(i, (kt + 3) % 4, kt + 3); });
    };
    if constexpr (!PADDING_OUT) {
        pipeline_barrier<copies_of(1) + copies_of(2)>();
        static_for<11>([&](auto f) { read(I0{}, f, I0{}, I0{}, 0); });
        landed(I0{});
        for (int kt = 0;;) {
            tile(I0{}, kt);
            if (++kt >= KTn) break;
            tile(I1{}, kt);
            if (++kt >= KTn) break;
            tile(std::integral_constant<int, 2>{}, kt);
            if (++kt >= KTn) break;
            tile(std::integral_constant<int, 3>{}, kt);
            if (++kt >= KTn) break;
        }
    } else {
#pragma clang loop unroll(disable)
        for (int kt = 0; kt < KTn; ++kt) careful(kt);
    }
    __builtin_amdgcn_s_waitcnt((0xF) | (0x3 << 14) | (0x7 << 4) | (0x0 << 8));
    asm volatile("s_nop 15");
    asm volatile("s_nop 15");

    // ---- the groups' sums meet in LDS; rows of 32 channels per (filter, tap) from there ------------------------------
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __syncthreads();
    float *const meet = (float *)smem;
    static_for<2>([&](auto mi) {
        static_for<9>([&](auto tap) {
            *(f32x4_t *)(meet + (kg * 64 + wm * 32 + mi * 16 + l) * LD + tap * 32 + wn * 16 + 4 * g) = acc[mi][tap];
        });
    });
    __syncthreads();
    float nan = 0.f;                                              // (one at the latest where a sum is)
    const int64_t row_elems = 9 * (int64_t)a.C;
    static_for<9>([&](auto i) {
        const int u = i * 512 + tid, ko = u / 72, rest = u - ko * 72, tap = rest >> 3, c = (rest & 7) * 4;
        const f32x4_t v = *(const f32x4_t *)(meet + ko * LD + tap * 32 + c) + *(const f32x4_t *)(meet + (64 + ko) * LD + tap * 32 + c);
        if constexpr (!PADDING_OUT) nan = __builtin_fmaf(v[2], v[3], __builtin_fmaf(v[0], v[1], nan));
        if (k0 + ko < a.Kout && c0 + c < a.C) {
            const int64_t at = (int64_t)(k0 + ko) * row_elems + tap * a.C + c0 + c;
            if (a.slices > 1) {
                __builtin_nontemporal_store(v, (f32x4_t *)(a.partials + (int64_t)slice * a.Kout * row_elems + at));
            } else if (a.dtD == UCL_F32) {
                *(f32x4_t *)((float *)a.dw + at) = v * a.alpha;
            } else {
                uint32_t b[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) b[e] = f32_to_bits16(v[e] * a.alpha, a.dtD);
                *(u32x2_t *)((uint16_t *)a.dw + at) = u32x2_t{b[0] | (b[1] << 16), b[2] | (b[3] << 16)};
            }
        }
    });
    if constexpr (PADDING_OUT) return false;
    // (beside the stores, which nobody waits for)
    uint32_t *const nans = (uint32_t *)(smem + MEET_BYTES);
    const bool any = __ballot(__builtin_isnan(nan)) != 0;
    if (lane == 0) nans[wave] = any;
    pipeline_barrier<63>();
    const u32x4_t f = *(const u32x4_t *)nans | *(const u32x4_t *)(nans + 4);
    return __builtin_amdgcn_readfirstlane(f[0] | f[1] | f[2] | f[3]) != 0;
}

template <int DT, int ST>
__global__ __launch_bounds__(512, 2) void wgrad_taps_kernel(const WgradTaps a) {
    __shared__ __attribute__((aligned(1024))) char smem[TapsLds<ST>::BYTES];
    if (__builtin_expect(!wgrad_taps_pass<DT, ST, false>(a, smem), 1)) return;
    __syncthreads();                                              // (the stores are out, and the next copies go where sums and flags were read)
    wgrad_taps_pass<DT, ST, true>(a, smem);
}

template <int DT>
hipError_t launch_wgrad_taps(const KParams &p, const GroupTable *, int grid, hipStream_t stream) {
    WgradTaps a;
    a.dy = p.A; a.x = p.B; a.dw = p.D; a.partials = p.ws_partials;
    a.n_img = p.K / (p.cP * p.cQ); a.P = p.cP; a.Q = p.cQ; a.H = p.cH; a.W = p.cW; a.C = p.cC; a.Kout = p.M;
    a.tiles_k = (p.M + 63) / 64; a.tiles_c = (p.cC + 31) / 32;
    a.slices = p.split_k; a.px_per_slice = p.k_per_slice; a.px = a.n_img * (a.P + 1) * (a.Q + 1);
    const int kt = p.str_h == 1 ? 128 : 64, row = a.Q + 1, img = (a.P + 1) * row;
    a.step_n = kt / img; a.step_p = kt % img / row; a.step_q = kt % img % row;
    a.rcp_q = 1.f / (float)row; a.rcp_p = 1.f / (float)(a.P + 1);
    a.dtD = p.dtD;
    a.alpha = p.fused.has_scale ? p.fused.alpha : 1.f;
    a.dy_bytes = (uint32_t)((int64_t)p.K * p.M * 2);
    a.x_bytes = (uint32_t)p.b_bytes;
    if (p.str_h == 1) hipLaunchKernelGGL((wgrad_taps_kernel<DT, 1>), dim3((unsigned)grid), dim3(512), 0, stream, a);
    else hipLaunchKernelGGL((wgrad_taps_kernel<DT, 2>), dim3((unsigned)grid), dim3(512), 0, stream, a);
    return hipGetLastError();
}

}  // namespace ucl

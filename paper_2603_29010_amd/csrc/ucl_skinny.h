// Kernel for problems of few rows (decoding: 1 .. 64 tokens against a weight matrix) or few tiles: gemm / batched_gemm /
// grouped_gemm with both operands contiguous along K.
//
// Such a call is a read of B.  The tile kernel walks B through LDS in 64-column tiles: 64 workgroups for 4096 columns,
// each one serial chain of k-tiles.  Here a workgroup owns a narrow strip of 16 * NI columns and 16 * MI rows and its W
// waves take the 64-wide steps of K in turn, each wave on its own: it copies its step's rows (128-byte lines, eight rows per
// copy) into stage buffers of its own in LDS, waits for its own copies only and multiplies; no barrier until the sums of
// the waves meet in LDS, in wave order (a fixed order).  The chain runs there, 8 consecutive columns per thread, with the
// element-wise functions of the tile kernel.
// Bound by what a CU copies: 100 to 110 GB/s of the 112 to 130 that copies of whole lines reach from L2 (16 KB in flight are
// enough for that: the tile kernels' 64 GB/s are their barriers').  Loading the fragments straight into registers was tried
// first: sixteen consecutive lanes then read sixteen different rows, and a CU takes in 38 GB/s whatever is in flight.
// What the chain reads (bias, residual) is requested at the start: at the end it cost another trip to memory (0.3 us of 5).
// 64x64 tiles have eight waves and one stage buffer each: a step's fragments go to registers, the buffer is refilled while they are
// multiplied.  No barrier in the loop and half the LDS reads of 32x32 wave tiles; ahead of the tile kernel with two K groups where rows
// are not whole 128-byte lines, which it feels more: 1000x1001x1992 fp16 16.0 -> 14.3 us by themselves (K = 1984: 13.2 -> 12.9 us), 13.0 us with the
// chain's operands requested first and bands of 512 rows.  64x64 tiles of four waves with two stages, or with steps of 128, were slower (16.0
// and 15.0 us).  Every wave has one step on its way: with tiles for fewer than half of the CUs that is too little from memory (few_rows_apply).
// Measured, 64x64x64x4 tiles with two K groups -> here: 16x4096x4096 bf16 14.5 -> 8.5 us (18.2 before the K groups; the
// weight's trip from memory is 6.8), 2x792x7744 21.5 -> 8.4 us, 185x584x6960 34.5 -> 12.3 us, 305x336x1984 10.0 -> 6.2 us.
#pragma once
#include "ucl_kernel.h"
#include "ucl_variants.h"

namespace ucl {

template <int MI_, int NI_, int W_ /*waves*/, int S_ /*stage buffers per wave*/, int DT_, int MODE_ /*0 gemm + batched, 1 grouped, 2 conv fprop*/>
struct SkinnyCfg {
    static constexpr int MI = MI_, NI = NI_, W = W_, S = S_, DT = DT_, MODE = MODE_;
    static constexpr int TM = MI * 16, TN = NI * 16, THREADS = W * 64;
    static constexpr int STEP = 64;                               // k (pairs of k for 8-bit inputs) per step: rows of 128 bytes
    static constexpr int STAGE_BYTES = (TM + TN) * 128;
    static constexpr int LD = TN + 4;                             // floats per row where the sums meet (padding against bank conflicts)
    static constexpr int MEET_BYTES = W * TM * LD * 4;
    static constexpr int LDS_BYTES = W * S * STAGE_BYTES > MEET_BYTES ? W * S * STAGE_BYTES : MEET_BYTES;
    static constexpr int PER_CU = kLdsBytesPerCU / LDS_BYTES * W / 4 > 4 ? 4 : kLdsBytesPerCU / LDS_BYTES * W / 4;   // waves per SIMD
    static_assert(W == 4 || W == 8, "one or two waves per SIMD");
    static_assert(LDS_BYTES <= kLdsBytesPerCU, "stage buffers exceed LDS");
    static_assert(S > 1 || MODE != 2, "gathered copies step through the taps and are issued for every step");
    static constexpr int UNITS = TM * TN / 8, UPT = (UNITS + THREADS - 1) / THREADS;      // 8-column pieces of the output, per thread
    using Groups = typename std::conditional<MODE == 1, GroupTable, NoGroupTable>::type;
};

template <int DT>
__device__ __forceinline__ f32x4_t mfma_step(const u32x4_t &a, const u32x4_t &b, f32x4_t c) {
    if constexpr (DT == 0) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
    } else if constexpr (DT == 1) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
    } else {
        // 8-bit inputs: a 16-byte fragment holds 16 consecutive k, its halves go through one 32-deep MFMA each (see mfma16)
        const long a0 = __builtin_bit_cast(long, u32x2_t{a[0], a[1]}), a1 = __builtin_bit_cast(long, u32x2_t{a[2], a[3]});
        const long b0 = __builtin_bit_cast(long, u32x2_t{b[0], b[1]}), b1 = __builtin_bit_cast(long, u32x2_t{b[2], b[3]});
        if constexpr (DT == 2) {
            c = __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a0, b0, c, 0, 0, 0);
            return __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a1, b1, c, 0, 0, 0);
        } else {
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf8_bf8(a0, b0, c, 0, 0, 0);
            return __builtin_amdgcn_mfma_f32_16x16x32_bf8_bf8(a1, b1, c, 0, 0, 0);
        }
    }
}

template <class Cfg>
__global__ __launch_bounds__(Cfg::THREADS, Cfg::PER_CU) void ucl_skinny_kernel(const KParams p_arg, const typename Cfg::Groups gt) {
    constexpr int MI = Cfg::MI, NI = Cfg::NI, W = Cfg::W, S = Cfg::S, TM = Cfg::TM, TN = Cfg::TN, LD = Cfg::LD, MODE = Cfg::MODE;
    __shared__ __attribute__((aligned(1024))) char smem[Cfg::LDS_BYTES];
    // (the arguments are read through a pointer into the argument segment: the chain is indexed at run time)
    typedef const __attribute__((address_space(4))) KParams ConstKParams;
    ConstKParams &p = *(ConstKParams *)__builtin_amdgcn_kernarg_segment_ptr();
    (void)p_arg;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int first_tile = 0;
    if constexpr (MODE == 1) first_tile = gt.tile_start[lane];
    touch_arguments<MODE>(p);
    int t = xcd_remap(blockIdx.x, p.total_tiles);
    int batch = 0, group = -1, tm, tn, Mloc = p.M;
    const char *Ab = (const char *)p.A, *Bb = (const char *)p.B;
    char *Db = (char *)p.D;
    if constexpr (MODE == 1) {
        group = find_group_wave(gt, first_tile, p.groups, t, lane);
        const void *a_g = p.A_g[group], *b_g = p.B_g[group], *d_g = p.D_g[group];
        t -= gt.tile_start[group];
        Mloc = gt.m[group];
        band_raster(t, (Mloc + TM - 1) / TM, p.tiles_n, p.raster, tm, tn);
        Ab = uniform_ptr((const char *)a_g);
        Bb = uniform_ptr((const char *)b_g);
        Db = (char *)uniform_ptr((const char *)d_g);
    } else {
        batch = t / p.tiles_per_batch;
        t -= batch * p.tiles_per_batch;
        band_raster(t, p.tiles_m, p.tiles_n, p.raster, tm, tn);
        Ab += (int64_t)batch * p.a_bs * 2;
        Bb += (int64_t)batch * p.b_bs * 2;
    }
    const int m0 = tm * TM, n0 = tn * TN, K = p.K;

    const int a_rows = Mloc - m0 < TM ? Mloc - m0 : TM, b_rows = p.N - n0 < TN ? p.N - n0 : TN;
    // ---- the chain's operands, requested first: at the end they would cost another trip to memory --------------------
    const __attribute__((address_space(4))) FusedEpi &f = p.fused;
    constexpr int UPT = Cfg::UPT;
    Raw8 bias_raw[UPT], res_raw[UPT];
    static_for<UPT>([&](auto q) {
        const int u = q * Cfg::THREADS + tid, row = u / (TN / 8), n = n0 + (u % (TN / 8)) * 8;
        const int nvalid = row < a_rows ? p.N - n : 0;
        if (f.enabled && f.has_bias) bias_raw[q] = load8(group >= 0 ? ((const void *const *)f.bias)[group] : f.bias, f.bias_dt & 0xff, n, nvalid);
        if (f.enabled && f.has_res)
            res_raw[q] = load8(group >= 0 ? ((const void *const *)f.res)[group] : f.res, f.res_dt & 0xff,
                               (int64_t)batch * f.res_bs + (int64_t)(m0 + row) * f.res_ld + n, nvalid);
    });

    // ---- copies: a wave instruction fills eight rows of 128 bytes, chunks XORed by row as in the tile kernel ----------
    // Buffer resources over the rows that exist: rows past the edge and (by an out-of-range offset) k past the end
    // land as zeros and cost no traffic.
    const int f_row = lane & 15, f_kg = lane >> 4;
    const rsrc_t a_rsrc = MODE == 2 ? buffer_rsrc(Ab, (uint32_t)p.a_bytes)
                                    : buffer_rsrc(Ab + (int64_t)m0 * p.lda * 2, (uint32_t)(((int64_t)(a_rows - 1) * p.lda + K) * 2));
    const rsrc_t b_rsrc = buffer_rsrc(Bb + (int64_t)n0 * p.ldb * 2, (uint32_t)(((int64_t)(b_rows - 1) * p.ldb + K) * 2));
    constexpr int CA = TM / 8, CB = TN / 8;                       // copies per step
    const int c_row = lane >> 3;
    // (swz(row + 8) = swz(row) ^ 1: two chunk positions serve all of a wave's copies)
    const int kc[2] = {((lane & 7) ^ lds_swz<8>(c_row)) * 8, ((lane & 7) ^ lds_swz<8>(c_row + 8)) * 8};
    uint32_t a_off[CA], b_off[CB];
    // conv: the row's output pixel as its first tap's input pixel, and the (tap, channel) each chunk position stands at
    int a_h0[MODE == 2 ? CA : 1], a_w0[MODE == 2 ? CA : 1], t_c[2], t_r[2], t_s[2];
    if constexpr (MODE == 2) {
#pragma unroll
        for (int i = 0; i < CA; ++i) {
            const bool there = i * 8 + c_row < a_rows;
            const int row = m0 + (there ? i * 8 + c_row : 0);
            const int pq = row / p.cQ, q = row - pq * p.cQ, nb = pq / p.cP, pp = pq - nb * p.cP;
            a_h0[i] = there ? pp * p.str_h - p.pad_h : -(1 << 28);       // (a row past the edge: outside every image)
            a_w0[i] = q * p.str_w - p.pad_w;
            a_off[i] = (uint32_t)(((nb * p.cH + a_h0[i]) * p.cW + a_w0[i]) * p.cC * 2);      // (only used at taps inside the image)
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k = wave * Cfg::STEP + kc[h], tap = k / p.cC;
            t_c[h] = k - tap * p.cC;
            t_r[h] = tap / p.cS;
            t_s[h] = tap - t_r[h] * p.cS;
        }
    } else {
#pragma unroll
        for (int i = 0; i < CA; ++i) a_off[i] = i * 8 + c_row < a_rows ? (uint32_t)(((int64_t)(i * 8 + c_row) * p.lda + kc[i & 1]) * 2) : kOobOffset;
    }
#pragma unroll
    for (int i = 0; i < CB; ++i) b_off[i] = i * 8 + c_row < b_rows ? (uint32_t)(((int64_t)(i * 8 + c_row) * p.ldb + kc[i & 1]) * 2) : kOobOffset;
    char *const mine = smem + wave * (S * Cfg::STAGE_BYTES);
    constexpr int COPIES = CA + CB;
    auto copy = [&](int step, auto stage_) __attribute__((always_inline)) {
        char *dst = mine + decltype(stage_)::value * Cfg::STAGE_BYTES;
        const int k = step * Cfg::STEP;
        const bool ok[2] = {k + kc[0] < K, k + kc[1] < K};
        static_for<CB>([&](auto i) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(b_rsrc, UCL_LDS_PTR(dst + i * 1024), 16, ok[i & 1] ? b_off[i] : kOobOffset, k * 2, 0, 0);
        });
        if constexpr (MODE == 2) {
            // (steps come in order, W apart: the taps move on with every call)
            uint32_t tap_off[2];
            int dh[2], dw[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                dh[h] = t_r[h] * p.dil_h;
                dw[h] = t_s[h] * p.dil_w;
                tap_off[h] = (uint32_t)(((dh[h] * p.cW + dw[h]) * p.cC + t_c[h]) * 2);
            }
            static_for<CA>([&](auto i) {
                const int h = a_h0[i] + dh[i & 1], w = a_w0[i] + dw[i & 1];
                const bool in = ok[i & 1] && (unsigned)h < (unsigned)p.cH && (unsigned)w < (unsigned)p.cW;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, UCL_LDS_PTR(dst + TN * 128 + i * 1024), 16, in ? a_off[i] + tap_off[i & 1] : kOobOffset, 0, 0, 0);
            });
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                t_c[h] += W * Cfg::STEP;
                while (t_c[h] >= p.cC) {
                    t_c[h] -= p.cC;
                    if (++t_s[h] == p.cS) { t_s[h] = 0; ++t_r[h]; }
                }
            }
        } else {
            static_for<CA>([&](auto i) {
                __builtin_amdgcn_raw_ptr_buffer_load_lds(a_rsrc, UCL_LDS_PTR(dst + TN * 128 + i * 1024), 16, ok[i & 1] ? a_off[i] : kOobOffset, k * 2, 0, 0);
            });
        }
    };
    f32x4_t acc[MI][NI];
    static_for<MI>([&](auto i) { static_for<NI>([&](auto j) { acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f}; }); });
    // (B as the first operand: a lane then holds 4 consecutive columns of one row)
    const int f_x = lds_swz<8>(f_row);
    u32x4_t fa[2][MI], fb[2][NI];
    auto fetch = [&](auto stage_) __attribute__((always_inline)) {
        const char *src = mine + decltype(stage_)::value * Cfg::STAGE_BYTES + f_row * 128;
        static_for<2>([&](auto h) {
            const int x = ((h * 4 + f_kg) ^ f_x) << 4;
            static_for<NI>([&](auto j) { fb[h][j] = *(const u32x4_t *)(src + j * 2048 + x); });
            static_for<MI>([&](auto i) { fa[h][i] = *(const u32x4_t *)(src + TN * 128 + i * 2048 + x); });
        });
    };
    auto multiply = [&]() __attribute__((always_inline)) {
        static_for<2>([&](auto h) {
            static_for<MI>([&](auto i) { static_for<NI>([&](auto j) { acc[i][j] = mfma_step<Cfg::DT>(fb[h][j], fa[h][i], acc[i][j]); }); });
        });
    };
    // Wave w takes steps w, w + W, ...; S - 1 of them are in flight while one is multiplied.  The copies are
    // unconditional (past the end of K they read nothing), so what is waited for is always the oldest step alone.
    const int steps = (K + Cfg::STEP - 1) / Cfg::STEP;
    if constexpr (S == 1) {
        // one stage buffer: all of a step's fragments go to registers, then its buffer is refilled while they are multiplied
        copy(wave, std::integral_constant<int, 0>{});
        for (int c = wave; c < steps; c += W) {
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
            asm volatile("" ::: "memory");
            fetch(std::integral_constant<int, 0>{});
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt((0xF) | (0x3 << 14) | (0x7 << 4) | (0x0 << 8));   // lgkmcnt(0)
            __builtin_amdgcn_sched_barrier(0);
            if (c + W < steps) copy(c + W, std::integral_constant<int, 0>{});
            multiply();
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        static_for<S - 1>([&](auto d) { copy(wave + d * W, d); });
        for (int c = wave; c < steps;) {
            static_for<S>([&](auto d) {
                copy(c + (S - 1) * W, std::integral_constant<int, (decltype(d)::value + S - 1) % S>{});
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_waitcnt(vmcnt_imm((S - 1) * COPIES));
                asm volatile("" ::: "memory");
                fetch(d);
                multiply();
                __builtin_amdgcn_sched_barrier(0);     // (its buffer is refilled next: every read of it has returned by then)
                c += W;
            });
        }
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __syncthreads();                               // every wave is done with its stage buffers
    float *const part = (float *)smem;

    // ---- the waves' sums meet in LDS; 8 consecutive columns of a row per thread from here on ---------------------
    static_for<MI>([&](auto i) {
        static_for<NI>([&](auto j) { *(f32x4_t *)(part + (wave * TM + i * 16 + f_row) * LD + j * 16 + f_kg * 4) = acc[i][j]; });
    });
    __syncthreads();
    typedef const __attribute__((address_space(4))) EpiStepDev ConstStep;
    ConstStep *const ksteps = (ConstStep *)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(KParams, steps));
    static_for<UPT>([&](auto q) {
        const int u = q * Cfg::THREADS + tid;
        const int row = u / (TN / 8), col = (u % (TN / 8)) * 8;
        EpiCtx cx;
        cx.m = m0 + row;
        cx.n = n0 + col;
        cx.nvalid = row < a_rows ? p.N - cx.n : 0;
        cx.batch = batch;
        cx.group = group;
        if (u >= Cfg::UNITS || cx.nvalid <= 0) return;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = 0.f;
        static_for<W>([&](auto w) {
            const f32x4_t lo = *(const f32x4_t *)(part + (w * TM + row) * LD + col), hi = *(const f32x4_t *)(part + (w * TM + row) * LD + col + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] += lo[e];
                v[4 + e] += hi[e];
            }
        });
        if (f.enabled) {
            // act(alpha * acc + bias[n] + beta * R[m, n])
            float b8[8], r8[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) b8[e] = 0.f;
            if (f.has_bias) decode8(bias_raw[q], f.bias_dt & 0xff, b8);
            const float alpha = f.has_scale ? f.alpha : 1.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = v[e] * alpha + b8[e];
            if (f.has_res) {
                decode8(res_raw[q], f.res_dt & 0xff, r8);
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] += f.beta * r8[e];
            }
            switch (f.act) {
#define UCL_ACT_CASE(OP)                                                                                    \
    case OP:                                                                                                \
        _Pragma("unroll") for (int e = 0; e < 8; ++e) v[e] = act_f32<OP>(v[e], f.act_p0, f.act_p1);          \
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
        } else {
            Raw8 none;
            none.lo = none.hi = u32x4_t{0, 0, 0, 0};
            none.packed = false;
            for (int s = 0; s < p.n_steps; ++s) {
                EpiStepDev st;
                st.op = ksteps[s].op; st.dtype = ksteps[s].dtype; st.p0 = ksteps[s].p0; st.p1 = ksteps[s].p1;
                st.ptr = ksteps[s].ptr; st.ld = ksteps[s].ld; st.bs = ksteps[s].bs;
                apply_step(v, st, cx, none, false);
            }
        }
        store8(Db, p.dtD, (MODE == 1 ? 0 : (int64_t)batch * p.d_bs) + cx.m * p.ldd + cx.n, v, cx.nvalid);
    });
}

template <class Cfg>
hipError_t launch_skinny(const KParams &p, const GroupTable *gt, int grid, hipStream_t stream) {
    if constexpr (Cfg::MODE == 1) {
        hipLaunchKernelGGL(ucl_skinny_kernel<Cfg>, dim3(grid), dim3(Cfg::THREADS), 0, stream, p, *gt);
    } else {
        (void)gt;
        hipLaunchKernelGGL(ucl_skinny_kernel<Cfg>, dim3(grid), dim3(Cfg::THREADS), 0, stream, p, NoGroupTable{});
    }
    return hipGetLastError();
}

// Two stage depths of one tile: with a workgroup per CU at most, what is in flight are the stages of its waves; with more, workgroups that
// share a CU have as much in flight with one buffer each, and one's start and end hide under the others' copies.  (32 rows, 64 columns,
// three stages -> one buffer: 64x16384x1024 bf16, 512 tiles 14.3 -> 10.3 us; 16x16: 16x4096x4096, 256 tiles 8.7 us with four stages, 10.5 us with one.
// 3000 problems of more tiles than CUs and K from 272 to 4096, decoding, batched or tall: 0.4 to 0.98 of the time with one buffer, least for short K and
// many tiles; 16x16 tiles at K above 2048 the 0.98, so the line is drawn at 4096.  Beyond it, 3900 problems up to K = 16384: 16x16 tiles 0.96
// to 1.09, the others 0.82 to 1.01; nothing prices them there.)
template <class Deep, class One>
hipError_t launch_skinny_pair(const KParams &p, const GroupTable *gt, int grid, hipStream_t stream) {
    return takes_one_buffer(grid, p.K) ? launch_skinny<One>(p, gt, grid, stream) : launch_skinny<Deep>(p, gt, grid, stream);
}

// (stages 1 tells these from the tile kernels of the same shape; k_groups = waves)
template <class Cfg>
constexpr VariantDesc describe_skinny() {
    return VariantDesc{Cfg::TM, Cfg::TN, 64, 1, Cfg::DT, Cfg::MODE, Cfg::MODE == 2 ? 2 : 0, 0, Cfg::LDS_BYTES, 0, kLdsBytesPerCU / Cfg::LDS_BYTES, Cfg::W, 0, &launch_skinny<Cfg>, nullptr};
}

template <int MI, int NI, int S, int DT, int MODE>
constexpr VariantDesc describe_skinny_pair() {
    VariantDesc v = describe_skinny<SkinnyCfg<MI, NI, 4, S, DT, MODE>>();
    v.launch = &launch_skinny_pair<SkinnyCfg<MI, NI, 4, S, DT, MODE>, SkinnyCfg<MI, NI, 4, 1, DT, MODE>>;
    return v;
}

// A kernel of one buffer per wave under a name of its own: the stages it has are those of its waves together.
template <class Cfg>
constexpr VariantDesc describe_one_buffer() {
    static_assert(Cfg::S == 1, "one stage buffer per wave");
    VariantDesc v = describe_skinny<Cfg>();
    v.stages = Cfg::W;
    return v;
}

}  // namespace ucl

// Kernel for problems of few rows (decoding: 1 .. 64 tokens against a weight matrix): gemm / batched_gemm /
// grouped_gemm with both operands contiguous along K.
//
// Such a call is a read of B.  The tile kernel walks B through LDS in 64-column tiles: 64 workgroups for 4096 columns,
// each a serial chain of k-tiles with a few ten KB in flight.  Here a workgroup owns a narrow strip of 16 * NI columns and
// 16 * MI rows, its W waves take the chunks of K in turn, and every wave loads its MFMA fragments straight into registers
// (a fragment is 16 bytes of one row per lane, which is what the matrix instruction wants: nothing is shared between
// waves, so LDS would only add a trip), two chunks in flight.  The waves' sums meet in LDS in wave order (a fixed
// order) and the chain runs there, 8 consecutive columns per lane, with the element-wise functions of the tile kernel.
#pragma once
#include "ucl_kernel.h"
#include "ucl_variants.h"

namespace ucl {

template <int MI_, int NI_, int W_ /*waves*/, int U_ /*32-wide k steps per chunk*/, int DT_, int MODE_ /*0 gemm + batched, 1 grouped*/>
struct SkinnyCfg {
    static constexpr int MI = MI_, NI = NI_, W = W_, U = U_, DT = DT_, MODE = MODE_;
    static constexpr int TM = MI * 16, TN = NI * 16, THREADS = W * 64;
    static constexpr int LD = TN + 4;                             // floats per staged row (padding against bank conflicts)
    static constexpr int LDS_BYTES = W * TM * LD * 4;
    static constexpr int CHUNK = U * 32;                          // k (pairs of k for 8-bit inputs) per chunk
    static_assert(W == 4 || W == 8, "one or two waves per SIMD");
    static_assert(LDS_BYTES <= 64 * 1024, "two workgroups per CU");
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
__global__ __launch_bounds__(Cfg::THREADS, Cfg::W / 4) void ucl_skinny_kernel(const KParams p_arg, const typename Cfg::Groups gt) {
    constexpr int MI = Cfg::MI, NI = Cfg::NI, W = Cfg::W, U = Cfg::U, TM = Cfg::TM, TN = Cfg::TN, LD = Cfg::LD, MODE = Cfg::MODE;
    __shared__ __attribute__((aligned(16))) float part[W * TM * LD];
    // (the arguments are read through a pointer into the argument segment: the chain is indexed at run time)
    typedef const __attribute__((address_space(4))) KParams ConstKParams;
    ConstKParams &p = *(ConstKParams *)__builtin_amdgcn_kernarg_segment_ptr();
    (void)p_arg;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int t = xcd_remap(blockIdx.x, p.total_tiles);
    int batch = 0, group = -1, tm, tn, Mloc = p.M;
    const char *Ab = (const char *)p.A, *Bb = (const char *)p.B;
    char *Db = (char *)p.D;
    if constexpr (MODE == 1) {
        group = find_group(gt.tile_start, p.groups, t);
        t -= gt.tile_start[group];
        Mloc = gt.m[group];
        band_raster(t, (Mloc + TM - 1) / TM, p.tiles_n, p.raster, tm, tn);
        Ab = uniform_ptr((const char *)p.A_g[group]);
        Bb = uniform_ptr((const char *)p.B_g[group]);
        Db = (char *)uniform_ptr((const char *)p.D_g[group]);
    } else {
        batch = t / p.tiles_per_batch;
        t -= batch * p.tiles_per_batch;
        band_raster(t, p.tiles_m, p.tiles_n, p.raster, tm, tn);
        Ab += (int64_t)batch * p.a_bs * 2;
        Bb += (int64_t)batch * p.b_bs * 2;
    }
    const int m0 = tm * TM, n0 = tn * TN, K = p.K;

    // ---- fragments: row lane % 16 of a 16-row block, 16 bytes at k = 8 * (lane / 16) of a 32-wide step ----------
    // Buffer resources over the rows that exist: rows past the edge and (by an out-of-range offset) k past the end
    // read zeros and cost no traffic.
    const int f_row = lane & 15, f_kg = lane >> 4;
    const int a_rows = Mloc - m0 < TM ? Mloc - m0 : TM, b_rows = p.N - n0 < TN ? p.N - n0 : TN;
    const rsrc_t a_rsrc = buffer_rsrc(Ab + (int64_t)m0 * p.lda * 2, (uint32_t)(((int64_t)(a_rows - 1) * p.lda + K) * 2));
    const rsrc_t b_rsrc = buffer_rsrc(Bb + (int64_t)n0 * p.ldb * 2, (uint32_t)(((int64_t)(b_rows - 1) * p.ldb + K) * 2));
    uint32_t a_off[MI], b_off[NI];
#pragma unroll
    for (int i = 0; i < MI; ++i) a_off[i] = i * 16 + f_row < a_rows ? (uint32_t)(((int64_t)(i * 16 + f_row) * p.lda + f_kg * 8) * 2) : kOobOffset;
#pragma unroll
    for (int i = 0; i < NI; ++i) b_off[i] = i * 16 + f_row < b_rows ? (uint32_t)(((int64_t)(i * 16 + f_row) * p.ldb + f_kg * 8) * 2) : kOobOffset;

    u32x4_t fa[2][U][MI], fb[2][U][NI];
    auto load = [&](auto set_, int chunk) __attribute__((always_inline)) {
        constexpr int set = decltype(set_)::value;
        static_for<U>([&](auto u) {
            const int k = chunk * Cfg::CHUNK + u * 32;
            const bool ok = k + f_kg * 8 < K;
            static_for<NI>([&](auto i) { fb[set][u][i] = __builtin_amdgcn_raw_buffer_load_b128(b_rsrc, ok ? b_off[i] : kOobOffset, k * 2, 0); });
            static_for<MI>([&](auto i) { fa[set][u][i] = __builtin_amdgcn_raw_buffer_load_b128(a_rsrc, ok ? a_off[i] : kOobOffset, k * 2, 0); });
        });
    };
    f32x4_t acc[MI][NI];
    static_for<MI>([&](auto i) { static_for<NI>([&](auto j) { acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f}; }); });
    // (B as the first operand: a lane then holds 4 consecutive columns of one row)
    auto multiply = [&](auto set_) __attribute__((always_inline)) {
        constexpr int set = decltype(set_)::value;
        static_for<U>([&](auto u) {
            static_for<MI>([&](auto i) { static_for<NI>([&](auto j) { acc[i][j] = mfma_step<Cfg::DT>(fb[set][u][j], fa[set][u][i], acc[i][j]); }); });
        });
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    const int chunks = (K + Cfg::CHUNK - 1) / Cfg::CHUNK;
    int c = wave;
    if (c < chunks) load(I0{}, c);
    while (c < chunks) {
        if (c + W < chunks) load(I1{}, c + W);
        multiply(I0{});
        c += W;
        if (c >= chunks) break;
        if (c + W < chunks) load(I0{}, c + W);
        multiply(I1{});
        c += W;
    }

    // ---- the waves' sums meet in LDS; 8 consecutive columns of a row per thread from here on ---------------------
    static_for<MI>([&](auto i) {
        static_for<NI>([&](auto j) { *(f32x4_t *)(part + (wave * TM + i * 16 + f_row) * LD + j * 16 + f_kg * 4) = acc[i][j]; });
    });
    __syncthreads();
    typedef const __attribute__((address_space(4))) EpiStepDev ConstStep;
    ConstStep *const ksteps = (ConstStep *)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(KParams, steps));
    const __attribute__((address_space(4))) FusedEpi &f = p.fused;
    constexpr int UNITS = TM * TN / 8;
#pragma clang loop unroll(disable)
    for (int u = tid; u < UNITS; u += Cfg::THREADS) {
        const int row = u / (TN / 8), col = (u % (TN / 8)) * 8;
        EpiCtx cx;
        cx.m = m0 + row;
        cx.n = n0 + col;
        cx.nvalid = row < a_rows ? p.N - cx.n : 0;
        cx.batch = batch;
        cx.group = group;
        if (cx.nvalid <= 0) continue;
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
            if (f.has_bias) {
                const void *bp = group >= 0 ? ((const void *const *)f.bias)[group] : f.bias;
                decode8(load8(bp, f.bias_dt & 0xff, cx.n, (f.bias_dt & 0x100) != 0, cx.nvalid), f.bias_dt & 0xff, b8);
            }
            const float alpha = f.has_scale ? f.alpha : 1.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = v[e] * alpha + b8[e];
            if (f.has_res) {
                const void *rp = group >= 0 ? ((const void *const *)f.res)[group] : f.res;
                decode8(load8(rp, f.res_dt & 0xff, (int64_t)batch * f.res_bs + cx.m * f.res_ld + cx.n, (f.res_dt & 0x100) != 0, cx.nvalid), f.res_dt & 0xff, r8);
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
        store8(Db, p.dtD, (MODE == 1 ? 0 : (int64_t)batch * p.d_bs) + cx.m * p.ldd + cx.n, v, p.d_vec != 0, cx.nvalid);
    }
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

// (tile_k 32, stages 1: operands are not staged; k_groups = waves; workgroups per CU from the register budget)
template <class Cfg>
constexpr VariantDesc describe_skinny() {
    return VariantDesc{Cfg::TM, Cfg::TN, 32, 1, Cfg::DT, Cfg::MODE, 0, 0, Cfg::LDS_BYTES, 0, 1, Cfg::W, 0, &launch_skinny<Cfg>, nullptr};
}

}  // namespace ucl

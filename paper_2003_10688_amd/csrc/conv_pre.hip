// 1x1 convolution with BN + ReLU on its input side, over whole 64-channel chunks (gfx950, bf16): the transitions of a DenseNet-shaped list.
//
// The map has to be applied between memory and the matrix instruction, so the register-staged kernel (conv_igemm.hip) takes
// every pixel row through registers into LDS and back, one chunk in flight.  But the map is per channel, and a 1x1 convolution's
// pixel fragment -- 8 consecutive channels of one pixel per lane -- lies in memory as the matrix instruction wants it: here a wave owns 32
// pixels and loads their fragments straight into registers, PD chunks of 64 channels ahead, applies the map there (28 instructions for
// 8 channels, constants from LDS), rounds to bf16 where the staged kernel does, and multiplies them with 128 filters, whose rows
// come through an LDS ring by DMA.  A pixel is transformed once per channel tile instead of once per wave that reads it.
// Bound by the length of a workgroup's path (operands, a few chunks, stores; two workgroups per CU), not by bytes: 103 MB in 44 us on the
// first of them.  Batch 64, us, register-staged kernel -> here: 256 -> 128 + 2x2 average pool at 56x56 54 -> 44, 512 -> 256 at 28x28 46 -> 35, 1024 ->
// 512 at 14x14 42 -> 30.  A ring of four stages: 47, 37, 30.  The constants written to LDS in front of the first operands' requests: 1.5 more each.
#include "conv_common.h"

namespace sol {

using lds_pipe::u32x4_t;

constexpr int PRE_CMAX = 1024;             // input channels whose constants fit beside the ring

// NS: ring stages (64 reduction elements of 128 filters); NS - 1 chunks of pixel fragments are in flight in registers
template <int NS>
__global__ void __launch_bounds__(256, 2) conv_pre_kernel(const ConvArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
    using namespace lds_pipe;
    constexpr int PD = NS - 1, BP = 128, BC = 128, TC = 4, STAGE = BC * 128, WL = 4;   // WL: DMA instructions (8 rows) per wave and stage
    static_assert(4 * 32 * (64 + 4) * 4 <= NS * STAGE, "epilogue strips go over the dead ring");
    __shared__ __align__(1024) unsigned char lds[NS * STAGE + PRE_CMAX * 8 + 1024];   // ring; input side's scale and shift [C]; output side's [128]
    const unsigned cst = lds_addr(lds) + NS * STAGE;

    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile = (int)(blockIdx.x & 7) * ((a.ntiles + 7) >> 3) + (int)(blockIdx.x >> 3);   // a contiguous run of tiles per XCD
    if (tile >= a.ntiles) return;
    const int p0 = (tile / a.ntc) * BP, c0 = (tile % a.ntc) * BC;

    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.w), 0, (int)((unsigned)a.Cout * a.Kp * 2u), 0x00020000);
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.x), 0, (int)((unsigned)a.N * a.H * a.W * a.ldx * 2u), 0x00020000);
    unsigned wo[WL];
#pragma unroll
    for (int i = 0; i < WL; i++) {
        const int row = (wave * WL + i) * 8 + (lane >> 3);
        wo[i] = (unsigned)(c0 + row) * (unsigned)(a.Kp * 2) + (((unsigned)(lane & 7) ^ (unsigned)swz<128>(row)) << 4);
    }
    const int nc = a.C >> 6;
    int is = 0;
    auto issue = [&](int slot) {                           // chunks beyond the last: out of range -> zeros
#pragma unroll
        for (int i = 0; i < WL; i++)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, (__attribute__((address_space(3))) void *)(lds + slot * STAGE + (wave * WL + i) * 1024), 16,
                                                     is < nc ? wo[i] + (unsigned)is * 128u : 0xffffffffu, 0, 0, 0);
        is++;
    };
    unsigned xo;
    {
        const int m = p0 + wave * 32 + lr;
        int n, op, oq;
        decode_pixel(a, m, n, op, oq);
        xo = m < a.P ? (unsigned)((n * a.H + op) * a.W + oq) * (unsigned)(a.ldx * 2) + (unsigned)(lh * 16) : 0x80000000u;
    }
    u32x4_t raw[PD][4];
    auto fetch = [&](u32x4_t (&to)[4], int c) {            // beyond the last chunk: the last again, never used
        const int s = min(c, nc - 1) * 128;
#pragma unroll
        for (int k = 0; k < 4; k++) to[k] = __builtin_amdgcn_raw_buffer_load_b128(xr, xo, s + k * 32, 0);
    };
    // The constants are asked for first and written to LDS behind the first operands' requests, by opaque stores (the compiler would make its
    // own wait for every DMA in flight)
    const int cc = min(tid * 4, a.C - 4), co = tid & 127;
    const f32x4_t ps = *reinterpret_cast<const f32x4_t *>(a.pre_scale + cc), ph = *reinterpret_cast<const f32x4_t *>(a.pre_shift + cc);
    const float *ap = tid < 128 ? a.scale : a.shift;
    const float av = ap ? ap[c0 + co] : tid < 128 ? 1.f : 0.f;
    // a chunk's filters, then its pixels: the order in which the loop goes on, and which its first wait counts on
    keep_order();
    static_for<PD>([&](auto S) {
        issue(decltype(S)::value);
        keep_order();
        fetch(raw[decltype(S)::value], decltype(S)::value);
        keep_order();
    });
    asm volatile("ds_write_b128 %0, %1" ::"v"(cst + (unsigned)cc * 4u), "v"(ps) : "memory");
    asm volatile("ds_write_b128 %0, %1" ::"v"(cst + (unsigned)(a.C + cc) * 4u), "v"(ph) : "memory");
    asm volatile("ds_write_b32 %0, %1" ::"v"(cst + PRE_CMAX * 8u + (unsigned)tid * 4u), "v"(av) : "memory");
    wait_lgkmcnt<0>();                                     // written; everyone's are behind the first chunk's barrier

    f32x16_t acc[TC];
#pragma unroll
    for (int i = 0; i < TC; i++)
#pragma unroll
        for (int e = 0; e < 16; e++) acc[i][e] = 0.f;
    const unsigned fsw = swz<128>(lr), fw = lds_addr(lds) + lr * 128, shift_at = (unsigned)(a.C * 4);
    int slot = 0;
    auto chunk = [&](auto U, int at) {                     // chunk `at`, whose pixels are in raw[U]
        constexpr int u = decltype(U)::value;
        // the chunk's filters have landed once what was issued behind them -- the filters of NS - 2 chunks, the pixels
        // of NS - 1 -- is all that is outstanding
        wait_vmcnt<(NS - 2) * WL + (NS - 1) * 4>();
        __builtin_amdgcn_s_barrier();
        const unsigned fb = fw + slot * STAGE, cb = cst + (unsigned)(at * 256 + lh * 32);
        u32x4_t fa[2][TC], k4[2][4];               // filters; scale and shift of the lane's 8 channels
        auto read = [&](auto KS, u32x4_t (&w)[TC], u32x4_t (&q)[4]) {
            constexpr int ks = decltype(KS)::value;
            lds_read16<ks * 64>(q[0], cb);
            lds_read16<ks * 64 + 16>(q[1], cb);
            lds_read16<ks * 64>(q[2], cb + shift_at);
            lds_read16<ks * 64 + 16>(q[3], cb + shift_at);
            static_for<TC>([&](auto I) { lds_read16<decltype(I)::value * 32 * 128>(w[decltype(I)::value], fb + (((2 * ks + lh) ^ fsw) << 4)); });
        };
        read(std::integral_constant<int, 0>{}, fa[0], k4[0]);
        issue(slot == 0 ? NS - 1 : slot - 1);
        static_for<4>([&](auto KS) {
            constexpr int ks = decltype(KS)::value, cur = ks & 1;
            if constexpr (ks < 3) {
                read(std::integral_constant<int, ks + 1>{}, fa[cur ^ 1], k4[cur ^ 1]);
                wait_lgkmcnt<4 + TC>();
            } else {
                wait_lgkmcnt<0>();
            }
            static_for<4>([&](auto I) { landed(k4[cur][decltype(I)::value]); });
            static_for<TC>([&](auto I) { landed(fa[cur][decltype(I)::value]); });
            u32x4_t b;
#pragma unroll
            for (int d = 0; d < 4; d++) {
                const uint32_t v = raw[u][ks][d];
                const float s0 = __uint_as_float(k4[cur][d >> 1][2 * (d & 1)]), s1 = __uint_as_float(k4[cur][d >> 1][2 * (d & 1) + 1]);
                const float h0 = __uint_as_float(k4[cur][2 + (d >> 1)][2 * (d & 1)]), h1 = __uint_as_float(k4[cur][2 + (d >> 1)][2 * (d & 1) + 1]);
                const float f0 = __uint_as_float(v << 16) * s0 + h0, f1 = __uint_as_float(v & 0xffff0000u) * s1 + h1;
                b[d] = pack_bf16x2(__builtin_fmaxf(f0, 0.f), __builtin_fmaxf(f1, 0.f));
            }
            static_for<TC>([&](auto I) { Mma<bf16_t>::run(acc[decltype(I)::value], fa[cur][decltype(I)::value], b); });
        });
        fetch(raw[u], at + PD);
        slot = slot + 1 == NS ? 0 : slot + 1;
    };
    // Whole turns, then what is left of one: a chunk skipped inside the loop would join its end, and the compiler, which then cannot know
    // what was requested last, waited at every other chunk for nearly everything (64 images of 7x7, 512 -> 256 11.6 -> 10.5 us without that,
    // 16 of 28x28, 1024 -> 128 18.1 -> 16.6)
    int c = 0;
    for (; c + PD <= nc; c += PD) static_for<PD>([&](auto U) { chunk(U, c + decltype(U)::value); });
    static_for<PD - 1>([&](auto U) {
        if (c + decltype(U)::value < nc) chunk(U, c + decltype(U)::value);
    });
    wait_vmcnt<0>();                                       // the DMAs beyond the last chunk
    __syncthreads();                                       // the ring becomes strips
    static_for<TC / 2>([&](auto H) {                       // 64 channels at a time
        constexpr int h = decltype(H)::value;
        f32x16_t part[2][1];
        part[0][0] = acc[2 * h];
        part[1][0] = acc[2 * h + 1];
        const int cw = c0 + h * 64;
        Affine8 aff;
        const float *c = reinterpret_cast<const float *>(lds + NS * STAGE + PRE_CMAX * 8) + h * 64 + (lane & 7) * 8;
#pragma unroll
        for (int e = 0; e < 8; e++) { aff.sc[e] = c[e]; aff.sf[e] = c[128 + e]; }
        ResidualRegs<bf16_t, 1, 2> res;
        prefetch_residual<bf16_t, 1, 2>(a, lane, p0 + wave * 32, cw, LinearRows{a.P}, res);
        conv_epilogue_auto<bf16_t, 1, 2>(a, part, reinterpret_cast<float *>(lds), wave, lane, p0 + wave * 32, cw, aff, LinearRows{a.P}, res);
    });
#endif
}

bool pre_kernel_applies(const ConvArgs &a, int dt) {
    return dt == SOL_BF16 && a.pre_scale && a.R == 1 && a.S == 1 && a.ph == 0 && a.pw == 0 && a.sh == 1 && a.sw == 1 && a.C % 64 == 0 && a.C <= PRE_CMAX && a.Cvalid == a.C &&
           a.ldx % 8 == 0 && a.Cout % 128 == 0 && (a.pool == 0 || a.pool == 1 || a.pool == 2) && (double)a.N * a.H * a.W * a.ldx * 2 < 2147483648.0 &&
           (double)a.Cout * a.Kp * 2 < 2147483648.0;
}

sol_status launch_conv_pre(const ConvArgs &in, hipStream_t st) {
    ConvArgs a = in;
    a.ntc = a.Cout / 128;
    a.ntiles = ceil_div(a.P, 128) * a.ntc;
    hipLaunchKernelGGL((conv_pre_kernel<3>), dim3(((a.ntiles + 7) / 8) * 8), dim3(256), 0, st, a);
    SOL_HIP(hipGetLastError());
    return SOL_OK;
}

}  // namespace sol

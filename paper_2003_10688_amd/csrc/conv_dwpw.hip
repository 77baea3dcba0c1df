// Depthwise 3x3 + pointwise 1x1 pair as ONE depth-first kernel (gfx950, bf16):
//
//     t = act(sd * dw3x3(x, wd) + hd)      depthwise, stride 1 or 2, pad 1       (one layer of a separable block)
//     y = act(s * (t . W) + h)             1x1, C -> K channels                 (the next)
//
// Run as two layers, t is written and read back and both launches pay their ramp-up and tail; the depthwise one is bound by
// arithmetic and latency, the pointwise one by memory, and neither does anything for the other.  Here a workgroup owns a tile of
// 8 columns x TH rows of output pixels and ALL channels (the paper's depth-first processing, Sec. III-A): phase 1 computes t for
// the tile straight from global memory -- every load of a thread's window is in flight at once -- and parks it in LDS as bf16,
// the rounding point of the stored tensor; phase 2 takes it into registers as MFMA fragments and contracts it with W, whose rows
// come through an LDS ring that fills by DMA while phase 1 runs, in passes of WC * TC * 32 output channels.  Every W row travels once per
// tile, so the pair pays where pixels are many next to the output channels: see dwpw_pays.
// What bounds it: phase 1's vector instructions (about 16 per element of t: nine products, the widening, addresses, the epilogue) and,
// from 256 channels on, the W rows, which a CU takes into LDS at 50 bytes per clock; the two follow each other inside a workgroup.
// Tiles of other heights, one or two 32-channel blocks per wave, one to four rows per thread and more workgroups per CU all
// measured within 5 % of one another; waves that keep tiles of their own with W resident in LDS, the next window fetched
// ahead, 42 us instead of 44 on the first pair below and no gain on the others.
// The products of a 1x1 output are added from channel 0 on, in one chain, where the kernels of the two launches start at a tile's own chunk,
// so a bf16 rounding turns now and then: of 6.15 million outputs over nine shapes 1261 are not the rounded exact value, 1248 as two launches; the
// logits of the separable list are 0.0029 to 0.0050 from 64 bits (2-norm, eight sizes) both ways, here the nearer in six and the same in two.
// Batch 64, us, two launches (without the gap between them) -> here: 32 -> 64 at 112x112 56 -> 44, 64 -> 128 stride 2 41 -> 31, 128 -> 128 at
// 56x56 48 -> 33, 128 -> 256 stride 2 29 -> 23, 256 -> 256 at 28x28 36 -> 27, 512 -> 512 at 14x14 25 -> 18.
#include <algorithm>

#include "conv_common.h"

namespace sol {

using lds_pipe::u32x4_t;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2_t;

struct DwPwArgs {
    DwPwLaunch d;
    int Ho, Wo, tw, th, ntiles, Kp;        // output extent, tiles across and down an image
    FastDiv dtw, dth;
};

// Phase 1 for one thread: RR x TQ output pixels of four channels.  All loads of the window are issued before the first is used; pixels
// outside the image are fetched out of range -> zeros.
template <int C, int S, int RR> struct DwWindow {
    static constexpr int TQ = S == 1 ? 4 : 2, NCOL = (TQ - 1) * S + 3, NROW = (RR - 1) * S + 3;
    u32x2_t raw[NROW][NCOL];
    float wv[9][4], sc[4], sf[4];

    // oh, ow: first output pixel of this thread
    __device__ __forceinline__ void fetch(const DwPwLaunch &d, const __amdgpu_buffer_rsrc_t &xr, int n, int oh, int ow, int c0) {
        const int ih0 = oh * S - 1, iw0 = ow * S - 1;
        unsigned coff[NCOL];
#pragma unroll
        for (int c = 0; c < NCOL; c++) coff[c] = (unsigned)(iw0 + c) < (unsigned)d.W ? (unsigned)((iw0 + c) * C + c0) * 2u : 0x80000000u;
#pragma unroll
        for (int r = 0; r < NROW; r++) {
            const unsigned rb = (unsigned)(ih0 + r) < (unsigned)d.H ? (unsigned)(n * d.H + ih0 + r) * (unsigned)(d.W * C * 2) : 0x80000000u;
#pragma unroll
            for (int c = 0; c < NCOL; c++) raw[r][c] = __builtin_amdgcn_raw_buffer_load_b64(xr, rb + coff[c] < rb ? 0xffffffffu : rb + coff[c], 0, 0);
        }
    }
    __device__ __forceinline__ void constants(const DwPwLaunch &d, int c0) {
        const bf16_t *__restrict__ wd = static_cast<const bf16_t *>(d.wd);
#pragma unroll
        for (int k = 0; k < 9; k++) {
            const uint2 u = *reinterpret_cast<const uint2 *>(wd + (long)k * C + c0);
            wv[k][0] = __uint_as_float(u.x << 16); wv[k][1] = __uint_as_float(u.x & 0xffff0000u);
            wv[k][2] = __uint_as_float(u.y << 16); wv[k][3] = __uint_as_float(u.y & 0xffff0000u);
        }
        const float4 s4 = *reinterpret_cast<const float4 *>(d.sd + c0), h4 = *reinterpret_cast<const float4 *>(d.hd + c0);
        sc[0] = s4.x; sc[1] = s4.y; sc[2] = s4.z; sc[3] = s4.w;
        sf[0] = h4.x; sf[1] = h4.y; sf[2] = h4.z; sf[3] = h4.w;
    }
    // t of the thread's pixels into the plane of its channels; row0, col0: the first one's place in the tile of 8 columns
    __device__ __forceinline__ void compute(unsigned char *plane, int row0, int col0, int c0, float lo) const {
        float acc[RR][TQ][4];
#pragma unroll
        for (int o = 0; o < RR; o++)
#pragma unroll
            for (int t = 0; t < TQ; t++)
#pragma unroll
                for (int e = 0; e < 4; e++) acc[o][t][e] = 0.f;
        static_for<NROW>([&](auto J) {                                 // an input row is widened once and feeds the up to three output rows that read it
            constexpr int j = decltype(J)::value;
            float v[NCOL][4];
#pragma unroll
            for (int c = 0; c < NCOL; c++) {
                v[c][0] = __uint_as_float(raw[j][c][0] << 16); v[c][1] = __uint_as_float(raw[j][c][0] & 0xffff0000u);
                v[c][2] = __uint_as_float(raw[j][c][1] << 16); v[c][3] = __uint_as_float(raw[j][c][1] & 0xffff0000u);
            }
            static_for<RR>([&](auto O) {
                constexpr int o = decltype(O)::value, r = j - o * S;
                if constexpr (r >= 0 && r < 3) {
#pragma unroll
                    for (int s2 = 0; s2 < 3; s2++)
#pragma unroll
                        for (int t = 0; t < TQ; t++)
#pragma unroll
                            for (int e = 0; e < 4; e++) acc[o][t][e] = fmaf(v[t * S + s2][e], wv[r * 3 + s2][e], acc[o][t][e]);
                    if constexpr (r == 2) {
#pragma unroll
                        for (int t = 0; t < TQ; t++) {
                            float f[4];
#pragma unroll
                            for (int e = 0; e < 4; e++) f[e] = __builtin_fmaxf(fmaf(acc[o][t][e], sc[e], sf[e]), lo);
                            const int px = (row0 + o) * 8 + col0 + t;
                            *reinterpret_cast<uint2 *>(plane + px * 128 + (((unsigned)((c0 & 63) >> 3) ^ (unsigned)lds_pipe::swz<128>(px)) << 4) + (c0 & 4) * 2) =
                                make_uint2(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]));
                        }
                    }
                }
            });
        });
    }
};

// C: channels of x and t; S: stride; TH: tile rows; WP x WC waves of 32 pixels x TC * 32 channels; NS: ring stages (a stage is 64
// reduction elements of a pass's W rows); RR: output rows per thread in phase 1
template <int C, int S, int TH, int WP, int WC, int TC, int NS, int RR>
__global__ void __launch_bounds__(WP *WC * 64, 2) conv_dwpw_kernel(const DwPwArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
    using namespace lds_pipe;
    constexpr int NW = WP * WC, NT = NW * 64, BP = TH * 8, PL = (C + 63) / 64, BC = WC * TC * 32;
    constexpr int STAGE = BC * 128, WL = BC / 8 / NW;                  // DMA instructions (8 rows of 128 bytes) per wave and stage
    constexpr int TB = PL * BP * 128, STRIPS = NW * 32 * (TC * 32 + 4) * 4, PARK = TB > STRIPS ? TB : STRIPS;
    constexpr int TQ = DwWindow<C, S, RR>::TQ, QUADS = C / 4, XS = 8 / TQ, ITEMS = QUADS * XS * (TH / RR);
    static_assert(BP == WP * 32 && BC % (8 * NW) == 0 && TH % RR == 0 && NS >= 2 && PARK + NS * STAGE <= 160 * 1024, "tile");
    __shared__ __align__(1024) unsigned char lds[PARK + NS * STAGE];
    unsigned char *const ring = lds + PARK;

    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wp = wave % WP, wc = wave / WP;
    const int tile = (int)(blockIdx.x & 7) * ((a.ntiles + 7) >> 3) + (int)(blockIdx.x >> 3);   // a contiguous run of tiles per XCD
    if (tile >= a.ntiles) return;
    uint32_t rest, tx, n, ty;
    a.dtw.divmod((uint32_t)tile, rest, tx);
    a.dth.divmod(rest, n, ty);
    const int oh0 = (int)ty * TH, ow0 = (int)tx * 8;
    const DwPwLaunch &d = a.d;

    // ---- W ring: stage s = plane s % PL of pass s / PL
    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(d.w), 0, (int)((unsigned)d.K * a.Kp * 2u), 0x00020000);
    unsigned wo[WL];
#pragma unroll
    for (int i = 0; i < WL; i++) {
        const int row = (wave * WL + i) * 8 + (lane >> 3);
        wo[i] = (unsigned)row * (unsigned)(a.Kp * 2) + (((unsigned)(lane & 7) ^ (unsigned)swz<128>(row)) << 4);
    }
    const int npass = (d.K + BC - 1) / BC, nst = npass * PL;
    int is = 0, ipl = 0;                                               // next stage to issue, its plane
    unsigned isoff = 0, ipass = 0;
    auto issue = [&](int slot) {                                       // rows beyond K and stages beyond the last: out of range -> zeros
        const unsigned soff = isoff;
#pragma unroll
        for (int i = 0; i < WL; i++) {
            const unsigned off = wo[i] + soff;                         // the whole offset in the lane's part: the range check is on it
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, (__attribute__((address_space(3))) void *)(ring + slot * STAGE + (wave * WL + i) * 1024), 16,
                                                     is < nst ? off : 0xffffffffu, 0, 0, 0);
        }
        is++;
        if (++ipl == PL) { ipl = 0; ipass += (unsigned)(BC * a.Kp * 2); isoff = ipass; } else isoff += 128;
    };
#pragma unroll
    for (int s = 0; s < NS - 1; s++) issue(s);

    // ---- phase 1
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(d.x), 0, (int)((unsigned)d.N * d.H * d.W * C * 2u), 0x00020000);
    const float lo = d.act_d == SOL_ACT_RELU ? 0.f : __builtin_nanf("");   // lower bound of t (none: NaN, which the maximum ignores)
    for (int it = tid; it < ITEMS; it += NT) {
        const int q = it % QUADS, r2 = it / QUADS, xs = r2 % XS, yr = r2 / XS, c0 = q * 4;
        DwWindow<C, S, RR> win;
        win.fetch(d, xr, (int)n, oh0 + yr * RR, ow0 + xs * TQ, c0);
        win.constants(d, c0);
        win.compute(lds + (c0 >> 6) * (BP * 128), yr * RR, xs * TQ, c0, lo);
    }
    if constexpr (C % 64 != 0) {                                       // channels 32 .. 63 of the one plane: W holds zeros there, 0 * 0
        for (int it = tid; it < BP * 4; it += NT) {
            const int px = it >> 2, sl = 4 + (it & 3);
            *reinterpret_cast<uint4 *>(lds + px * 128 + (((unsigned)sl ^ (unsigned)swz<128>(px)) << 4)) = make_uint4(0u, 0u, 0u, 0u);
        }
    }
    ConvArgs ea;                                                       // what the shared epilogue looks at
    ea.y = d.y; ea.res = nullptr; ea.act = d.act; ea.Cout = d.K; ea.scale = d.s; ea.shift = d.h;
    __syncthreads();

    // ---- t as fragments: lane = pixel, 8 reduction elements per k-step; the parking place is free afterwards
    u32x4_t ft[PL * 4];
    const unsigned fsw = swz<128>(lr);
    static_for<PL * 4>([&](auto I) {
        constexpr int i = decltype(I)::value;
        lds_read16<(i / 4) * (BP * 128)>(ft[i], lds_addr(lds) + (wp * 32 + lr) * 128 + (((2 * (i % 4) + lh) ^ fsw) << 4));
    });
    wait_lgkmcnt<0>();
    static_for<PL * 4>([&](auto I) { landed(ft[decltype(I)::value]); });

    const unsigned fw = lds_addr(ring) + (wc * TC * 32 + lr) * 128;
    const unsigned rowpitch = (unsigned)a.Wo * (unsigned)d.ldy;
    const TileRowOffset ro{(unsigned)(((int)n * a.Ho + oh0 + wp * 4) * a.Wo + ow0) * (unsigned)d.ldy, rowpitch, (unsigned)d.ldy, a.Ho - oh0 - wp * 4, a.Wo - ow0};
    ResidualRegs<bf16_t, 1, TC> nores;
    nores.on = false;
    int slot = 0;
    for (int p = 0; p < npass; p++) {
        f32x16_t acc[TC][1];
#pragma unroll
        for (int i = 0; i < TC; i++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[i][0][e] = 0.f;
        static_for<PL>([&](auto Q) {
            constexpr int q = decltype(Q)::value;
            wait_vmcnt<(NS - 2) * WL>();                               // this stage has landed
            __builtin_amdgcn_s_barrier();                              // ... for every wave, and nobody still reads the stage before (p = q = 0: everybody has t)
            const unsigned fb = fw + slot * STAGE;
            u32x4_t fa[2][TC];
            static_for<TC>([&](auto I) { lds_read16<decltype(I)::value * 32 * 128>(fa[0][decltype(I)::value], fb + ((lh ^ fsw) << 4)); });
            issue(slot == 0 ? NS - 1 : slot - 1);
            static_for<4>([&](auto KS) {
                constexpr int ks = decltype(KS)::value, cur = ks & 1;
                if constexpr (ks < 3) {
                    static_for<TC>([&](auto I) { lds_read16<decltype(I)::value * 32 * 128>(fa[cur ^ 1][decltype(I)::value], fb + (((2 * (ks + 1) + lh) ^ fsw) << 4)); });
                    wait_lgkmcnt<TC>();
                } else {
                    wait_lgkmcnt<0>();
                }
                static_for<TC>([&](auto I) { landed(fa[cur][decltype(I)::value]); });
                static_for<TC>([&](auto I) { Mma<bf16_t>::run(acc[decltype(I)::value][0], fa[cur][decltype(I)::value], ft[q * 4 + ks]); });
            });
            slot = slot + 1 == NS ? 0 : slot + 1;
        });
        const int cw = p * BC + wc * TC * 32;
        if (cw < d.K) {                                                // K % (TC * 32) == 0: the wave's channels exist or none does
            const Affine8 aff = load_affine_unconditional<TC>(ea, lane, cw);
            conv_epilogue_interior<bf16_t, 1, TC, false>(ea, acc, reinterpret_cast<float *>(lds), wave, lane, cw, aff, nores, ro);
        }
    }
    wait_vmcnt<0>();                                                   // the DMAs beyond the last stage
#endif
}

bool dwpw_kernel_applies(int dt, int N, int H, int W, int C, int S, int K, int ldy) {
    if (dt != SOL_BF16 || !(S == 1 || S == 2) || !(C == 32 || C == 64 || C == 128 || C == 256 || C == 512)) return false;
    const int Ho = out_size(H, 3, S, 1), Wo = out_size(W, 3, S, 1);
    return K % 64 == 0 && ldy % 8 == 0 && Ho > 0 && Wo > 0 && (double)N * H * W * C * 2 < 2147483648.0 && (double)N * Ho * Wo * ldy < 2147483648.0 &&
           (double)K * round_up((size_t)C, 64) * 2 < 2147483648.0;
}

// A workgroup passes all of W, so a launch takes at least that long however few its tiles are, while two launches spread the output
// channels of few pixels over the chip.  The line is therefore one of output channels against output pixels, K <= few + pixels / per, both
// fitted for each channel count and stride on 4000 pairs of random sizes (1 to 64 images of 4x4 to 160x160, K of 64 to 2048; launches replayed
// from a graph, the gap between two of them included) and looked at on 2500 others: of those 6500 one launch is the slower by more than 5 % in
// 21 that the rule takes (at most 23 %, just beyond a whole round of workgroups), and they take 0.920 of the time of two launches,
// 0.914 if every pair went its faster way.  us, two launches / one: stride 1, 2 images of 7x8, 32 -> 192 8.3 / 7.9; 1 of 7x7, 32 -> 256 8.5 / 8.9, 128 -> 128
// 9.2 / 8.5, 128 -> 256 9.4 / 11.3; 1 of 14x14, 32 -> 1024 8.1 / 24.7, 256 -> 128 9.0 / 8.0, 512 -> 64 8.9 / 9.5; 3 of 120x120, 64 -> 384 20.4 / 18.1; 3 of 125x125,
// 128 -> 512 33.7 / 26.4; 7 of 40x28, 256 -> 512 13.8 / 15.2; 2 of 45x31, 512 -> 128 13.0 / 9.8; stride 2, 2 of 11x11, 128 -> 384 8.6 / 10.1; 24 of 12x12,
// 256 -> 64 8.8 / 9.7; 8 of 20x20, 512 -> 64 9.3 / 13.9.  At 512 channels and stride 2 a tile takes 14 us for any K: two launches (the auto-tuner tries one).
bool dwpw_pays(int N, int H, int W, int C, int S, int K) {
    const int Ho = out_size(H, 3, S, 1), Wo = out_size(W, 3, S, 1);
    const long wk = (long)C * K;
    if (wk > 262144 || (wk > 65536 && (long)N * ceil_div(Ho, 8) * ceil_div(Wo, 8) < 128)) return false;
    const int i = C <= 32 ? 0 : C <= 64 ? 1 : C <= 128 ? 2 : C <= 256 ? 3 : 4;
    constexpr int few[2][5] = {{192, 192, 128, 128, 0}, {128, 128, 192, 0, 0}}, per[2][5] = {{160, 100, 100, 25, 12}, {150, 100, 25, 34, 0}};
    return per[S - 1][i] > 0 && K <= few[S - 1][i] + (long)N * Ho * Wo / per[S - 1][i];
}

template <int C, int S, int TH, int WP, int WC, int TC, int NS, int RR> static void launch_dwpw_cfg(const DwPwLaunch &d, hipStream_t st) {
    DwPwArgs a;
    a.d = d;
    a.Ho = out_size(d.H, 3, S, 1); a.Wo = out_size(d.W, 3, S, 1);
    a.tw = ceil_div(a.Wo, 8); a.th = ceil_div(a.Ho, TH);
    a.ntiles = d.N * a.tw * a.th;
    a.Kp = (int)round_up((size_t)C, 64);
    a.dtw = FastDiv((uint32_t)a.tw); a.dth = FastDiv((uint32_t)a.th);
    hipLaunchKernelGGL((conv_dwpw_kernel<C, S, TH, WP, WC, TC, NS, RR>), dim3(((a.ntiles + 7) / 8) * 8), dim3(WP * WC * 64), 0, st, a);
}

sol_status launch_conv_dwpw(const DwPwLaunch &d, hipStream_t st) {
    if ((long)d.N * d.H * d.W == 0) return SOL_OK;
    if (d.S == 1) {
        switch (d.C) {
            case 32: launch_dwpw_cfg<32, 1, 16, 4, 1, 2, 2, 2>(d, st); break;
            case 64: launch_dwpw_cfg<64, 1, 16, 4, 1, 2, 2, 2>(d, st); break;
            case 128: launch_dwpw_cfg<128, 1, 16, 4, 1, 1, 3, 4>(d, st); break;
            case 256: launch_dwpw_cfg<256, 1, 8, 2, 2, 2, 2, 4>(d, st); break;
            default: launch_dwpw_cfg<512, 1, 8, 2, 4, 1, 4, 4>(d, st); break;
        }
    } else {
        switch (d.C) {
            case 32: launch_dwpw_cfg<32, 2, 16, 4, 1, 2, 2, 2>(d, st); break;
            case 64: launch_dwpw_cfg<64, 2, 16, 4, 1, 2, 2, 4>(d, st); break;
            case 128: launch_dwpw_cfg<128, 2, 8, 2, 2, 1, 3, 2>(d, st); break;
            case 256: launch_dwpw_cfg<256, 2, 8, 2, 2, 2, 2, 4>(d, st); break;
            default: launch_dwpw_cfg<512, 2, 8, 2, 4, 1, 4, 4>(d, st); break;
        }
    }
    SOL_HIP(hipGetLastError());
    return SOL_OK;
}

}  // namespace sol

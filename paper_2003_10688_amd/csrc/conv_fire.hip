// Fire module -- 1x1 squeeze, then a 1x1 and a 3x3 expand side by side, joined along the channels -- as ONE depth-first kernel
// (gfx950, bf16):
//
//     s = act(ss * (x . Ws) + hs)                      C -> SP channels (32, the plan's padding included)
//     y[:, o1 ..] = act(s1 * (s . W1) + h1)            1x1, E1 channels
//     y[:, o3 ..] = act(s3 * (s * W3) + h3)            3x3, pad 1, E3 channels
//
// Run as three launches, s is written once and read twice, nine times over by the 3x3 kernel's taps, and on the small images each
// launch is mostly ramp-up.  Here a workgroup owns 8 x 8 output pixels and all channels (the paper's depth-first processing,
// Sec. III-A): phase A computes s for the tile and its halo of one pixel, 10 x 10, with both operands' fragments straight from global
// memory, and parks it in LDS as bf16 -- the rounding point of the stored tensor -- with zeros where the 3x3 convolution pads;
// phase B contracts it with the two expand weights, whose rows come through an LDS ring that fills by DMA while phase A runs, in passes
// of 64 output channels, the nine taps read from the patch.  The price is the halo, 1.56 times the squeeze's work.
// What bounds it is the length of a tile's one path -- operands of s from memory, patch, nine taps, stores, 10 us with three workgroups
// per CU -- so it pays while tiles are few (fire_pays).  us, three launches (without the gaps between them, about 3.5) -> here: 64 -> 16 ->
// 64 + 64 at 55x55, 1 image 13.4 -> 7.1, 8 images 16.0 -> 9.8, 64 images 38.8 -> 38.4; 128 -> 32 -> 128 + 128 at 27x27, 1 image 11.9 -> 10.1, 16
// images 17.3 -> 13.2.  Squeezes of 64 stored channels were slower at every size (384 -> 64 -> 256 + 256 at 13x13, 1 image 11 and 24,
// 64 images 25 and 30: the weights pass every tile) and are not built.
#include <algorithm>

#include "conv_common.h"

namespace sol {

using lds_pipe::u32x4_t;

struct FireArgs {
    FireLaunch f;
    int tw, th, ntiles, Kp3;               // tiles across and down an image; packed reduction length of the 3x3 weights
    FastDiv dtw, dth;
};

// ME: room for the affine constants of that many output channels of the two expands together
template <int NS, int ME>
__global__ void __launch_bounds__(256, 2) conv_fire_kernel(const FireArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
    using namespace lds_pipe;
    constexpr int SP = 32, ROWB = SP * 2, KS = SP / 16;                // stored squeeze channels; bytes of a patch row; k-steps of a tap
    constexpr int NPOS = 100, PATCH = (NPOS * ROWB + 1023) / 1024 * 1024, STAGE = 64 * 128, WL = 2;
    constexpr int ST3 = (9 * SP + 63) / 64;                            // stages of a pass of the 3x3 expand: 64 reduction elements of 64 W3 rows
    constexpr int STRIPS = 4 * 32 * (32 + 4) * 4;
    __shared__ __align__(1024) unsigned char lds[PATCH + NS * STAGE + STRIPS + ME * 8];
    unsigned char *const ring = lds + PATCH;
    float *const strips = reinterpret_cast<float *>(ring + NS * STAGE), *const cst = strips + STRIPS / 4;   // cst: scale, shift of the expands' channels

    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 31, lh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wp = wave & 1, wc = wave >> 1;
    const int tile = (int)(blockIdx.x & 7) * ((a.ntiles + 7) >> 3) + (int)(blockIdx.x >> 3);   // a contiguous run of tiles per XCD
    if (tile >= a.ntiles) return;
    uint32_t rest, tx, n, ty;
    a.dtw.divmod((uint32_t)tile, rest, tx);
    a.dth.divmod(rest, n, ty);
    const int oh0 = (int)ty * 8, ow0 = (int)tx * 8;
    const FireLaunch &f = a.f;

    // ---- expand weights: the passes of the 1x1 (one stage each), then those of the 3x3 (ST3 stages each)
    const int n1 = f.E1 >> 6, n3 = f.E3 >> 6, nst = n1 + n3 * ST3;
    unsigned wrow[WL], wslot[WL];
#pragma unroll
    for (int i = 0; i < WL; i++) {
        const int row = (wave * WL + i) * 8 + (lane >> 3);
        wrow[i] = (unsigned)row;
        wslot[i] = ((unsigned)(lane & 7) ^ (unsigned)swz<128>(row)) << 4;
    }
    int is = 0, ist = 0;                                               // next stage to issue; of the 3x3: its place in the pass
    unsigned base3 = 0;
    auto issue = [&](int slot) {
        const bool one = is < n1, real = is < nst;
        const unsigned pitch = one ? 128u : (unsigned)(a.Kp3 * 2), base = one ? (unsigned)(is * 64 * 128) : base3 + (unsigned)(ist * 128);
        const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(one ? f.w1 : f.w3), 0, one ? f.E1 * 128 : f.E3 * a.Kp3 * 2, 0x00020000);
#pragma unroll
        for (int i = 0; i < WL; i++)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, (__attribute__((address_space(3))) void *)(ring + slot * STAGE + (wave * WL + i) * 1024), 16,
                                                     real ? base + wrow[i] * pitch + wslot[i] : 0xffffffffu, 0, 0, 0);
        if (!one && ++ist == ST3) { ist = 0; base3 += (unsigned)(64 * a.Kp3 * 2); }
        is++;
    };
#pragma unroll
    for (int s = 0; s < NS - 1; s++) issue(s);

    // ---- phase A: a wave computes s at 32 of the 100 positions (the last wave at four)
    {
        const int pos = wave * 32 + lr, py = pos / 10, px = pos - py * 10;
        const int ih = oh0 - 1 + py, iw = ow0 - 1 + px;
        const bool in = pos < NPOS && (unsigned)ih < (unsigned)f.H && (unsigned)iw < (unsigned)f.W;
        const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(f.x), 0, (int)((unsigned)f.N * f.H * f.W * f.C * 2u), 0x00020000);
        const __amdgpu_buffer_rsrc_t sr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(f.ws), 0, SP * f.C * 2, 0x00020000);
        const unsigned xo = in ? (unsigned)(((int)n * f.H + ih) * f.W + iw) * (unsigned)(f.C * 2) + (unsigned)(lh * 16) : 0x80000000u;
        const unsigned so = (unsigned)lr * (unsigned)(f.C * 2) + (unsigned)(lh * 16);
        f32x16_t acc;
#pragma unroll
        for (int e = 0; e < 16; e++) acc[e] = 0.f;
        typedef __attribute__((ext_vector_type(4))) unsigned q_t;
        q_t bq[2][4], aq[2][4];
        auto fetch = [&](q_t (&b)[4], q_t (&w)[4], int kc) {           // 64 reduction elements of the wave's rows and of Ws
#pragma unroll
            for (int k = 0; k < 4; k++) {
                b[k] = __builtin_amdgcn_raw_buffer_load_b128(xr, xo, kc * 128 + k * 32, 0);
                w[k] = __builtin_amdgcn_raw_buffer_load_b128(sr, so, kc * 128 + k * 32, 0);
            }
        };
        const int nc = f.C >> 6;
        fetch(bq[0], aq[0], 0);
        // Everything else that comes from memory is asked for beside the first operands: the affine constants of s in registers, those of the
        // expands on their way to LDS (a load in front of its use is a trip to L2 on the tile's one path).  The compiler puts these in front
        // and waits for everything at every other chunk below; pinned behind the first operands, with a chunk in flight throughout, 500
        // random modules took 0.998 of the time: three workgroups on a CU cover for one another.
        float4 sc[4], sf[4];
#pragma unroll
        for (int g = 0; g < 4; g++) {
            sc[g] = *reinterpret_cast<const float4 *>(f.ss + 8 * g + 4 * lh);
            sf[g] = *reinterpret_cast<const float4 *>(f.hs + 8 * g + 4 * lh);
        }
        constexpr int CN = ME / 256;
        float c1[CN], c2[CN];
#pragma unroll
        for (int k = 0; k < CN; k++) {
            const int c = min(tid + k * 256, f.E1 + f.E3 - 1);
            c1[k] = *(c < f.E1 ? f.s1 + c : f.s3 + (c - f.E1));
            c2[k] = *(c < f.E1 ? f.h1 + c : f.h3 + (c - f.E1));
        }
        for (int kc = 0; kc < nc; kc += 2) {
            static_for<2>([&](auto U) {
                constexpr int u = decltype(U)::value;
                if (u == 0 || kc + 1 < nc) {
                    fetch(bq[u ^ 1], aq[u ^ 1], min(kc + u + 1, nc - 1));
#pragma unroll
                    for (int k = 0; k < 4; k++) Mma<bf16_t>::run(acc, aq[u][k], bq[u][k]);
                }
            });
        }
#pragma unroll
        for (int k = 0; k < CN; k++) { cst[tid + k * 256] = c1[k]; cst[ME + tid + k * 256] = c2[k]; }
        // accumulator register e of lane l: channel 8 * (e / 4) + 4 * (l / 32) + e % 4, position l % 32
        const float lo = f.act_s == SOL_ACT_RELU ? 0.f : __builtin_nanf("");
        if (pos < NPOS) {
#pragma unroll
            for (int g = 0; g < 4; g++) {
                const int c = 8 * g + 4 * lh;
                const float4 a4 = sc[g], b4 = sf[g];
                const float v0 = __builtin_fmaxf(acc[4 * g] * a4.x + b4.x, lo), v1 = __builtin_fmaxf(acc[4 * g + 1] * a4.y + b4.y, lo);
                const float v2 = __builtin_fmaxf(acc[4 * g + 2] * a4.z + b4.z, lo), v3 = __builtin_fmaxf(acc[4 * g + 3] * a4.w + b4.w, lo);
                const uint2 u = in ? make_uint2(pack_bf16x2(v0, v1), pack_bf16x2(v2, v3)) : make_uint2(0u, 0u);
                *reinterpret_cast<uint2 *>(lds + pos * ROWB + (((unsigned)(c >> 3) ^ (unsigned)swz<ROWB>(pos)) << 4) + (c & 4) * 2) = u;
            }
        }
    }
    __syncthreads();

    // ---- phase B
    const int m = wp * 32 + lr, pos0 = (m >> 3) * 10 + (m & 7);        // position of this lane's pixel under tap (0, 0)
    const unsigned fsw = swz<128>(lr), fw = lds_addr(ring) + (wc * 32 + lr) * 128;
    const TileRowOffset ro{(unsigned)(((int)n * f.H + oh0 + wp * 4) * f.W + ow0) * (unsigned)f.ldy, (unsigned)f.W * (unsigned)f.ldy, (unsigned)f.ldy,
                           f.H - oh0 - wp * 4, f.W - ow0};
    ResidualRegs<bf16_t, 1, 1> nores;
    nores.on = false;
    int slot = 0;
    f32x16_t acc[1][1];
    // one stage: CNT k-steps, the I-th of them tap (T0 + I / KS), its k-step I % KS
    auto stage = [&](auto T0, auto CNT) {
        constexpr int t0 = decltype(T0)::value, cnt = decltype(CNT)::value;
        wait_vmcnt<(NS - 2) * WL>();                                   // this stage has landed
        __builtin_amdgcn_s_barrier();                                  // ... for every wave, and nobody still reads the stage before
        const unsigned fb = fw + slot * STAGE;
        u32x4_t fa[cnt], fx[cnt];
        static_for<cnt>([&](auto I) {
            constexpr int i = decltype(I)::value, tap = t0 + i / KS, off = (tap / 3) * 10 + tap % 3;
            const int pos = pos0 + off;
            lds_read16<0>(fa[i], fb + (((2 * i + lh) ^ fsw) << 4));
            lds_read16<0>(fx[i], lds_addr(lds) + pos * ROWB + (((unsigned)(2 * (i % KS) + lh) ^ (unsigned)swz<ROWB>(pos)) << 4));
        });
        issue(slot == 0 ? NS - 1 : slot - 1);
        static_for<cnt>([&](auto I) {
            constexpr int i = decltype(I)::value;
            wait_lgkmcnt<2 * (cnt - 1 - i)>();
            landed(fa[i]);
            landed(fx[i]);
            Mma<bf16_t>::run(acc[0][0], fa[i], fx[i]);
        });
        slot = slot + 1 == NS ? 0 : slot + 1;
    };
    auto clear = [&]() {
#pragma unroll
        for (int e = 0; e < 16; e++) acc[0][0][e] = 0.f;
    };
    auto finish = [&](void *y, int act, int E, int first, int p) {
        const int cw = p * 64 + wc * 32;
        ConvArgs ea;                                                   // what the shared epilogue looks at
        ea.y = y; ea.res = nullptr; ea.act = act; ea.Cout = E;
        Affine8 aff;
        const float *c = cst + first + cw + (lane & 3) * 8;
#pragma unroll
        for (int e = 0; e < 8; e++) { aff.sc[e] = c[e]; aff.sf[e] = c[ME + e]; }
        conv_epilogue_interior<bf16_t, 1, 1, false>(ea, acc, strips, wave, lane, cw, aff, nores, ro);
    };
    for (int p = 0; p < n1; p++) {
        clear();
        stage(std::integral_constant<int, 4>{}, std::integral_constant<int, KS>{});    // the centre tap
        finish(f.y1, f.act1, f.E1, 0, p);
    }
    for (int p = 0; p < n3; p++) {
        clear();
        static_for<ST3>([&](auto S) {
            constexpr int s = decltype(S)::value, t0 = s * 4 / KS, left = 9 * KS - s * 4;
            stage(std::integral_constant<int, t0>{}, std::integral_constant<int, left < 4 ? left : 4>{});
        });
        finish(f.y3, f.act3, f.E3, f.E1, p);
    }
    wait_vmcnt<0>();                                                   // the DMAs beyond the last stage
#endif
}

bool fire_kernel_applies(int dt, int N, int H, int W, int C, int SP, int E1, int E3, int ldy) {
    return dt == SOL_BF16 && SP == 32 && C % 64 == 0 && C <= 4096 && E1 % 64 == 0 && E3 % 64 == 0 && E1 > 0 && E3 > 0 && E1 + E3 <= 512 && ldy % 8 == 0 &&
           (double)N * H * W * C * 2 < 2147483648.0 && (double)N * H * W * ldy < 2147483648.0;
}

// A tile is one path through C / 64 chunks of the squeeze, E1 / 64 stages of the 1x1 expand and five for 64 channels of the 3x3, while the
// separate launches spread few pixels' channels over the chip; and beyond a tile per CU the halo's 1.56 times the squeeze counts, the
// more the wider the input.  Fitted on 1700 modules of random sizes (squeezes of 16 and 32, 1 to 128 images of 4x4 to 130x130, replayed from a
// graph, gaps included) and looked at on 900 others: of those 2600 one launch is the slower by more than 5 % in 13 that the rule takes (at
// most 14 %), and they take 0.931 of the time of three launches, 0.921 if every module went its faster way.  us, three launches / one: 64 ->
// 64 + 64, 740 tiles 15.8 / 11.2, 1176 tiles 18.2 / 16.5, 2880 tiles 35.7 / 33.1, 3075 tiles 36.4 / 35.4, 4180 tiles 44.1 / 45.4, 6512 tiles 64.2 / 66.5; 512 -> 256 + 256,
// 32 tiles 12.3 / 19.0; 512 -> 128 + 256, 18 tiles 12.0 / 17.9; 64 -> 128 + 128, 1404 tiles 23.5 / 26.7.
bool fire_pays(int N, int H, int W, int C, int E1, int E3) {
    const long tiles = (long)N * ceil_div(H, 8) * ceil_div(W, 8), over = std::max(0l, tiles - 256);
    return C + E1 + 2 * E3 + (C <= 64 ? over / 8 : C * over / 128) <= 640;
}

sol_status launch_conv_fire(const FireLaunch &f, hipStream_t st) {
    if ((long)f.N * f.H * f.W == 0) return SOL_OK;
    FireArgs a;
    a.f = f;
    a.tw = ceil_div(f.W, 8); a.th = ceil_div(f.H, 8);
    a.ntiles = f.N * a.tw * a.th;
    a.Kp3 = (int)round_up((size_t)9 * f.SP, 64);
    a.dtw = FastDiv((uint32_t)a.tw); a.dth = FastDiv((uint32_t)a.th);
    const dim3 grid(((a.ntiles + 7) / 8) * 8);
    if (f.E1 + f.E3 <= 256) hipLaunchKernelGGL((conv_fire_kernel<3, 256>), grid, dim3(256), 0, st, a);   // 53 KB: three workgroups per CU
    else hipLaunchKernelGGL((conv_fire_kernel<3, 512>), grid, dim3(256), 0, st, a);
    SOL_HIP(hipGetLastError());
    return SOL_OK;
}

}  // namespace sol

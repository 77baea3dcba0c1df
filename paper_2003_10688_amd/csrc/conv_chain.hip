// fp32 convolution for the forward pass of a training step on small layers: small tiles, each output still ONE chain of fused
// multiply-adds over the whole reduction, in the order of the 64x64 ring tile (gfx950).
//
// A training step in fp32 keeps the kernels whose sums run in one order (see launch_conv): a last bit that moves takes ReLU and
// pooling decisions with it.  On a layer with few pixels the ring kernel's 64x64 tiles then leave most of the chip idle, and what
// a tile costs is the length of the chain: v_mfma_f32_32x32x2_f32 takes 64 cycles for two reduction elements, 147 thousand
// cycles for 4608.  v_mfma_f32_16x16x4_f32 takes 32 cycles for four, a quarter of that per element, over a quarter of the
// outputs -- and both instructions accumulate one reduction element after the other, rounding each time (checked against fmaf
// on the host, 200 random blocks of 64 elements, every bit).  So this kernel gives a wave one 16x16 block and no split of the
// reduction, and feeds the instructions in the ring kernel's order: inside 8 elements 0 4 1 5 2 6 3 7 (the two half-waves'
// 16 bytes in turn), the walk over the reduction starting at the chunk that the pixel's 64-row tile starts at there.  Same bits.
//
// What bounds it is what one wave can issue: eight matrix instructions of 32 cycles, eight fragment reads, sixteen picks, four
// DMA instructions and the walk take 535 cycles per stage instead of 260; leaving out the DMA, or the reads, or fetching the same
// line for every row changes nothing.  Measured before, on 512 -> 512, 3x3, 9 images of 4x4: 32x32 tiles of four waves, shared ring,
// 57 us (barrier, then reads and DMA at once); two dwords per lane by ds_read2_b32 (10 cycles each, two rows on a bank) 57;
// one wave, reads and DMA between the matrix instructions 57; with the walk and the ring addresses as constants 41 and, here,
// 38.  Two blocks per wave, two chains: 55; four: 88.
// 3x3, 9 images, us, 64x64 ring tile -> here: 512 -> 512 at 4x4 100 -> 38, 256 -> 256 at 8x8 53 -> 23, 128 -> 128 at 15x15 28 -> 15, 64 -> 64
// at 29x29 18.1 -> 13.9.
#include "conv_common.h"

namespace sol {

using lds_pipe::u32x4_t;

// One wave per workgroup with a ring of NS stages of 128 bytes of every tile row of its own (no barrier).  With one wave on a SIMD
// nothing hides what stands between two matrix instructions of a chain but the 32 cycles that the first of them takes: fragment
// reads, picks and DMA are dealt one by one into those gaps.
template <int NS>
__global__ void __launch_bounds__(64) conv_chain_kernel(const ConvArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
    using namespace lds_pipe;
    constexpr int BP = 16, BC = 16, ROWB = 128, BK = 32;   // pixels, channels; bytes and elements of a stage's row
    constexpr int XL = BP / 8, WL = BC / 8, L = XL + WL;   // DMA instructions (8 rows each) per stage
    constexpr int STAGE = (BP + BC) * ROWB;
    static_assert(NS >= 4 && NS % 2 == 0 && NS * STAGE <= 160 * 1024 && NS * L < 64, "LDS, vmcnt");
    __shared__ __align__(1024) unsigned char lds[NS * STAGE];

    const int lane = threadIdx.x, lr = lane & 15, lg = lane >> 4;
    const int lslot = lane & 7, lrow = lane >> 3;

    // XCD-aware tile order (see conv_dma.hip)
    const int xcd = (int)(blockIdx.x & 7);
    int tile;
    if (a.cpx > 0) {
        const int j = (int)(blockIdx.x >> 3);
        tile = (j / a.cpx) * a.ntc + xcd * a.cpx + j % a.cpx;
    } else {
        tile = xcd * ((a.ntiles + 7) >> 3) + (int)(blockIdx.x >> 3);
    }
    if (tile >= a.ntiles) return;
    const int p0 = (tile / a.ntc) * BP, c0 = (tile % a.ntc) * BC;

    // resources and zero fill of padding taps and missing rows as in conv_direct.hip
    const unsigned bias = (unsigned)((a.ph * a.W + a.pw) * a.C) * 4u;
    const unsigned xbytes = (unsigned)a.N * a.H * a.W * a.C * 4u, wbytes = (unsigned)a.Cout * a.Kp * 4u;
    __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<unsigned char *>(static_cast<const unsigned char *>(a.x)) - bias, 0, (int)(xbytes + bias), 0x00020000);
    __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.w), 0, (int)wbytes, 0x00020000);

    unsigned xo[XL], xinv[XL], wo[WL];                     // this lane's rows; bit t of xinv: filter tap t reads padding
#pragma unroll
    for (int i = 0; i < XL; i++) {
        const int row = i * 8 + lrow, m = p0 + row;
        int n, op, oq;
        decode_pixel(a, m, n, op, oq);
        const int ih0 = op * a.sh - a.ph, iw0 = oq * a.sw - a.pw;
        const unsigned off = (unsigned)(((n * a.H + ih0) * a.W + iw0) * a.C) * 4u + bias + ((lslot ^ swz<ROWB>(row)) << 4);
        const int slo = max(0, -iw0), shi = min(a.S, a.W - iw0), rlo = max(0, -ih0), rhi = min(a.R, a.H - ih0);
        const unsigned cval = shi > slo ? (unsigned)((1ull << shi) - 1ull) & ~((1u << slo) - 1u) : 0u;
        unsigned val = 0;
        for (int r = 0; r < a.R; r++) val |= (r >= rlo && r < rhi) ? cval << (r * a.S) : 0u;
        xo[i] = m < a.P ? off : 0xffffffffu;
        xinv[i] = ~val;
    }
#pragma unroll
    for (int i = 0; i < WL; i++) {
        const int row = i * 8 + lrow, co = c0 + row;
        wo[i] = co < a.Cout ? (unsigned)(co * a.Kp) * 4u + ((lslot ^ swz<ROWB>(row)) << 4) : 0xffffffffu;
    }

    const int cpt = a.C / BK, nk = a.R * a.S * cpt;        // chunks per filter tap, in all
    const int rot = (p0 >> 6) % cpt;                       // where the ring kernel's 64-pixel tile starts its walk
    // The walk in runs of chunks of one tap: tap 0 from chunk rot on, the other taps, tap 0 up to chunk rot, then nothing (resources
    // of size 0 -> zeros).  Inside a run a stage costs two additions and a count: what one wave issues between two matrix
    // instructions of its chain is what this kernel's time is made of (5 cycles per instruction).
    const int taps = a.R * a.S;
    int run = 0, left = cpt - rot, tr = 0, ts = 0;
    unsigned xs = (unsigned)rot * ROWB, ws = xs, xov[XL];
#pragma unroll
    for (int i = 0; i < XL; i++) xov[i] = xo[i] | (unsigned)__builtin_amdgcn_sbfe(xinv[i], 0, 1);
    auto next_stage = [&]() {
        xs += ROWB; ws += ROWB;
        if (__builtin_expect(--left == 0, 0)) {
            if (++run < taps) {
                if (++ts == a.S) { ts = 0; ++tr; }
                left = cpt;
            } else if (run == taps && rot > 0) {
                ts = tr = 0;
                left = rot;
            } else {
                left = 1 << 30;
                xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.x), 0, 0, 0x00020000);
                wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.w), 0, 0, 0x00020000);
            }
            const int tap = tr * a.S + ts;
            xs = (unsigned)((tr * a.W + ts) * a.C) * 4u;
            ws = (unsigned)(tap * a.C) * 4u;
#pragma unroll
            for (int i = 0; i < XL; i++) xov[i] = xo[i] | (unsigned)__builtin_amdgcn_sbfe(xinv[i], tap, 1);
        }
    };
    // the D-th DMA instruction of the next stage, into ring slot BUF
    auto issue_one = [&](auto D, auto BUF) {
        constexpr int d = decltype(D)::value;
        unsigned char *lx = lds + decltype(BUF)::value * STAGE, *lw = lx + BP * ROWB;
        if constexpr (d < WL)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, (__attribute__((address_space(3))) void *)(lw + d * 1024), 16, wo[d], ws, 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (__attribute__((address_space(3))) void *)(lx + (d - WL) * 1024), 16, xov[d - WL], xs, 0, 0);
    };

    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};

    // fragments of a stage: per 8 reduction elements a lane needs elements 4 (lg & 1) + lg / 2 and that + 2 (the two
    // matrix instructions of those 8 then run through 0 4 1 5 and 2 6 3 7).  It reads the 16 bytes that hold them and picks:
    // two dwords by ds_read2_b32 took LDS 10 cycles per instruction (two rows on one bank), twice the time of the products
    const unsigned fsw = swz<ROWB>(lr);
    const unsigned sel = lg >= 2 ? 0x07060504u : 0x03020100u;  // one v_perm per pick: from a select the compiler made an indexed extract, three selects each
    auto pick = [&](unsigned even_el, unsigned odd_el) { return __uint_as_float(__builtin_amdgcn_perm(odd_el, even_el, sel)); };
    unsigned fa[4];
#pragma unroll
    for (int q = 0; q < 4; q++) fa[q] = lds_addr(lds) + lr * ROWB + (((2 * q + (lg & 1)) ^ fsw) << 4);
    typedef u32x4_t Frags[4];
    Frags fw[2], fx[2];
    // read R of the stage in ring slot BUF: 16 bytes of the weights (even R) or of the pixels (odd)
    auto read_one = [&](auto R, auto BUF, Frags &w, Frags &x) {
        constexpr int q = decltype(R)::value / 2, o = decltype(BUF)::value * STAGE;
        if constexpr (decltype(R)::value % 2 == 0) lds_read16<o + BP * ROWB>(w[q], fa[q]); else lds_read16<o>(x[q], fa[q]);
    };
    auto frags_landed = [](Frags &w, Frags &x) {
        wait_lgkmcnt<0>();
#pragma unroll
        for (int q = 0; q < 4; q++) {
            landed(w[q]);
            landed(x[q]);
        }
    };

    static_for<NS - 1>([&](auto S) {
        static_for<L>([&](auto D) { issue_one(D, S); });
        next_stage();
    });
    constexpr int NR = 8, SLOTS = 8;                       // fragment reads and matrix instructions of a stage
    wait_vmcnt<(NS - 2) * L>();
    static_for<NR>([&](auto R) { read_one(R, std::integral_constant<int, 0>{}, fw[0], fx[0]); });
    frags_landed(fw[0], fx[0]);
    for (int k = 0; k < nk; k += NS) {                     // a turn of the ring: slots and register sets are constants
        static_for<NS>([&](auto U) {
            constexpr int u = decltype(U)::value, cur = u & 1;
            if (u == 0 || __builtin_expect(k + u < nk, 1)) {
                // stage k + u + 1 has landed; stage k + u is in registers, so the slot of the stage before takes the next one
                wait_vmcnt<(NS - 3) * L>();
                float ew[2], ex[2];
                auto picks = [&](auto T) {
                    constexpr int t = decltype(T)::value, q = t / 2, h = t % 2;
                    ew[t & 1] = pick(fw[cur][q][2 * h], fw[cur][q][2 * h + 1]);
                    ex[t & 1] = pick(fx[cur][q][2 * h], fx[cur][q][2 * h + 1]);
                };
                picks(std::integral_constant<int, 0>{});
                static_for<SLOTS>([&](auto Z) {
                    constexpr int z = decltype(Z)::value;
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ew[z & 1], ex[z & 1], acc, 0, 0, 0);
                    if constexpr (z < 7) picks(std::integral_constant<int, z + 1>{});
                    // reads in the first half of the stage, to have landed by its end; DMA in the second
                    constexpr int H = SLOTS / 2, N = z < H ? NR : L, y = z % H, lo = y * N / H, hi = (y + 1) * N / H;
                    static_for<hi - lo>([&](auto A) {
                        constexpr int act = lo + decltype(A)::value;
                        if constexpr (z < H) read_one(std::integral_constant<int, act>{}, std::integral_constant<int, (u + 1) % NS>{}, fw[cur ^ 1], fx[cur ^ 1]);
                        else issue_one(std::integral_constant<int, act>{}, std::integral_constant<int, (u + NS - 1) % NS>{});
                    });
                    __builtin_amdgcn_sched_barrier(0);
                });
                next_stage();
                frags_landed(fw[cur ^ 1], fx[cur ^ 1]);
            }
        });
    }
    wait_vmcnt<0>();                                       // the zero-fill DMAs of the tail

    // accumulator register e of lane l: channel 4 * (l / 16) + e, pixel l % 16 of its block
    const float *__restrict__ resg = static_cast<const float *>(a.res);
    float *__restrict__ yg = static_cast<float *>(a.y);
    const bool vec = (a.Cout & 3) == 0;
    const int cb = c0 + lg * 4, nv = min(4, a.Cout - cb), m = p0 + lr;
    float sc[4], sf[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
        sc[e] = (a.scale && e < nv) ? a.scale[cb + e] : 1.f;
        sf[e] = (a.shift && e < nv) ? a.shift[cb + e] : 0.f;
    }
    if (m >= a.P || nv <= 0) return;
    const size_t o = (size_t)m * a.Cout + cb;
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
        v[e] = acc[e] * sc[e] + sf[e];
        if (resg && e < nv) v[e] += resg[o + e];
        if (a.act == SOL_ACT_RELU) v[e] = __builtin_fmaxf(v[e], 0.f);
    }
    if (vec) {
        *reinterpret_cast<float4 *>(yg + o) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
        for (int e = 0; e < 4; e++)
            if (e < nv) yg[o + e] = v[e];
    }
#endif
}

// Layers that the ring kernel would run on its 64x64 tile with 128-byte stages (the caller's condition), dense output, no pool, up
// to 2048 blocks: two waves on a SIMD.  Both sides of that line (3x3, us, ring / here): 64 -> 64, 1896 blocks 18.1 / 13.9, 2524 19.0 / 21.3;
// 128 -> 128, 1800 30.4 / 20.9, 2400 30.8 / 30.0, 4800 49.9 / 51.9; 512 -> 512, 1216 103 / 59, 2368 108 / 96.
static long chain_blocks(const ConvArgs &a) { return (long)ceil_div(a.P, 16) * ceil_div(a.Cout, 16); }
bool chain_kernel_applies(const ConvArgs &a) {
    const double xb = (double)a.N * a.H * a.W * a.C * 4 + (double)(a.ph * a.W + a.pw) * a.C * 4;
    return chain_blocks(a) <= 2048 && a.C % 32 == 0 && a.R * a.S <= 32 && a.pool == 0 && a.ldy == a.Cout && xb < 2147483648.0 && (double)a.Cout * a.Kp * 4 < 2147483648.0;
}

// Eight stages (32 KB) while a CU holds at most four waves: weights that come from HBM need them (512 -> 512 at 4x4 behind 256 MB of
// other data: 38 us, 46 with four stages); four stages beyond (64 -> 64, 1896 blocks: 13.9, 21.8 with eight).
sol_status launch_conv_chain(const ConvArgs &in, hipStream_t st) {
    ConvArgs a = in;
    a.ntc = ceil_div(a.Cout, 16);
    a.ntiles = ceil_div(a.P, 16) * a.ntc;
    const double xbytes = (double)a.N * a.H * a.W * a.C * 4, wbytes = (double)a.Cout * a.Kp * 4;
    a.cpx = (a.ntc % 8 == 0 && wbytes > xbytes && wbytes > 1.5 * 1048576) ? a.ntc / 8 : 0;
    const dim3 grid(((a.ntiles + 7) / 8) * 8);
    if (a.ntiles <= 1024) hipLaunchKernelGGL((conv_chain_kernel<8>), grid, dim3(64), 0, st, a);
    else hipLaunchKernelGGL((conv_chain_kernel<4>), grid, dim3(64), 0, st, a);
    SOL_HIP(hipGetLastError());
    return SOL_OK;
}

}  // namespace sol

// Fused convolution (implicit GEMM, up to 32 filter taps) for layers with few output pixels: small tiles, the reduction split
// over the waves of a workgroup, each with an LDS-DMA ring of its own (gfx950).
//
// What bounds these layers.  A 3x3 convolution over 512 channels of one 7x7 image is 0.23 GFLOP and 4.7 MB of weights, a few
// microseconds of the chip's time, but the ring and halo kernels give it to 8 workgroups (64x64 or 64x128 tiles) that each
// walk 4608 reduction elements in up to 72 dependent stages.  What is short is not bandwidth but work in flight: the tiles
// here go down to what one 16x16 MFMA block covers (16 pixels x 16 channels), the reduction is split over the four waves of
// the workgroup, and a wave neither shares tile data nor meets a barrier before the partial sums come together in LDS (added
// in wave order, so the result does not depend on timing).  A stage is 128 bytes of every row, fetched in whole lines by
// buffer_load ... lds (fragments loaded straight from global memory, 16 bytes of 16 rows per instruction, reached 16 bytes per
// clock and CU against 50 this way).  The price of small tiles is traffic, (BP + BC) / (BP * BC) rows per output, so the tile
// grows with the layer and large layers stay on the ring kernels (conv_choose.hip).
// Measured (layer behind 96 MB of other weights; us before -> now): bf16 3x3 512->512 at 7x7, batch 1: 60.3 -> 6.1, batch 8:
// 30.7 -> 8.8, batch 32: 24.4 -> 18.0; 3x3 256->256 at 14x14, batch 1: 21.5 -> 4.7; 1x1 2048->512 at 7x7, batch 1: 14.6 -> 4.5;
// fp32 3x3 512->512 at 7x7, batch 1: 107 -> 11.5, batch 8: 99 -> 25.
// What a launch of one or two stages per wave spends its time on is the way to the first load and the way from the last product to the
// store (an empty kernel 1.7 us, these 3.7 with warm weights): integer divisions for the tile and the first tap, some 380 instructions
// before the first load, a round trip for scale and shift and, for the residual, one per element.  With the divisors as
// multiplications, the weights requested before the pixels' addresses are worked out and the epilogue's operands on their way through the
// whole reduction: ResNet-50-shaped pass, batch 1, 256.3 -> 244.7 us; ResNet-18-shaped, 13 images of 193x193, 210.0 -> 205.0; fp32,
// ResNet-50-shaped, batch 8, 1118 -> 1096.
//
// fp32 runs the same 64-byte steps as four v_mfma_f32_16x16x4_f32 (true fp32 multiplies), whose reduction order inside a
// step is permuted identically for both operands.
//
// The same kernel computes a projection pair (a bottleneck's last 1x1 convolution and the strided 1x1 shortcut it adds): the
// two reductions are walked one behind the other into two sets of accumulators.
#include <math.h>

#include "conv_common.h"

namespace sol {

using lds_pipe::u32x4_t;

// second operand set of a projection pair: unpadded 1x1 convolution of stride `stride` over K2 channels of an H2 x W2 image
struct DirectPair {
    const void *x, *w;
    const float *scale, *shift;
    int H, W, C, Kp, stride;
};

// what the workgroups would otherwise divide for one after the other before their first load (some forty instructions each)
struct DirectGeom {
    FastDiv cpx, ntc, cps, S;              // cpx: of ConvArgs, 1 if that is 0; cps: stages per filter tap
    unsigned taprows;                      // bit r * S for every filter row r
};

// PB x CB: 16-pixel x 16-channel blocks of the tile; NW waves split the reduction; NS: ring stages of each wave
// PRE: relu(pre_scale[c] x + pre_shift[c]) of an unpadded 1x1 convolution's input, applied to the pixels' fragments in registers; the
// stage's constants travel with its weights (one 4-byte DMA instruction).  x may be a channel prefix (ldx)
template <typename T, int PB, int CB, int NW, int NS, bool PAIR, bool PRE>
__global__ void __launch_bounds__(NW * 64) conv_direct_kernel(const ConvArgs a, const DirectPair q, const DirectGeom g) {
#if defined(__HIP_DEVICE_COMPILE__)
    using namespace lds_pipe;
    constexpr int ES = (int)sizeof(T), BP = PB * 16, BC = CB * 16;
    constexpr int ROWB = 128, XL = BP / 8, WL = BC / 8, L = XL + WL + (PRE ? 1 : 0);   // bytes of a row per stage; DMA instructions (8 rows each) per stage
    constexpr int STAGE = (BP + BC) * ROWB + (PRE ? 256 : 0);
    static_assert(!PRE || (ES == 4 && !PAIR), "32 channels per stage");
    constexpr int LSTR = 68;                               // floats between the four 16-lane groups of a parked block: spreads the banks of the epilogue's reads
    constexpr int REDB = NW * PB * CB * 4 * LSTR * 4, RING = NW * NS * STAGE;
    static_assert(RING <= 160 * 1024 && (NS - 1) * L < 64, "LDS, vmcnt");
    __shared__ __align__(1024) unsigned char lds[RING > REDB ? RING : REDB];

    // every kernel argument the prologue needs, fetched in one batch
    asm volatile("" ::"s"(a.x), "s"(a.w), "s"(a.scale), "s"(a.shift), "s"(a.res), "s"(a.P), "s"(a.C), "s"(a.Cout), "s"(a.H), "s"(a.W), "s"(a.Kp),
                 "s"(a.cpx), "s"(a.dw.mul), "s"(a.dh.mul), "s"(a.sh), "s"(a.pool), "s"(a.ph), "s"(g.cpx.mul), "s"(g.ntc.mul), "s"(g.cps.mul), "s"(g.S.mul), "s"(g.taprows));
    if constexpr (PAIR) asm volatile("" ::"s"(q.x), "s"(q.w), "s"(q.scale), "s"(q.shift), "s"(q.H), "s"(q.W), "s"(q.C), "s"(q.Kp), "s"(q.stride));

    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lslot = lane & 7, lrow = lane >> 3;

    // XCD-aware tile order (see conv_dma.hip): a run of tiles per XCD, or a set of channel tiles when the weights are larger
    const int xcd = (int)(blockIdx.x & 7);
    int tile;
    if (a.cpx > 0) {
        uint32_t j, c;
        g.cpx.divmod(blockIdx.x >> 3, j, c);
        tile = (int)j * a.ntc + xcd * a.cpx + (int)c;
    } else {
        tile = xcd * ((a.ntiles + 7) >> 3) + (int)(blockIdx.x >> 3);
    }
    if (tile >= a.ntiles) return;
    uint32_t ptile, ctile;
    g.ntc.divmod((uint32_t)tile, ptile, ctile);
    const int p0 = (int)ptile * BP, c0 = (int)ctile * BC;

    // the activation resource starts `bias` bytes early so that window origins in the padding have offsets >= 0; padding
    // taps and rows beyond the tensor get an out-of-range offset, which the hardware answers with zeros
    const unsigned bias = (unsigned)((a.ph * a.W + a.pw) * a.C) * ES;
    const int ldx = PRE ? a.ldx : a.C;
    const unsigned xbytes = (unsigned)a.N * a.H * a.W * ldx * ES, wbytes = (unsigned)a.Cout * a.Kp * ES;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<unsigned char *>(static_cast<const unsigned char *>(a.x)) - bias, 0, (int)(xbytes + bias), 0x00020000);
    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.w), 0, (int)wbytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t xnull = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.x), 0, 0, 0x00020000);
    const __amdgpu_buffer_rsrc_t wnull = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.w), 0, 0, 0x00020000);

    // this wave's run of stages [s0, s1); a stage is 128 bytes of one filter tap of every row
    const int nmain = a.R * a.S * (int)g.cps.d, nsteps = nmain + (PAIR ? q.C * ES / ROWB : 0);
    const int s0 = (int)((long)nsteps * wave / NW), s1 = (int)((long)nsteps * (wave + 1) / NW);
    unsigned char *ring = lds + wave * (NS * STAGE);
    const unsigned x2bytes = PAIR ? (unsigned)a.N * q.H * q.W * q.C * ES : 0u, w2bytes = PAIR ? (unsigned)a.Cout * q.Kp * ES : 0u;

    // The weights go first: their addresses are cheap, and inside a network they come from the farthest memory.
    unsigned wo[WL], wo2[WL];                              // this lane's rows (wo2: of a projection pair's second convolution)
#pragma unroll
    for (int i = 0; i < WL; i++) {
        const int row = i * 8 + lrow, co = c0 + row;
        wo[i] = co < a.Cout ? (unsigned)(co * a.Kp) * ES + ((lslot ^ swz<ROWB>(row)) << 4) : 0xffffffffu;
        if constexpr (PAIR) wo2[i] = co < a.Cout ? (unsigned)(co * q.Kp) * ES + ((lslot ^ swz<ROWB>(row)) << 4) : 0xffffffffu;
    }
    auto issue_w = [&](int buf, int s) {                   // weights of stage s into ring slot buf; beyond s1 through a size-0 resource -> zeros
        const bool real = s < s1;
        unsigned char *lw = ring + buf * STAGE + BP * ROWB;
        if constexpr (PAIR) {                              // both convolutions are 1x1: stage s is chunk s of the main or chunk s - nmain of the shortcut
            const bool second = s >= nmain;
            const __amdgpu_buffer_rsrc_t wq = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(second ? q.w : a.w), 0, (int)(!real ? 0u : second ? w2bytes : wbytes), 0x00020000);
#pragma unroll
            for (int i = 0; i < WL; i++)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(wq, (__attribute__((address_space(3))) void *)(lw + i * 1024), 16, second ? wo2[i] : wo[i],
                                                         (unsigned)(second ? s - nmain : s) * ROWB, 0, 0);
        } else {
#pragma unroll
            for (int i = 0; i < WL; i++)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(real ? wr : wnull, (__attribute__((address_space(3))) void *)(lw + i * 1024), 16, wo[i], (unsigned)s * ROWB, 0, 0);
        }
        if constexpr (PRE) {                               // 32 factors, 32 summands; beyond s1 the last stage's again, never used
            const float *src = (lane < 32 ? a.pre_scale : a.pre_shift) + min(s, s1 - 1) * 32 + (lane & 31);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src, (__attribute__((address_space(3))) void *)(lw + BC * ROWB), 4, 0, 0);
        }
    };
    const bool any = s0 < s1;
    if (any) static_for<NS>([&](auto B) { issue_w(decltype(B)::value, s0 + decltype(B)::value); });
    keep_order();

    // Epilogue operands of this thread's four channels and IT pixels, behind the weights and ahead of the pixels (the loop's counts of
    // outstanding loads then need not know of them).  Loaded where they are used they cost a round trip, and the residual, whose
    // ragged form reads element by element, four more.
    constexpr int IT = PB * CB > 4 ? PB * CB / 4 : 1;      // pixels per thread without a pool
    static_assert(NW == 4 && (NW * 64) % (BC / 4) == 0, "a thread keeps its channels");
    const bool vec = (a.Cout & 3) == 0 && a.Cout <= 1 << 22;
    typedef __attribute__((ext_vector_type(ES == 2 ? 2 : 4))) unsigned ResVec;
    const int ecg = tid % (BC / 4), epx = tid / (BC / 4);
    u32x4_t esc, esf, esf2, psc[PAIR ? CB : 1], psc2[PAIR ? CB : 1];
    ResVec eres[IT];
    {
        auto floats = [&](const float *p) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p), 0, vec && p ? a.Cout * 4 : 0, 0x00020000); };
        const unsigned co = (unsigned)(c0 + ecg * 4) * 4u;
        esf = __builtin_amdgcn_raw_buffer_load_b128(floats(a.shift), co, 0, 0);
        if constexpr (PAIR) {
            esf2 = __builtin_amdgcn_raw_buffer_load_b128(floats(q.shift), co, 0, 0);
#pragma unroll
            for (int i = 0; i < CB; i++) {                 // of the channels of this lane's accumulators
                psc[i] = __builtin_amdgcn_raw_buffer_load_b128(floats(a.scale), (unsigned)(c0 + i * 16 + lg * 4) * 4u, 0, 0);
                psc2[i] = __builtin_amdgcn_raw_buffer_load_b128(floats(q.scale), (unsigned)(c0 + i * 16 + lg * 4) * 4u, 0, 0);
            }
        } else {
            esc = __builtin_amdgcn_raw_buffer_load_b128(floats(a.scale), co, 0, 0);
        }
        if (a.res && vec) {
            const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(static_cast<const T *>(a.res) + (size_t)p0 * a.Cout), 0,
                                                                                (int)((unsigned)min(BP, a.P - p0) * (unsigned)a.Cout * ES), 0x00020000);
#pragma unroll
            for (int u = 0; u < IT; u++) {
                const unsigned o = ((unsigned)(epx + u * (NW * 64 / (BC / 4))) * (unsigned)a.Cout + (unsigned)(c0 + ecg * 4)) * ES;
                if constexpr (ES == 2) eres[u] = __builtin_amdgcn_raw_buffer_load_b64(rr, o, 0, 0); else eres[u] = __builtin_amdgcn_raw_buffer_load_b128(rr, o, 0, 0);
            }
        }
    }
    keep_order();

    unsigned xo[XL], xinv[XL], xo2[XL];                    // this lane's rows; bit t of xinv: filter tap t reads padding
#pragma unroll
    for (int i = 0; i < XL; i++) {
        const int row = i * 8 + lrow, m = p0 + row;
        int n, op, oq;
        decode_pixel(a, m, n, op, oq);
        const int ih0 = op * a.sh - a.ph, iw0 = oq * a.sw - a.pw;
        const unsigned off = (unsigned)(((n * a.H + ih0) * a.W + iw0) * ldx) * ES + bias + ((lslot ^ swz<ROWB>(row)) << 4);
        const int slo = max(0, -iw0), shi = min(a.S, a.W - iw0), rlo = max(0, -ih0), rhi = min(a.R, a.H - ih0);
        const unsigned cval = shi > slo ? (unsigned)((1ull << shi) - 1ull) & ~((1u << slo) - 1u) : 0u;
        // filter rows [rlo, rhi) as bits r * S; times the columns' bits, of which a row has S: no carries
        const unsigned rval = rhi > rlo ? g.taprows & (unsigned)((1ull << (rhi * a.S)) - (1ull << (rlo * a.S))) : 0u;
        xo[i] = m < a.P ? off : 0xffffffffu;
        xinv[i] = ~(cval * rval);
        if constexpr (PAIR) xo2[i] = m < a.P ? (unsigned)(((n * q.H + op * q.stride) * q.W + oq * q.stride) * q.C) * ES + ((lslot ^ swz<ROWB>(row)) << 4) : 0xffffffffu;
    }
    uint32_t utap, utc, utr, uts;
    g.cps.divmod((uint32_t)s0, utap, utc);
    g.S.divmod(utap, utr, uts);
    const int cps = (int)g.cps.d;
    int s = s0, tap = (int)utap, tc = (int)utc, tr = (int)utr, ts = (int)uts;
    auto issue_x = [&](int buf) {                          // pixels of the next stage into ring slot buf
        const bool real = s < s1;
        unsigned char *lx = ring + buf * STAGE;
        if constexpr (PAIR) {
            const bool second = s >= nmain;
            const __amdgpu_buffer_rsrc_t xq = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(second ? q.x : a.x), 0, (int)(!real ? 0u : second ? x2bytes : xbytes), 0x00020000);
#pragma unroll
            for (int i = 0; i < XL; i++)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xq, (__attribute__((address_space(3))) void *)(lx + i * 1024), 16, second ? xo2[i] : xo[i],
                                                         (unsigned)(second ? s - nmain : s) * ROWB, 0, 0);
            ++s;
            return;
        }
        const unsigned xs = (unsigned)((tr * a.W + ts) * a.C) * ES + (unsigned)tc * ROWB;
#pragma unroll
        for (int i = 0; i < XL; i++) {
            const unsigned off = xo[i] | (unsigned)__builtin_amdgcn_sbfe(xinv[i], tap, 1);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(real ? xr : xnull, (__attribute__((address_space(3))) void *)(lx + i * 1024), 16, off, xs, 0, 0);
        }
        ++s;
        if (++tc == cps) { tc = 0; ++tap; if (++ts == a.S) { ts = 0; ++tr; } }
    };
    f32x4_t acc[CB][PB], acc2[CB][PB];
#pragma unroll
    for (int i = 0; i < CB; i++)
#pragma unroll
        for (int j = 0; j < PB; j++) acc[i][j] = acc2[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    const unsigned fsw = swz<ROWB>(lr);                    // block row bases are multiples of 16: the swizzle depends on lr only
    const unsigned f0 = lds_addr(ring) + lr * ROWB + ((lg ^ fsw) << 4), f1 = lds_addr(ring) + lr * ROWB + (((lg + 4) ^ fsw) << 4);

    if (any) {
        static_for<NS>([&](auto B) { issue_x(decltype(B)::value); });
        int buf = 0;
        // Stage k has landed once only what was issued after its pixels is outstanding (the ring is this wave's own: no barrier): the
        // pixels alone of the other stages that the loop found under way, and the stages that it issued.
        auto stage = [&](int k, auto OUTSTANDING) {
            wait_vmcnt<decltype(OUTSTANDING)::value>();
            u32x4_t fw[2][CB], fx[2][PB];
            const unsigned b0 = f0 + buf * STAGE, b1 = f1 + buf * STAGE;
            static_for<CB>([&](auto I) { lds_read16<BP * ROWB + decltype(I)::value * 16 * ROWB>(fw[0][decltype(I)::value], b0); });
            static_for<PB>([&](auto J) { lds_read16<decltype(J)::value * 16 * ROWB>(fx[0][decltype(J)::value], b0); });
            static_for<CB>([&](auto I) { lds_read16<BP * ROWB + decltype(I)::value * 16 * ROWB>(fw[1][decltype(I)::value], b1); });
            static_for<PB>([&](auto J) { lds_read16<decltype(J)::value * 16 * ROWB>(fx[1][decltype(J)::value], b1); });
            u32x4_t pk[PRE ? 4 : 1];                       // this lane's 4 + 4 channels: factors, summands
            if constexpr (PRE) {
                const unsigned cb = lds_addr(ring) + buf * STAGE + (BP + BC) * ROWB + lg * 16;
                lds_read16<0>(pk[0], cb); lds_read16<128>(pk[1], cb); lds_read16<64>(pk[2], cb); lds_read16<192>(pk[3], cb);
            }
            wait_lgkmcnt<0>();
            if constexpr (PRE) { landed(pk[0]); landed(pk[1]); landed(pk[2]); landed(pk[3]); }
            static_for<2>([&](auto H) {
                static_for<CB>([&](auto I) { landed(fw[decltype(H)::value][decltype(I)::value]); });
                static_for<PB>([&](auto J) { landed(fx[decltype(H)::value][decltype(J)::value]); });
            });
            if constexpr (PRE) {
#pragma unroll
                for (int h = 0; h < 2; h++)
#pragma unroll
                    for (int j = 0; j < PB; j++)
#pragma unroll
                        for (int e = 0; e < 4; e++)
                            fx[h][j][e] = __float_as_uint(__builtin_fmaxf(__uint_as_float(fx[h][j][e]) * __uint_as_float(pk[2 * h][e]) + __uint_as_float(pk[2 * h + 1][e]), 0.f));
            }
            issue_w(buf, s);                               // the slot's data is in registers: refill it
            issue_x(buf);
            auto contract = [&](f32x4_t (&to)[CB][PB]) {
#pragma unroll
                for (int h = 0; h < 2; h++)
#pragma unroll
                    for (int i = 0; i < CB; i++)
#pragma unroll
                        for (int j = 0; j < PB; j++) Mma16<T>::run(to[i][j], fw[h][i], fx[h][j]);
            };
            if (PAIR && k >= nmain) contract(acc2); else contract(acc);
            buf = buf + 1 == NS ? 0 : buf + 1;
        };
        stage(s0, std::integral_constant<int, (NS - 1) * XL>{});
        int k = s0 + 1;
        if constexpr (NS > 2) {
            static_assert(NS <= 3, "a wait for every stage under way");
            if (k < s1) stage(k++, std::integral_constant<int, (NS - 2) * XL + L>{});
        }
        for (; k < s1; k++) stage(k, std::integral_constant<int, (NS - 1) * L>{});
        wait_vmcnt<0>();                                   // the zero-fill DMAs of the tail
    }
    if constexpr (PAIR) {                                  // fold the two sums: their scales differ, so they meet here; the shifts follow in the epilogue
#pragma unroll
        for (int i = 0; i < CB; i++)
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const int co = c0 + i * 16 + lg * 4 + e, cc = co < a.Cout ? co : 0;
                const float sm = !a.scale ? 1.f : vec ? __uint_as_float(psc[i][e]) : a.scale[cc];
                const float ss = !q.scale ? 1.f : vec ? __uint_as_float(psc2[i][e]) : q.scale[cc];
#pragma unroll
                for (int j = 0; j < PB; j++) acc[i][j][e] = acc[i][j][e] * sm + acc2[i][j][e] * ss;
            }
    }
    __syncthreads();                                       // every ring is dead: the LDS becomes the parking place of the partial sums
    typedef float Block[4 * LSTR];
    Block *red = reinterpret_cast<Block *>(lds);           // [wave][block]

    // accumulator register e of lane l: channel 4 * (l / 16) + e, pixel l % 16 of its block
#pragma unroll
    for (int i = 0; i < CB; i++)
#pragma unroll
        for (int j = 0; j < PB; j++)
            *reinterpret_cast<float4 *>(&red[wave * PB * CB + j * CB + i][lg * LSTR + lr * 4]) = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
    __syncthreads();

    // four channels of one pixel (of one pooling window) per thread, channels fastest
    T *__restrict__ yg = static_cast<T *>(a.y);
    const T *__restrict__ resg = static_cast<const T *>(a.res);
    const int npix = a.pool ? BP / 4 : BP, cg = ecg, cb = c0 + cg * 4, nv = min(4, a.Cout - cb);
    if (nv <= 0) return;
    float sc[4], sf[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
        if (vec) {
            sc[e] = !PAIR && a.scale ? __uint_as_float(esc[e]) : 1.f;
            sf[e] = __uint_as_float(esf[e]);
            if (PAIR) sf[e] += __uint_as_float(esf2[e]);
        } else {
            sc[e] = (!PAIR && a.scale && e < nv) ? a.scale[cb + e] : 1.f;
            sf[e] = (a.shift && e < nv) ? a.shift[cb + e] : 0.f;
            if (PAIR) sf[e] += (q.shift && e < nv) ? q.shift[cb + e] : 0.f;
        }
    }
#pragma unroll
    for (int u = 0; u < IT; u++) {
        const int px = epx + u * (NW * 64 / (BC / 4)), m0 = p0 + (a.pool ? px * 4 : px);
        if (px >= npix || m0 >= a.P) break;
        float out[4];
        auto finish = [&](int row, float v[4]) {           // act(scale * sum + shift + residual) of tile row `row`
            const int blk = (row >> 4) * CB + (cg >> 2), at = (cg & 3) * LSTR + (row & 15) * 4;
            float4 t = *reinterpret_cast<const float4 *>(&red[blk][at]);
#pragma unroll
            for (int w = 1; w < NW; w++) {
                const float4 q = *reinterpret_cast<const float4 *>(&red[w * PB * CB + blk][at]);
                t.x += q.x; t.y += q.y; t.z += q.z; t.w += q.w;
            }
            v[0] = t.x * sc[0] + sf[0]; v[1] = t.y * sc[1] + sf[1]; v[2] = t.z * sc[2] + sf[2]; v[3] = t.w * sc[3] + sf[3];
            if (resg && vec) {
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    if constexpr (ES == 2) v[e] += __uint_as_float(e & 1 ? eres[u][e >> 1] & 0xffff0000u : eres[u][e >> 1] << 16);
                    else v[e] += __uint_as_float(eres[u][e]);
                }
            } else if (resg) {
                const T *rp = resg + (long)(p0 + row) * a.Cout + cb;
#pragma unroll
                for (int e = 0; e < 4; e++) v[e] += e < nv ? Elem<T>::load(rp + e) : 0.f;
            }
            if (a.act == SOL_ACT_RELU) {
#pragma unroll
                for (int e = 0; e < 4; e++) v[e] = __builtin_fmaxf(v[e], 0.f);
            }
        };
        if (!a.pool) {
            finish(px, out);
        } else {                                           // rows 4w .. 4w + 3 are pooling window w, in row-major order
            finish(px * 4, out);
#pragma unroll
            for (int d = 1; d < 4; d++) {
                float v[4];
                finish(px * 4 + d, v);
#pragma unroll
                for (int e = 0; e < 4; e++) out[e] = a.pool == 1 ? (v[e] > out[e] ? v[e] : out[e]) : out[e] + v[e];
            }
            if (a.pool == 2) {
#pragma unroll
                for (int e = 0; e < 4; e++) out[e] *= 0.25f;
            }
        }
        T *yp = yg + (long)(a.pool ? m0 >> 2 : m0) * a.ldy + cb;
        if (nv == 4 && ((a.ldy | a.Cout) & 3) == 0) {
            if constexpr (ES == 2) *reinterpret_cast<uint2 *>(yp) = make_uint2(pack_bf16x2(out[0], out[1]), pack_bf16x2(out[2], out[3]));
            else *reinterpret_cast<float4 *>(yp) = make_float4(out[0], out[1], out[2], out[3]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; e++)
                if (e < nv) Elem<T>::store(yp + e, out[e]);
        }
    }
#endif
}

template <typename T, int PB, int CB, int NW, int NS>
static sol_status launch_direct_cfg(ConvArgs a, const DirectPair *q, hipStream_t st) {
    a.ntc = ceil_div(a.Cout, CB * 16);
    a.ntiles = ceil_div(a.P, PB * 16) * a.ntc;
    const int grid = ((a.ntiles + 7) / 8) * 8;
    const double xbytes = (double)a.N * a.H * a.W * a.C * sizeof(T), wbytes = (double)a.Cout * a.Kp * sizeof(T);
    a.cpx = (a.ntc % 8 == 0 && wbytes > xbytes) ? a.ntc / 8 : 0;
    DirectGeom g{FastDiv((uint32_t)(a.cpx > 0 ? a.cpx : 1)), FastDiv((uint32_t)a.ntc), FastDiv((uint32_t)(a.C * sizeof(T) / 128)), FastDiv((uint32_t)a.S), 0u};
    for (int r = 0; r < a.R; r++) g.taprows |= 1u << (r * a.S);
    if constexpr (sizeof(T) == 2) {
        if (q) {
            hipLaunchKernelGGL((conv_direct_kernel<T, PB, CB, NW, NS, true, false>), dim3(grid), dim3(NW * 64), 0, st, a, *q, g);
            SOL_HIP(hipGetLastError());
            return SOL_OK;
        }
    }
    if constexpr (sizeof(T) == 4) {
        if (a.pre_scale) {
            hipLaunchKernelGGL((conv_direct_kernel<T, PB, CB, NW, NS, false, true>), dim3(grid), dim3(NW * 64), 0, st, a, DirectPair{}, g);
            SOL_HIP(hipGetLastError());
            return SOL_OK;
        }
    }
    hipLaunchKernelGGL((conv_direct_kernel<T, PB, CB, NW, NS, false, false>), dim3(grid), dim3(NW * 64), 0, st, a, DirectPair{}, g);
    SOL_HIP(hipGetLastError());
    return SOL_OK;
}

// Stages of 128 bytes inside one filter tap, one validity bit per tap, 32-bit byte offsets; no winners / pre-pool tensor, no
// residual in front of a pool.
bool direct_kernel_applies(const ConvArgs &a, int dt) {
    const double es = (double)dtype_size(dt), xb = (double)a.N * a.H * a.W * a.C * es + (double)(a.ph * a.W + a.pw) * a.C * es;
    return a.R * a.S <= 32 && (a.C * (int)es) % 128 == 0 && a.pool <= 2 && !(a.pool && a.res) && !a.argmax && !a.prepool && xb < 2147483648.0 &&
           (double)a.Cout * a.Kp * es < 2147483648.0;
}

template <typename T> static sol_status launch_direct_typed(const ConvArgs &a, int tile, const DirectPair *q, hipStream_t st) {
    switch (tile) {
        //                                              PB CB NW NS
        case S_16x16: return launch_direct_cfg<T, 1, 1, 4, 3>(a, q, st);      // 48 KB of LDS: three workgroups per CU
        case S_16x32: return launch_direct_cfg<T, 1, 2, 4, 3>(a, q, st);      // 72 KB: two
        case S_32x32: return launch_direct_cfg<T, 2, 2, 4, 2>(a, q, st);      // 64 KB: two
        case S_64x32: return launch_direct_cfg<T, 4, 2, 4, 2>(a, q, st);      // 96 KB: one
        case S_64x64: return launch_direct_cfg<T, 4, 4, 4, 2>(a, q, st);      // 128 KB: one
        default: SOL_FAIL(SOL_ERR_UNSUPPORTED, "unknown direct conv tile id %d", tile);
    }
}

sol_status launch_conv_direct(const ConvArgs &a, int dt, int tile, hipStream_t st) {
    return dt == SOL_BF16 ? launch_direct_typed<bf16_t>(a, tile, nullptr, st) : launch_direct_typed<float>(a, tile, nullptr, st);
}

// The projection pair (bf16) on this kernel: which tile, or T_AUTO for the pair kernels, whose one 128x128 tile per workgroup
// walks (K + K2) / 64 chunks of 0.87 us behind a start of 2.8 us as long as the tiles do not fill the chip.  The two operand
// sets cost this kernel about a fifth on top of the estimate of one.  Measured (K + K2 -> channels, pixels; us pair kernel ->
// this one): 512 + 1024 -> 2048, 49: 23.4 -> 5.8; the same, 392: 26.8 -> 15.7; 256 + 512 -> 1024, 784: 15.9 -> 12.3; the same,
// 1568: 16.3, 20.8 here; 64 + 64 -> 256, 3136: 4.8, 8.5 here.
int direct_choose_pair_tile(const ConvArgs &a, int K2) {
    if (!direct_kernel_applies(a, SOL_BF16) || K2 % 64 != 0) return T_AUTO;
    int best = T_AUTO;
    float bt = 2.8f + 0.87f * (float)((a.C + K2) / 64);
    for (int t = S_FIRST; t <= S_64x32; t++) {
        const float c = 1.2f * conv_tile_estimate(t, SOL_BF16, a.P, a.Cout, 2.f * (float)(a.C + K2), 0.f, 0.f);
        if (c < bt) { best = t; bt = c; }
    }
    return best;
}

// A pre-activated 1x1 convolution in fp32 on this kernel (see PRE), or T_AUTO: whole 32-channel stages, all of them valid, no padding (which
// the activation would not leave at 0).  The register-staged kernel has one 128-pixel tile per workgroup, one wave per SIMD in step with the
// others, whatever the layer's size: a DenseNet-121-shaped pass (us, it alone -> here): 1 image of 224x224 3377 -> 698, 3 of 64x64 3331 -> 657,
// 8 of 100x100 3381 -> 741, 8 of 224x224 3744 -> 1249.
int direct_choose_pre_tile(const ConvArgs &a, int dt) {
    if (dt != SOL_F32 || !a.pre_scale || a.R * a.S != 1 || a.ph || a.pw || a.Cvalid != a.C || !direct_kernel_applies(a, dt) ||
        (double)a.N * a.H * a.W * a.ldx * 4.0 >= 2147483648.0) return T_AUTO;
    int best = S_FIRST;
    float bt = INFINITY;
    for (int t = S_FIRST; t <= S_LAST; t++) {
        const float c = conv_tile_estimate(t, SOL_F32, a.P, a.Cout, 4.f * (float)a.C, a.res ? 1.f : 0.f, 0.f);
        if (c < bt) { best = t; bt = c; }
    }
    return best;
}
sol_status launch_conv_direct_pair(const ConvArgs &a, int tile, const void *x2, const void *w2, const float *scale2, const float *shift2, int H2,
                                   int W2, int K2, int Kp2, int stride, hipStream_t st) {
    const DirectPair q{x2, w2, scale2, shift2, H2, W2, K2, Kp2, stride};
    return launch_direct_typed<bf16_t>(a, tile, &q, st);
}

}  // namespace sol

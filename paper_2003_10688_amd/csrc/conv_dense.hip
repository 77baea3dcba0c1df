// A dense layer of a DenseNet-shaped block as one depth-first kernel (gfx950):
//   t1 = relu(s1 * conv1x1(relu(ps * x + ph), w1) + h1)      C -> 128 channels, x a channel prefix of the block's buffer
//   y  = act(s2 * conv3x3(t1, w2) + h2)                       128 -> 32 channels, stride 1, pad 1, written in place behind the prefix
//
// The paper's layer-chain fusion (Sec. III-A) across two contractions: t1 never reaches device memory.  What bounded the two
// launches it replaces: the 1x1 convolution ran on the register-staged kernel (the one that can apply BN + ReLU to its input on
// the way to LDS), 104 to 1568 tiles of 128 pixels with one chunk of 64 channels in flight and every operand through
// registers and two barriers; the 3x3 convolution has only 32 filters, so its 256-pixel tiles were as few as 14.
//
// A workgroup owns `bp` consecutive pixels (n, h, w flattened) and computes t1 for the PR rows [p0 - W - 1, p0 + bp + W + 1).
//  Phase A walks C in chunks of 64 channels.  x rows go global -> registers (DX chunks ahead) -> BN + ReLU -> LDS (two chunk
//    buffers); w1 chunks (128 rows x 128 B) travel by LDS DMA through a ring of NSW stages of 16 KB.  One barrier per chunk.
//  t1 takes the place of the two chunk buffers (PR rows x 256 B, rounded to bf16 where the layer-by-layer path stores it).
//  Phase B runs the nine taps from that patch (row of pixel m, tap (r, s): m + r * W + s; taps outside the image are redirected
//    to a zero row); w2 continues in the same ring, two taps to a stage.  The waves split the reduction KSB ways, and
//    the partial sums meet in LDS in a fixed order.
// Measured (batch 64, two launches -> one): 56x56, 64..224 channels: 76 -> 41..66 us; 28x28, 128..480: 30 -> 14..22; 14x14,
// 256..992: 29 -> 10..18; 7x7, 512..992: 24 -> 10..13; DenseNet-121-shaped pass 2343 -> 1292 us.  A chunk of phase A costs a
// workgroup 0.4 us (64 rows) to 1.5 us (384): BN + ReLU, fragment reads, MFMAs and DMA issue of a chunk take about a
// quarter of that each and hardly overlap, since all eight waves run the same sequence between two barriers.  (Half of the
// waves in the other order, transform against multiply: slower, 18.0 -> 20.2 us at 14x14; it doubles the code and the registers.)
// All LDS accesses between DMAs are opaque statements (the compiler would make each of them wait for every DMA in flight).
#include "conv_common.h"

namespace sol {

namespace {
using lds_pipe::u32x4_t;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2_t;

template <int O> __device__ __forceinline__ void lds_write16(unsigned addr, const u32x4_t &v) {
    asm volatile("ds_write_b128 %0, %1 offset:%2" ::"v"(addr), "v"(v), "n"(O) : "memory");
}
__device__ __forceinline__ void lds_write8(unsigned addr, const u32x2_t &v) { asm volatile("ds_write_b64 %0, %1" ::"v"(addr), "v"(v) : "memory"); }

constexpr int DN_MID = 128, DN_OUT = 32, DN_CMAX = 1024;   // filters of the 1x1 / of the 3x3 convolution; widest input prefix

// Taps of pixel m of a workgroup's bp pixels, bit t = 3 r + s: those inside the image (cols: bits of the three columns; up, down:
// the rows above and below exist).  A pixel past bp has none: its tap (r, s) would be patch row m + r W + s, and with
// bp = rows - 2 W - 2 that lies behind the patch, in the ring that a DMA is filling or past the end of LDS.
__host__ __device__ constexpr unsigned dense_taps(int m, int bp, unsigned cols, bool up, bool down) {
    return m < bp ? (up ? cols : 0u) | cols << 3 | (down ? cols << 6 : 0u) : 0u;
}
constexpr bool dense_taps_inside(int rows) {               // the ninth tap is the farthest
    for (int W = 1; W < rows / 2; W++)
        for (int m = 0; m < rows; m++)
            if ((dense_taps(m, rows - 2 * W - 2, 7u, true, true) >> 8 & 1u) && m + 2 * W + 2 >= rows) return false;
    return true;
}
static_assert(dense_taps_inside(64) && dense_taps_inside(96) && dense_taps_inside(128) && dense_taps_inside(192) && dense_taps_inside(256) &&
              dense_taps_inside(384), "every tap read lies in the patch");

struct DenseArgs {
    DenseLaunch d;
    int bp, ntiles, nc;        // pixels per workgroup; workgroups; chunks of 64 input channels
};

// PA x CA: 16-pixel x 16-channel blocks of t1 per wave; WPA x (8 / WPA): wave grid of phase A; KSB: reduction split of phase B
// (the other 8 / KSB waves split the pixels); DX: x chunks in flight in registers; NSW: weight ring stages
template <int PA, int CA, int WPA, int KSB, int DX, int NSW>
__global__ void __launch_bounds__(512) conv_dense_kernel(const DenseArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
    using namespace lds_pipe;
    constexpr int WCA = 8 / WPA, PR = WPA * PA * 16, WPB = 8 / KSB, NB = PR / 16 / WPB, KPW = 8 / KSB;
    static_assert(WCA * CA * 16 == DN_MID && PR / 16 % WPB == 0, "wave grids");
    constexpr int XR = (PR * 8 + 511) / 512;               // 16-byte pieces of an x chunk per thread
    constexpr int WST = 16384, LSTR = 68;
    constexpr int TB = PR * 256, ZROW = TB, RING0 = TB + 256, PRE0 = RING0 + NSW * WST, AFF0 = PRE0 + 2 * DN_CMAX * 4, LDSB = AFF0 + 2 * (DN_MID + DN_OUT) * 4;
    static_assert(LDSB <= 160 * 1024 && KSB * WPB * NB * 2 * 4 * LSTR * 4 <= PRE0, "LDS");
    static_assert((NSW - 1) * (XR + 2) < 60 && (DX - 1) * (XR + 2) + 2 < 60, "vmcnt");
    __shared__ __align__(1024) unsigned char lds[LDSB];

    const DenseLaunch &d = a.d;
    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile = (int)(blockIdx.x & 7) * ((a.ntiles + 7) >> 3) + (int)(blockIdx.x >> 3);     // a contiguous run of tiles per XCD
    if (tile >= a.ntiles) return;
    const int W = d.W, P = d.N * d.H * W, p0 = tile * a.bp, bp = min(a.bp, P - p0), nc = a.nc;
    const unsigned lbase = lds_addr(lds);

    const unsigned xbytes = (unsigned)P * d.ldx * 2, w1bytes = (unsigned)DN_MID * d.Kp1 * 2, w2bytes = (unsigned)DN_OUT * 9 * DN_MID * 2;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(d.x), 0, (int)xbytes, 0x00020000);

    // ---- weight ring: stages 0 .. nc - 1 are chunks of w1 (128 rows x 128 B), nc .. nc + 4 pairs of taps of w2 (2 x 32 rows x 256 B)
    unsigned wo1[2], wo2[2];
#pragma unroll
    for (int i = 0; i < 2; i++) {
        const int seg = wave * 2 + i, r1 = seg * 8 + (lane >> 3), r2 = (seg & 7) * 4 + (lane >> 4);
        wo1[i] = (unsigned)(r1 * d.Kp1) * 2 + (((lane & 7) ^ swz<128>(r1)) << 4);
        wo2[i] = (unsigned)(r2 * 9 * DN_MID) * 2 + (seg >> 3) * 256 + (((lane & 15) ^ (r2 & 15)) << 4);
    }
    int wslot = 0, wstage = 0;
    auto issue_w = [&]() {
        const bool second = wstage >= nc;
        const int j = wstage - nc;
        const unsigned size = !second ? w1bytes : j < 5 ? w2bytes : 0u;          // past the end (and the tap beyond the ninth): zeros
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(second ? d.w2 : d.w1), 0, (int)size, 0x00020000);
        const unsigned so = second ? (unsigned)j * 512u : (unsigned)wstage * 128u;
#pragma unroll
        for (int i = 0; i < 2; i++) {
            const bool none = second && j == 4 && wave >= 4;                      // the tenth tap does not exist
            const unsigned off = none ? 0xffffffffu : second ? wo2[i] : wo1[i];
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)(lds + RING0 + wslot * WST + (wave * 2 + i) * 1024), 16, off, so, 0, 0);
        }
        wslot = wslot + 1 == NSW ? 0 : wslot + 1;
        ++wstage;
    };
    // ---- x rows: piece i of this thread = 16-byte slot (tid & 7) of patch row (tid >> 3) + 64 * i
    const int xslot = tid & 7;
    // byte offset of piece 0 in x; rows outside x wrap or run past its end, where the buffer's own check returns zeros (nothing reads
    // what becomes of them: their taps are padding).  The other pieces' offsets are added up at each load and not kept in registers.
    const unsigned xo = (unsigned)((p0 - W - 1 + (tid >> 3)) * d.ldx) * 2 + (xslot << 4), xstep = (unsigned)d.ldx * 128;
    // LDS offset of piece 0 inside a chunk buffer; piece i lies 64 rows on, where the slot permutation is the same: an immediate
    // offset (an address per piece took the 384-row variant over 256 registers, 16 bytes of scratch per lane;
    // without them the DenseNet-121-shaped pass, batch 64, takes 1292 us instead of 1300)
    const unsigned xl = (unsigned)(tid >> 3) * 128 + ((xslot ^ swz<128>(tid >> 3)) << 4);
    u32x4_t xv[DX][XR];
    auto load_x = [&](auto S, int c) {
        constexpr int s = decltype(S)::value;
        const unsigned so = (unsigned)min(c, nc - 1) * 128u;
        unsigned off = xo, by = xstep;
        asm volatile("" : "+s"(by));                       // not an invariant of the loop, to the compiler
#pragma unroll
        for (int i = 0; i < XR; i++, off += by)
            xv[s][i] = __builtin_amdgcn_raw_buffer_load_b128(xr, XR * 64 == PR || (tid >> 3) + 64 * i < PR ? off : 0xffffffffu, so, 0);
    };
    // input-side constants of this thread's eight channels of the next chunk to go to LDS; fetched one iteration ahead
    u32x4_t q[4];
    auto read_pre = [&](int c) {
        const unsigned pa = lbase + PRE0 + (unsigned)(min(c, nc - 1) * 64 + xslot * 8) * 4;
        lds_read16<0>(q[0], pa);
        lds_read16<16>(q[1], pa);
        lds_read16<DN_CMAX * 4>(q[2], pa);
        lds_read16<DN_CMAX * 4 + 16>(q[3], pa);
    };
    auto pre_landed = [&]() {
#pragma unroll
        for (int e = 0; e < 4; e++) landed(q[e]);
    };
    // relu(scale * x + shift) of chunk c from register set S into chunk buffer c & 1; channels past the prefix are zeros
    auto put_x = [&](auto S, int c) {
        constexpr int s = decltype(S)::value;
        const unsigned xb = lbase + (c & 1) * (PR * 128) + xl;
        static_for<XR>([&](auto I) {
            constexpr int i = decltype(I)::value;
            u32x4_t o;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const unsigned u = xv[s][i][e];
                const float lo = __uint_as_float(u << 16), hi = __uint_as_float(u & 0xffff0000u);
                const float a0 = lo * __uint_as_float(q[e >> 1][(e & 1) * 2]) + __uint_as_float(q[2 + (e >> 1)][(e & 1) * 2]);
                const float a1 = hi * __uint_as_float(q[e >> 1][(e & 1) * 2 + 1]) + __uint_as_float(q[2 + (e >> 1)][(e & 1) * 2 + 1]);
                o[e] = pack_bf16x2(__builtin_fmaxf(a0, 0.f), __builtin_fmaxf(a1, 0.f));
            }
            if (c * 64 + 64 > d.Cvalid) {
                const int left = d.Cvalid - (c * 64 + xslot * 8);                  // real channels among this piece's eight
#pragma unroll
                for (int e = 0; e < 4; e++) o[e] = left >= 2 * e + 2 ? o[e] : left == 2 * e + 1 ? o[e] & 0xffffu : 0u;
            }
            if (XR * 64 == PR || (tid >> 3) + 64 * i < PR) lds_write16<i * 8192>(xb, o);
        });
    };

    // ---- prologue
#pragma unroll
    for (int s = 0; s < NSW - 1; s++) issue_w();
    static_for<DX>([&](auto S) { load_x(S, decltype(S)::value); });
    {   // every per-channel constant into LDS: all loads in flight before the first is stored
        float *pre = reinterpret_cast<float *>(lds + PRE0), *aff = reinterpret_cast<float *>(lds + AFF0);
        float v[5];
        const int c0 = min(tid, d.Cvalid - 1), c1 = min(tid + 512, d.Cvalid - 1);
        v[0] = d.ps[c0]; v[1] = d.ph[c0]; v[2] = d.ps[c1]; v[3] = d.ph[c1];
        const float *src = tid < 128 ? d.s1 + tid : tid < 256 ? d.h1 + (tid - 128) : tid < 288 ? d.s2 + (tid - 256) : tid < 320 ? d.h2 + (tid - 288) : d.s1;
        v[4] = *src;
        __builtin_amdgcn_sched_barrier(0);
        pre[tid] = v[0]; pre[DN_CMAX + tid] = v[1]; pre[512 + tid] = v[2]; pre[DN_CMAX + 512 + tid] = v[3];
        if (tid < 2 * (DN_MID + DN_OUT)) aff[tid] = v[4];
        if (tid < 64) reinterpret_cast<unsigned *>(lds + ZROW)[tid] = 0u;
    }
    __syncthreads();

    f32x4_t acc[CA][PA];
#pragma unroll
    for (int i = 0; i < CA; i++)
#pragma unroll
        for (int j = 0; j < PA; j++) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const int wpa = wave % WPA, wca = wave / WPA;
    // slot of the first k-step's fragment included; the second one's is four slots away: bit 6 of the address flipped
    const unsigned so0 = (lg ^ swz<128>(lr)) << 4, fx = lbase + (wpa * PA * 16 + lr) * 128 + so0, fw = lbase + RING0 + (wca * CA * 16 + lr) * 128 + so0;

    read_pre(0);
    wait_lgkmcnt<0>();
    pre_landed();
    put_x(std::integral_constant<int, 0>{}, 0);
    load_x(std::integral_constant<int, 0>{}, DX);
    // ---- phase A.  Iteration c uses chunk c, moves chunk c + 1 from register set (c + 1) % DX to LDS and refills that set.
    // (Opaque LDS reads are always waited for before the next branch: a register they have yet to fill must not be copied.)
    constexpr bool BOTH = PA * CA <= 16;                   // registers for the fragments of both k-steps at once
    int rs = 0;                                            // ring slot of the current stage
    auto step = [&](auto S, auto TAIL, int c) {            // S: register set of chunk c + 1
        wait_vmcnt<XR + (NSW - 2) * (XR + 2)>();           // weight stage c: only what was issued after it is outstanding
        wait_lgkmcnt<0>();
        __builtin_amdgcn_s_barrier();                      // ... for every wave; chunk c is in LDS; nobody still reads chunk c - 1
        const unsigned xb = fx + (c & 1) * (PR * 128), wb = fw + rs * WST;
        u32x4_t fa[BOTH ? 2 : 1][CA], fb[BOTH ? 2 : 1][PA];
        auto read = [&](auto H, auto F) {
            constexpr int f = decltype(F)::value;
            constexpr unsigned flip = decltype(H)::value * 64;
            static_for<CA>([&](auto I) { lds_read16<decltype(I)::value * 2048>(fa[f][decltype(I)::value], wb ^ flip); });
            static_for<PA>([&](auto J) { lds_read16<decltype(J)::value * 2048>(fb[f][decltype(J)::value], xb ^ flip); });
        };
        auto frags_landed = [&](auto F) {
            constexpr int f = decltype(F)::value;
            static_for<CA>([&](auto I) { landed(fa[f][decltype(I)::value]); });
            static_for<PA>([&](auto J) { landed(fb[f][decltype(J)::value]); });
        };
        auto contract = [&](auto F) {
            constexpr int f = decltype(F)::value;
#pragma unroll
            for (int i = 0; i < CA; i++)
#pragma unroll
                for (int j = 0; j < PA; j++) Mma16<bf16_t>::run(acc[i][j], fa[f][i], fb[f][j]);
        };
        using I0 = std::integral_constant<int, 0>;
        using I1 = std::integral_constant<int, 1>;
        read_pre(c + 1);
        read(I0{}, I0{});
        if constexpr (BOTH) read(I1{}, I1{});
        issue_w();
        wait_lgkmcnt<0>();
        pre_landed();
        frags_landed(I0{});
        if constexpr (BOTH) frags_landed(I1{});
        if constexpr (decltype(TAIL)::value) { if (c + 1 < nc) put_x(S, c + 1); } else put_x(S, c + 1);
        load_x(S, c + 1 + DX);
        contract(I0{});
        if constexpr (BOTH) {
            contract(I1{});
        } else {
            read(I1{}, I0{});
            wait_lgkmcnt<0>();
            frags_landed(I0{});
            contract(I0{});
        }
        rs = rs + 1 == NSW ? 0 : rs + 1;
    };
    // whole groups of DX iterations without a branch, so that the compiler can tell how many loads are outstanding where; the
    // last iterations behind them (put_x of chunk nc - 1 belongs to iteration nc - 2: the group loop stops short of nc - 1)
    int c = 0;
    for (; c + DX < nc; c += DX)
        static_for<DX>([&](auto S) { step(std::integral_constant<int, (decltype(S)::value + 1) % DX>{}, std::false_type{}, c + decltype(S)::value); });
    static_for<DX>([&](auto S) {
        if (c + decltype(S)::value < nc) step(std::integral_constant<int, (decltype(S)::value + 1) % DX>{}, std::true_type{}, c + decltype(S)::value);
    });
    // ---- t1: affine + ReLU in the accumulator layout (4 channels of one pixel per lane), rounded to bf16, over the chunk buffers
    wait_lgkmcnt<0>();
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int i = 0; i < CA; i++) {
        const int ch = (wca * CA + i) * 16 + lg * 4;
        u32x4_t s4, h4;
        lds_read16<0>(s4, lbase + AFF0 + ch * 4);
        lds_read16<DN_MID * 4>(h4, lbase + AFF0 + ch * 4);
        wait_lgkmcnt<0>();
        landed(s4);
        landed(h4);
#pragma unroll
        for (int j = 0; j < PA; j++) {
            const int row = (wpa * PA + j) * 16 + lr;
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; e++) v[e] = __builtin_fmaxf(acc[i][j][e] * __uint_as_float(s4[e]) + __uint_as_float(h4[e]), 0.f);
            u32x2_t o;
            o[0] = pack_bf16x2(v[0], v[1]);
            o[1] = pack_bf16x2(v[2], v[3]);
            lds_write8(lbase + row * 256 + (((ch >> 3) ^ (row & 15)) << 4) + ((ch & 4) << 1), o);
        }
    }

    // ---- phase B
    const int wpb = wave % WPB, kq = wave / WPB;
    unsigned val[NB];                                      // the taps of this lane's pixel of block b
    f32x4_t acc2[NB][2];
    {
        int m = wpb * NB * 16 + lr, p = min(p0 + m, P - 1);
        int w = p % W, h = (p / W) % d.H;
#pragma unroll
        for (int b = 0; b < NB; b++) {
            const unsigned cm = (w > 0 ? 1u : 0u) | 2u | (w + 1 < W ? 4u : 0u);
            val[b] = dense_taps(m, bp, cm, h > 0, h + 1 < d.H);
            m += 16;
            w += 16;
            while (w >= W) { w -= W; h = h + 1 == d.H ? 0 : h + 1; }
            acc2[b][0] = acc2[b][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
    }
    for (int j = 0; j < 5; j++) {
        wait_vmcnt<(NSW - 2) * 2>();
        wait_lgkmcnt<0>();
        __builtin_amdgcn_s_barrier();                      // stage nc + j has landed for every wave (j = 0: and t1 is written)
        issue_w();
        const unsigned wb = lbase + RING0 + rs * WST + lr * 256;
        constexpr int QG = NB <= 4 ? 2 : 1;                // k-steps whose fragments are requested together
#pragma unroll
        for (int q0 = 0; q0 < KPW; q0 += QG) {
            u32x4_t fa[QG][2], fb[QG][NB];
            static_for<QG>([&](auto Q) {
                constexpr int q = decltype(Q)::value;
                // the tenth tap of the last stage reads zeros of w2 and, as bit 9 is never set, the zero row: any pixel there
                // could be an infinity, and its product with zero a NaN
                const int ks = kq * KPW + q0 + q, t = 2 * j + (ks >> 2), tap = min(t, 8);
                const int r = tap / 3, s = tap - 3 * r, toff = r * W + s;
                const unsigned slot = (ks & 3) * 4 + lg, wa = wb + (ks >> 2) * 8192 + ((slot ^ lr) << 4);
                lds_read16<0>(fa[q][0], wa);
                lds_read16<4096>(fa[q][1], wa);
                // the pixel blocks of a wave lie 16 rows apart: one address (the slot permutation depends on row % 16), block b at
                // an immediate offset; lanes whose tap is padding go to the zero row instead
                const int row0 = wpb * NB * 16 + lr + toff;
                const unsigned at = lbase + row0 * 256 + ((slot ^ (row0 & 15)) << 4), zero = lbase + ZROW + (slot << 4), bit = 1u << t;
                static_for<NB>([&](auto B) {
                    constexpr int b = decltype(B)::value;
                    lds_read16<b * 4096>(fb[q][b], (val[b] & bit) ? at : zero - b * 4096);
                });
            });
            wait_lgkmcnt<0>();
            static_for<QG>([&](auto Q) {
                constexpr int q = decltype(Q)::value;
                landed(fa[q][0]);
                landed(fa[q][1]);
                static_for<NB>([&](auto B) { landed(fb[q][decltype(B)::value]); });
#pragma unroll
                for (int b = 0; b < NB; b++) {
                    Mma16<bf16_t>::run(acc2[b][0], fa[q][0], fb[q][b]);
                    Mma16<bf16_t>::run(acc2[b][1], fa[q][1], fb[q][b]);
                }
            });
        }
        rs = rs + 1 == NSW ? 0 : rs + 1;
    }
    wait_vmcnt<0>();
    wait_lgkmcnt<0>();
    __builtin_amdgcn_s_barrier();                          // t1 and the ring are dead: the partial sums take their place
    typedef float Block[4 * LSTR];
    Block *red = reinterpret_cast<Block *>(lds);           // [kq][16-pixel block][16-channel block]
#pragma unroll
    for (int b = 0; b < NB; b++)
#pragma unroll
        for (int i = 0; i < 2; i++)
            *reinterpret_cast<float4 *>(&red[(kq * WPB * NB + wpb * NB + b) * 2 + i][lg * LSTR + lr * 4]) =
                make_float4(acc2[b][i][0], acc2[b][i][1], acc2[b][i][2], acc2[b][i][3]);
    __syncthreads();
    const float *aff2 = reinterpret_cast<const float *>(lds + AFF0) + 2 * DN_MID;
    bf16_t *__restrict__ yg = static_cast<bf16_t *>(d.y);
    const float lim = d.act == SOL_ACT_RELU ? 0.f : __builtin_nanf("");
    for (int it = tid; it < bp * 4; it += 512) {           // 8 channels of one pixel
        const int m = it >> 2, g = it & 3, blk = (m >> 4) * 2 + (g >> 1), at = (g & 1) * 2 * LSTR + (m & 15) * 4;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; e++) v[e] = 0.f;
#pragma unroll
        for (int k = 0; k < KSB; k++) {
            const float4 lo = *reinterpret_cast<const float4 *>(&red[k * WPB * NB * 2 + blk][at]);
            const float4 hi = *reinterpret_cast<const float4 *>(&red[k * WPB * NB * 2 + blk][at + LSTR]);
            v[0] += lo.x; v[1] += lo.y; v[2] += lo.z; v[3] += lo.w;
            v[4] += hi.x; v[5] += hi.y; v[6] += hi.z; v[7] += hi.w;
        }
#pragma unroll
        for (int e = 0; e < 8; e++) v[e] = __builtin_fmaxf(v[e] * aff2[g * 8 + e] + aff2[DN_OUT + g * 8 + e], lim);
        store_vec8<bf16_t>(yg + (long)(p0 + m) * d.ldy + g * 8, v);
    }
#endif
}

template <int PA, int CA, int WPA, int KSB, int DX, int NSW>
sol_status launch_dense_cfg(const DenseLaunch &d, int bp, hipStream_t st) {
    DenseArgs a{d, bp, ceil_div(d.N * d.H * d.W, bp), d.C / 64};
    const int grid = ((a.ntiles + 7) / 8) * 8;
    hipLaunchKernelGGL((conv_dense_kernel<PA, CA, WPA, KSB, DX, NSW>), dim3(grid), dim3(512), 0, st, a);
    SOL_HIP(hipGetLastError());
    return SOL_OK;
}
// Patch rows of the variants, and the microseconds of one workgroup apart from the launch: base + chunk * (C / 64).  Fitted to
// 7x7 .. 56x56 images of 64 .. 992 channels; one image or 64, as long as the tiles do not outnumber the CUs.
struct DenseVariant { int rows; float base, chunk; };
constexpr DenseVariant kVariant[] = {{64, 3.5f, 0.39f}, {96, 4.0f, 0.60f}, {128, 5.1f, 0.61f}, {192, 5.7f, 0.83f}, {256, 6.6f, 1.08f}, {384, 9.1f, 1.51f}};
}  // namespace

// bf16, C input channels (rounded up to 64, at most 1024; what lies between is masked) -> 128 -> 32; 32-bit byte offsets; a patch that holds some pixels
// besides its halo
bool dense_kernel_applies(int dt, int N, int H, int W, int C, int ldx, int mid, int cout, int ldy) {
    return dt == SOL_BF16 && mid == DN_MID && cout == DN_OUT && C % 64 == 0 && C <= DN_CMAX && ldx % 8 == 0 && ldy % 8 == 0 && 2 * W + 2 + 16 <= 384 &&
           (double)N * H * W * ldx * 2 < 2147483648.0 && (double)N * H * W * ldy * 2 < 4294967296.0;
}

namespace {
// The variant and the rounds of the 256 CUs it takes.  variant >= 0: forced, the first one from there on that the width allows.
int choose_variant(int P, int W, int C, int variant, int *rounds) {
    // Larger patches recompute less of the halo (2 W + 2 rows per tile) and take longer each: the fewest rounds of the 256 CUs,
    // weighted with the time of a round.  (14x14, 640 channels, 64 images: 64 rows 21.0 us, 96 rows 14.2, 128 rows 15.3.)
    int v = -1;
    float best = 0.f;
    for (int i = 0; i < 6; i++) {
        const int px = kVariant[i].rows - 2 * W - 2;
        if (px < 16 && i < 5) continue;
        const int n = ceil_div(ceil_div(P, px), 256);
        const float t = (float)n * (kVariant[i].base + kVariant[i].chunk * (C / 64));
        if (v < 0 || t < best || (variant >= 0 && i >= variant)) { v = i; best = t; *rounds = n; }
        if (variant >= 0 && i >= variant) break;
    }
    return v;
}
}  // namespace

// A patch recomputes 2 W + 2 rows of the 1x1 convolution for its pixels, so wide images lose by one launch what it saves.  Two
// launches (the 1x1 convolution on conv_pre) -> one, us, launches and events included, 64 images: W = 56, C = 64: 66 -> 46; 88, 256:
// 216 -> 200; 88, 512: 278 -> 273; 104, 64: 224 -> 200; 104, 128: 256 -> 236; 104, 256: 291 -> 307; 104, 512: 378 -> 418; 112, 128: 299 -> 298;
// 112, 256: 333 -> 374; 112, 512: 433 -> 517.  The line is where the narrow prefixes, which images so wide have, cross; for wide ones it is
// up to 11 % late between 88 and 104, which the auto-tuner finds.  A prefix that ends inside
// a chunk of 64 channels costs the 1x1 convolution on its own about three times as much, and the line lies further out:
// 148, 96: 927 -> 921; 152, 96: 976 -> 1072; 144, 224: 1362 -> 1041; 160, 224: 1665 -> 1934; 16 images, 144, 992: 1151 -> 564; 176, 224: 530 -> 1138.  One round of
// workgroups is about as fast as two launches at any width (one image, 144, 64: 31 -> 25; 84, 64: 20 -> 22; only strips such as
// 2 x 130 pixels, 19 -> 25, are not, which the auto-tuner finds).
bool dense_one_launch_pays(int N, int H, int W, int C, bool masked) {
    int rounds = 1;
    choose_variant(N * H * W, W, C, -1, &rounds);
    return rounds <= 1 || W <= (masked ? 148 : 104);
}

sol_status launch_conv_dense(const DenseLaunch &d, int variant, hipStream_t st) {
    const int P = d.N * d.H * d.W;
    if (P <= 0) return SOL_OK;
    int rounds;
    const int v = choose_variant(P, d.W, d.C, variant, &rounds);
    int bp = kVariant[v].rows - 2 * d.W - 2;
    const int nt = ceil_div(P, bp);
    bp = min(bp, (int)round_up(ceil_div(P, nt), 4));       // equal shares
    switch (v) {
        //                               PA CA WPA KSB DX NSW
        case 0: return launch_dense_cfg<2, 2, 2, 4, 4, 4>(d, bp, st);
        case 1: return launch_dense_cfg<3, 2, 2, 4, 4, 4>(d, bp, st);
        case 2: return launch_dense_cfg<4, 2, 2, 4, 4, 4>(d, bp, st);
        case 3: return launch_dense_cfg<3, 4, 4, 2, 2, 3>(d, bp, st);
        case 4: return launch_dense_cfg<4, 4, 4, 2, 2, 3>(d, bp, st);
        default: return launch_dense_cfg<6, 4, 4, 2, 2, 3>(d, bp, st);
    }
}

}  // namespace sol

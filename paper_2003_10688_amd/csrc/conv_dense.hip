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
//    buffers); w1 chunks (128 rows x 128 B) travel by LDS DMA through a ring of NSW stages of 16 KB, DW in flight.  One barrier per chunk.
//  t1 takes the place of the two chunk buffers (PR rows x 256 B, rounded to bf16 where the layer-by-layer path stores it).
//  Phase B runs the nine taps from that patch (row of pixel m, tap (r, s): m + r * W + s; taps outside the image are redirected
//    to a zero row); w2 continues in the same ring, two taps to a stage.  With five stages, which all but the largest patch leave room
//    for, all of w2 has been asked for when t1 is written, and the taps run without a barrier.  The waves split the reduction
//    KSB ways, and the partial sums meet in LDS in a fixed order.
// What bounds it: two waves per SIMD that meet at a barrier once per chunk issue one instruction in about nine cycles each, whatever its
// kind, so a chunk costs what it has of instructions, and what runs beside one another inside a wave.  Against a version that ran a
// chunk's fragment reads, BN + ReLU and MFMAs one behind the other, chose each stage's matrix anew, tested each tap of each lane
// and waited for everything at the start: DenseNet-121-shaped pass, batch 64, 1250 -> 1093 us (another card 1262 -> 1121); one layer, 64 images, us, that version ->
// this: 56x56, 64 / 192 channels 44 / 60 -> 37 / 52; 28x28, 128 / 480: 15.4 / 22 -> 11 / 18; 14x14, 256 / 640: 11 / 14 -> 8.2 / 12; 7x7, 512 / 992: 10 / 13 -> 8.1 /
// 11.  Cycles of a tile of 96 rows, 640 channels: start 5600 -> 4800, phase A 1410 -> 1210 a chunk (products alone 384, BN + ReLU alone
// 500, LDS 650), t1 1050 -> 1400, phase B 6500 -> 3400 (products 1730), sums and output 2000 -> 2200.  Without effect there: constants of two
// chunks in registers, fragments of phase B three steps ahead instead of two, padding taps on bank-neutral zeros.
// All LDS accesses between DMAs are opaque statements (the compiler would make each of them wait for every DMA in flight).
#include "conv_common.h"

namespace sol {

namespace {
using lds_pipe::u32x4_t;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2_t;

template <int O> __device__ __forceinline__ void lds_write16(unsigned addr, const u32x4_t &v) {
    asm volatile("ds_write_b128 %0, %1 offset:%2" ::"v"(addr), "v"(v), "n"(O) : "memory");
}
__device__ __forceinline__ void lds_write4(unsigned addr, float v) { asm volatile("ds_write_b32 %0, %1" ::"v"(addr), "v"(v) : "memory"); }
__device__ __forceinline__ void lds_read4(unsigned &dst, unsigned addr) { asm volatile("ds_read_b32 %0, %1" : "=&v"(dst) : "v"(addr)); }
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
    FastDiv dw, dh;            // image width, height
};

// PA x CA: 16-pixel x 16-channel blocks of t1 per wave; WPA x (8 / WPA): wave grid of phase A; KSB: reduction split of phase B
// (the other 8 / KSB waves split the pixels); DX: x chunks in flight in registers; NSW: weight ring stages; DW: those in flight in phase A
template <int PA, int CA, int WPA, int KSB, int DX, int NSW, int DW>
__global__ void __launch_bounds__(512) conv_dense_kernel(const DenseArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
    using namespace lds_pipe;
    constexpr int WCA = 8 / WPA, PR = WPA * PA * 16, WPB = 8 / KSB, NB = PR / 16 / WPB;
    static_assert(WCA * CA * 16 == DN_MID && PR / 16 % WPB == 0, "wave grids");
    constexpr int XR = (PR * 8 + 511) / 512;               // 16-byte pieces of an x chunk per thread
    constexpr int WST = 16384, LSTR = 68;
    constexpr int CB = XR * 8192;                          // a chunk buffer: rows behind the patch are written and never read
    constexpr int TB = 2 * CB > PR * 256 ? 2 * CB : PR * 256, ZROW = TB, RING0 = TB + 256, PRE0 = RING0 + NSW * WST, AFF0 = PRE0 + 2 * DN_CMAX * 4, VAL0 = AFF0 + 2 * (DN_MID + DN_OUT) * 4, LDSB = VAL0 + 512 * 4;
    static_assert(LDSB <= 160 * 1024 && KSB * WPB * NB * 2 * 4 * LSTR * 4 <= PRE0, "LDS");
    static_assert((DW + 1) * (XR + 2) < 60 && (DX + 1) * (XR + 2) < 60 && DX % 2 == 0 && DW <= DX && DW < NSW, "vmcnt, chunk parity, prologue order");
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
    // A wave brings two KB of it, 8 (4) rows of 8 (16) slots each.  The second KB lies 8 (4) rows on, where the slot permutation differs in one bit.
    const int r1 = wave * 16 + (lane >> 3), r2 = (wave & 3) * 8 + (lane >> 4);
    unsigned wo = (unsigned)(r1 * d.Kp1) * 2 + (((lane & 7) ^ swz<128>(r1)) << 4), whalf = (unsigned)d.Kp1 * 16;
    const unsigned wo2 = (unsigned)(r2 * 9 * DN_MID) * 2 + (wave >> 2) * 256 + (((lane & 15) ^ (r2 & 15)) << 4);
    // The next stage: matrix, offset in it, slot.  (The tenth tap of the last stage is the next filter's first, zeros behind the last filter;
    // nobody reads it.)  (Chosen anew from the number of the stage, with a bound of its own, this was 40 scalar instructions a chunk of 130 all told.)
    int wleft = nc, wslot = RING0 + wave * 2048;           // stages of w1 still to come; LDS offset of this wave's share
    unsigned wso = 0, wby = 128, wbytes = w1bytes;
    const void *wsrc = d.w1;
    auto issue_w_half = [&](auto I) __attribute__((always_inline)) {        // half i of the next stage
        constexpr int i = decltype(I)::value;
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(wsrc), 0, (int)wbytes, 0x00020000);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)(lds + wslot + i * 1024), 16, i == 0 ? wo : (wo ^ 64u) + whalf, wso, 0, 0);
        if constexpr (i == 1) {
            wslot = wslot + WST == RING0 + wave * 2048 + NSW * WST ? RING0 + wave * 2048 : wslot + WST;
            wso += wby;
            const bool turn = --wleft == 0;                // w2 from here on
            wsrc = turn ? d.w2 : wsrc;
            wso = turn ? 0 : wso;
            wby = turn ? 512 : wby;
            wbytes = turn ? w2bytes : wbytes;
            wo = turn ? wo2 : wo;
            whalf = turn ? 4 * 9 * DN_MID * 2 : whalf;
        }
    };
    auto issue_w = [&]() __attribute__((always_inline)) {
        issue_w_half(std::integral_constant<int, 0>{});
        issue_w_half(std::integral_constant<int, 1>{});
    };
    // ---- x rows: piece i of this thread = 16-byte slot (tid & 7) of patch row (tid >> 3) + 64 * i
    const int xslot = tid & 7;
    // byte offset of piece 0 in x; rows outside x wrap or run past its end, where the buffer's own check returns zeros (nothing reads
    // what becomes of them: their taps are padding).  The other pieces' offsets are added up at each load and not kept in registers,
    // but for the last one of a patch that ends inside its 64 rows.
    const unsigned xo = (unsigned)((p0 - W - 1 + (tid >> 3)) * d.ldx) * 2 + (xslot << 4), xstep = (unsigned)d.ldx * 128;
    const unsigned xo_last = (tid >> 3) + 64 * (XR - 1) < PR ? xo + (XR - 1) * xstep : 0xffffffffu;
    // LDS offset of piece 0 inside a chunk buffer; piece i lies 64 rows on, where the slot permutation is the same: an immediate
    // offset (an address per piece took the 384-row variant over 256 registers)
    const unsigned xl = (unsigned)(tid >> 3) * 128 + ((xslot ^ swz<128>(tid >> 3)) << 4);
    u32x4_t xv[DX][XR];
    auto load_piece = [&](auto S, auto I, int c) __attribute__((always_inline)) {
        constexpr int s = decltype(S)::value, i = decltype(I)::value;
        unsigned by = __builtin_amdgcn_readfirstlane(xstep);
        asm volatile("" : "+s"(by));                       // not an invariant of the loop, to the compiler
        const unsigned off = XR * 64 != PR && i == XR - 1 ? xo_last : xo + i * by;
        xv[s][i] = __builtin_amdgcn_raw_buffer_load_b128(xr, off, (unsigned)min(c, nc - 1) * 128u, 0);
    };
    auto load_x = [&](auto S, int c) __attribute__((always_inline)) { static_for<XR>([&](auto I) { load_piece(S, I, c); }); };
    // input-side constants of this thread's eight channels of the next chunk to go to LDS; fetched one iteration ahead
    u32x4_t q[4];
    auto read_pre = [&](int c) __attribute__((always_inline)) {
        const unsigned pa = lbase + PRE0 + (unsigned)(min(c, nc - 1) * 64 + xslot * 8) * 4;
        lds_read16<0>(q[0], pa);
        lds_read16<16>(q[1], pa);
        lds_read16<DN_CMAX * 4>(q[2], pa);
        lds_read16<DN_CMAX * 4 + 16>(q[3], pa);
    };
    auto pre_landed = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; e++) landed(q[e]);
    };
    // piece i of relu(scale * x + shift) of chunk c from register set S into chunk buffer c & 1
    auto put_piece = [&](auto S, auto I, auto PAR) __attribute__((always_inline)) {          // PAR = c & 1
        constexpr int s = decltype(S)::value, i = decltype(I)::value;
        u32x4_t o;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const unsigned u = xv[s][i][e];
            const float lo = __uint_as_float(u << 16), hi = __uint_as_float(u & 0xffff0000u);
            const float a0 = lo * __uint_as_float(q[e >> 1][(e & 1) * 2]) + __uint_as_float(q[2 + (e >> 1)][(e & 1) * 2]);
            const float a1 = hi * __uint_as_float(q[e >> 1][(e & 1) * 2 + 1]) + __uint_as_float(q[2 + (e >> 1)][(e & 1) * 2 + 1]);
            o[e] = pack_bf16x2(__builtin_fmaxf(a0, 0.f), __builtin_fmaxf(a1, 0.f));
        }
        constexpr int at = decltype(PAR)::value * CB + i * 8192, far = at < 65536 ? 0 : CB;      // 16-bit offsets
        lds_write16<at - far>(lbase + xl + far, o);
    };

    const int wpb = wave % WPB, kq = wave / WPB;           // of phase B
    // ---- prologue.  Everything is asked for in the order in which it is needed and waited for by count: the per-channel constants, then
    // x chunk v and weight stage v in turn.
    {
        const int c0 = min(tid, d.Cvalid - 1), c1 = min(tid + 512, d.Cvalid - 1);
        float v[8] = {d.ps[c0], d.ph[c0], d.ps[c1], d.ph[c1], d.s1[tid & 127], d.h1[tid & 127], d.s2[tid & 31], d.h2[tid & 31]};
        keep_order();
        static_for<DX>([&](auto S) {
            load_x(S, decltype(S)::value);
            if constexpr (decltype(S)::value < DW) issue_w();
            keep_order();
        });
        // meanwhile, for phase B: bits 5 b .. 5 b + 4 of val say which of the taps (0, 1), (1, 0), (1, 1), (1, 2), (2, 1) this lane's pixel of block b
        // has; the corner taps are there where both of their neighbours are.  It waits in LDS: the largest patch has no register for it.
        static_assert(NB * 5 <= 32, "bits");
        unsigned val = 0;
#pragma unroll
        for (int b = 0; b < NB; b++) {
            const int m = (wpb * NB + b) * 16 + lr;
            uint32_t row, w, n, h;
            a.dw.divmod((uint32_t)min(p0 + m, P - 1), row, w);
            a.dh.divmod(row, n, h);
            const unsigned t = dense_taps(m, bp, (w > 0 ? 1u : 0u) | 2u | ((int)w + 1 < W ? 4u : 0u), h > 0, (int)h + 1 < d.H);
            val |= ((t >> 1 & 1u) | (t >> 2 & 14u) | (t >> 3 & 16u)) << (5 * b);
        }
        lds_write4(lbase + VAL0 + tid * 4, __uint_as_float(val));
        // zeros behind the prefix: max(0 * x + 0, 0) is 0 whatever lies there (of a NaN and 0 the maximum is 0)
        const bool in0 = tid < d.Cvalid, in1 = tid + 512 < d.Cvalid;
        wait_vmcnt<DX * XR + DW * 2>();
#pragma unroll
        for (int e = 0; e < 8; e++) asm volatile("" : "+v"(v[e]));
        lds_write4(lbase + PRE0 + tid * 4, in0 ? v[0] : 0.f);
        lds_write4(lbase + PRE0 + DN_CMAX * 4 + tid * 4, in0 ? v[1] : 0.f);
        lds_write4(lbase + PRE0 + 2048 + tid * 4, in1 ? v[2] : 0.f);
        lds_write4(lbase + PRE0 + DN_CMAX * 4 + 2048 + tid * 4, in1 ? v[3] : 0.f);
        // scale / shift of the two convolutions, behind one another; threads that share a channel write the same value
        lds_write4(lbase + AFF0 + (tid & 127) * 4, v[4]);
        lds_write4(lbase + AFF0 + DN_MID * 4 + (tid & 127) * 4, v[5]);
        lds_write4(lbase + AFF0 + 2 * DN_MID * 4 + (tid & 31) * 4, v[6]);
        lds_write4(lbase + AFF0 + (2 * DN_MID + DN_OUT) * 4 + (tid & 31) * 4, v[7]);
        lds_write4(lbase + ZROW + lane * 4, 0.f);
    }
    wait_lgkmcnt<0>();
    __builtin_amdgcn_s_barrier();

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
    static_for<XR>([&](auto I) { put_piece(std::integral_constant<int, 0>{}, I, std::integral_constant<int, 0>{}); });
    load_x(std::integral_constant<int, 0>{}, DX);
    read_pre(1);
    wait_lgkmcnt<0>();
    pre_landed();
    // ---- phase A.  A chunk is U units: k-step u / NH, the pixel blocks of part u % NH.  While the fragments of unit u travel from
    // LDS, the matrix pipe has unit u - 1 and the vector units have a share of BN + ReLU of the next chunk: iteration c starts with the
    // last unit of chunk c - 1, transforms chunk c + 1 from register set S and refills that set.
    // (Opaque LDS reads are always waited for before the next branch: a register they have yet to fill must not be copied.)
    constexpr int NH = PA * CA > 16 ? PA / 2 : 1, PH = PA / NH, U = 2 * NH;
    static_assert(PH * NH == PA, "parts");
    u32x4_t fa[2][CA], fb[2][PH];
#pragma unroll
    for (int i = 0; i < CA; i++) fa[1][i] = u32x4_t{0u, 0u, 0u, 0u};       // in front of the first chunk: products of zeros
#pragma unroll
    for (int j = 0; j < PH; j++) fb[1][j] = u32x4_t{0u, 0u, 0u, 0u};
    auto contract = [&](auto UU) __attribute__((always_inline)) {
        constexpr int u = decltype(UU)::value, k = u / NH, h = u % NH;
#pragma unroll
        for (int i = 0; i < CA; i++)
#pragma unroll
            for (int j = 0; j < PH; j++) Mma16<bf16_t>::run(acc[i][h * PH + j], fa[k][i], fb[u & 1][j]);
    };
    int rs = 0;                                            // ring slot of the current stage
    // S: register set of chunk c + 1.  T: -1 inside the loop; t for the t-th step behind it, which asks for no more x; DX - 1 for the last
    // chunk's, which may be any of those.
    auto step = [&](auto S, auto T, int c) __attribute__((always_inline)) {
        constexpr bool last = decltype(T)::value == DX - 1, loads = decltype(T)::value < 0;
        // Weight stage c has landed once only what was issued after it is outstanding: what step c - DW asked for behind the stage's second half (x
        // pieces but those of its first unit) and all of the DW - 1 steps since, of which t asked for weights alone.  (The prologue
        // asked for more.)  Counted is what is in the program: a load whose registers nothing read would be taken out by the compiler, so none is written.
        constexpr int t = decltype(T)::value < 0 ? 0 : decltype(T)::value, x_behind = t < DW ? (DW - t) * XR - (XR + U - 1) / U : 0;
        wait_vmcnt<x_behind + (DW - 1) * 2>();
        __builtin_amdgcn_s_barrier();                      // ... for every wave; chunk c is in LDS; nobody still reads chunk c - 1
        // chunk c lies in buffer c & 1 = 1 - S & 1 (DX is even): an immediate offset, but for the last chunk
        constexpr int par = last ? 0 : (decltype(S)::value + 1) & 1;
        const unsigned xb = last ? fx + (c & 1) * CB : fx, wb = fw + rs * WST;
        static_for<U>([&](auto I) {
            constexpr int u = decltype(I)::value, k = u / NH, h = u % NH;
            if constexpr (h == 0) static_for<CA>([&](auto J) { lds_read16<decltype(J)::value * 2048>(fa[k][decltype(J)::value], wb ^ (k * 64)); });
            static_for<PH>([&](auto J) { lds_read16<par * CB + (h * PH + decltype(J)::value) * 2048>(fb[u & 1][decltype(J)::value], xb ^ (k * 64)); });
            __builtin_amdgcn_sched_barrier(0);             // the requests first
            contract(std::integral_constant<int, (u + U - 1) % U>{});
            constexpr int first = (u * XR + U - 1) / U, end = ((u + 1) * XR + U - 1) / U;      // pieces i with i * U / XR == u
            if constexpr (!last) static_for<end - first>([&](auto J) { put_piece(S, std::integral_constant<int, first + decltype(J)::value>{}, std::integral_constant<int, 1 - par>{}); });
            if constexpr (!last)                           // products and transforms in turn: both pipes of a SIMD have work
                static_for<CA * PH>([](auto) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, (28 * (end - first) + CA * PH - 1) / (CA * PH) + 1, 0);
                });
            if constexpr (u < 2) issue_w_half(I);
            keep_order();                                  // the count above
            if constexpr (last && u == 1) {                // the slots of all chunks but this one are free
#pragma unroll
                for (int e = DW + 1; e < NSW; e++) issue_w();
            }
            if constexpr (loads) static_for<end - first>([&](auto J) { load_piece(S, std::integral_constant<int, first + decltype(J)::value>{}, c + 1 + DX); });
            keep_order();
            if constexpr (u + 1 < U) {
                wait_lgkmcnt<last ? 0 : end - first>();
            } else {
                if constexpr (!last) read_pre(c + 2);
                wait_lgkmcnt<0>();
                if constexpr (!last) pre_landed();
            }
            if constexpr (h == 0) static_for<CA>([&](auto J) { landed(fa[k][decltype(J)::value]); });
            static_for<PH>([&](auto J) { landed(fb[u & 1][decltype(J)::value]); });
            __builtin_amdgcn_sched_barrier(0);
        });
        rs = rs + 1 == NSW ? 0 : rs + 1;
    };
    // whole groups of DX iterations without a branch, so that the compiler can tell how many loads are outstanding where
    int c = 0;
    for (; c + DX < nc; c += DX)
        static_for<DX>([&](auto S) { step(std::integral_constant<int, (decltype(S)::value + 1) % DX>{}, std::integral_constant<int, -1>{}, c + decltype(S)::value); });
    static_for<DX - 1>([&](auto S) {
        if (c + decltype(S)::value + 1 < nc) step(std::integral_constant<int, (decltype(S)::value + 1) % DX>{}, S, c + decltype(S)::value);
    });
    step(std::integral_constant<int, 0>{}, std::integral_constant<int, DX - 1>{}, nc - 1);
    contract(std::integral_constant<int, U - 1>{});
    // what the rest needs of the thread's number is computed again: kept over the loop it is two registers too many for the largest patch
    int tid2 = tid;
    asm volatile("" : "+v"(tid2));
    const int lane2 = tid2 & 63, lr2 = lane2 & 15, lg2 = lane2 >> 4;
    // ---- t1: affine + ReLU in the accumulator layout (4 channels of one pixel per lane), rounded to bf16, over the chunk buffers
    __builtin_amdgcn_s_barrier();                          // the chunk buffers and the last chunk's weights are dead
    issue_w();
#pragma unroll
    for (int i = 0; i < CA; i++) {
        const int ch = (wca * CA + i) * 16 + lg2 * 4;
        u32x4_t s4, h4;
        lds_read16<0>(s4, lbase + AFF0 + ch * 4);
        lds_read16<DN_MID * 4>(h4, lbase + AFF0 + ch * 4);
        wait_lgkmcnt<0>();
        landed(s4);
        landed(h4);
#pragma unroll
        for (int j = 0; j < PA; j++) {
            const int row = (wpa * PA + j) * 16 + lr2;
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
    unsigned val;
    lds_read4(val, lbase + VAL0 + tid2 * 4);
    wait_lgkmcnt<0>();
    asm volatile("" : "+v"(val));
    // lanes whose pixel of block b has the tap: the middle one, its row's left and right ones, its column's upper and lower ones
    unsigned long long mid[NB], left[NB], right[NB], up[NB], down[NB];
    f32x4_t acc2[NB][2];
#pragma unroll
    for (int b = 0; b < NB; b++) {
        up[b] = __builtin_amdgcn_ballot_w64(val >> (5 * b) & 1);
        left[b] = __builtin_amdgcn_ballot_w64(val >> (5 * b + 1) & 1);
        mid[b] = __builtin_amdgcn_ballot_w64(val >> (5 * b + 2) & 1);
        right[b] = __builtin_amdgcn_ballot_w64(val >> (5 * b + 3) & 1);
        down[b] = __builtin_amdgcn_ballot_w64(val >> (5 * b + 4) & 1);
        acc2[b][0] = acc2[b][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    // The pixel blocks of a wave lie 16 rows apart: one address (the slot permutation depends on row % 16), block b at an immediate
    // offset; lanes whose tap is padding go to the zero row instead.  What bounded this loop was the arithmetic of its addresses (a lane's
    // validity in one register, tested for each tap: 25 VALU instructions for 5 reads and 6 MFMAs, 4700 of the 27000 cycles of a 96-row tile).
    unsigned zrow[NB];
#pragma unroll
    for (int b = 0; b < NB; b++) zrow[b] = lbase + ZROW + (lane2 & 15) * 16 - b * 4096;
    // taps T0 .. T1 - 1, KQ of the four k-steps of each: the fragments of two steps travel under the products of the step before
    constexpr int KQ = 4 / KSB;
    const unsigned wl = lbase + RING0 + lr2 * 256 + (((kq * KQ * 4 + lg2) ^ lr2) << 4);
    auto taps = [&](auto T0, auto T1, unsigned r0) __attribute__((always_inline)) {       // r0: ring slot of tap T0
        constexpr int t0 = decltype(T0)::value, n = (decltype(T1)::value - t0) * KQ;
        constexpr int DB = 3;                              // steps in flight
        u32x4_t ga[DB][2], gb[DB][NB];
        auto read = [&](auto V) __attribute__((always_inline)) {
            constexpr int v = decltype(V)::value, t = t0 + v / KQ, r = t / 3, s = t % 3, flip = v % KQ * 64;
            unsigned rn = r0 + (t / 2 - t0 / 2);
            rn = rn >= NSW ? rn - NSW : rn;
            const unsigned wa = (wl ^ flip) + rn * WST;
            lds_read16<(t & 1) * 8192>(ga[v % DB][0], wa);
            lds_read16<(t & 1) * 8192 + 4096>(ga[v % DB][1], wa);
            const unsigned row0 = wpb * NB * 16 + lr2 + r * W + s, slot = (kq * KQ * 4 + lg2) ^ (row0 & 15);
            const unsigned at = lbase + (row0 << 8) + ((slot << 4) ^ flip);
            static_for<NB>([&](auto B) {
                constexpr int b = decltype(B)::value;
                const unsigned long long ok = (r == 0 ? up[b] : r == 2 ? down[b] : mid[b]) & (s == 0 ? left[b] : s == 2 ? right[b] : mid[b]);
                lds_read16<b * 4096>(gb[v % DB][b], __builtin_amdgcn_inverse_ballot_w64(ok) ? at : zrow[b]);
            });
        };
        static_for<DB - 1>([&](auto V) { if constexpr (decltype(V)::value < n) read(V); });
        static_for<n>([&](auto V) {
            constexpr int v = decltype(V)::value, left = n - 1 - v < DB - 1 ? n - 1 - v : DB - 1;
            if constexpr (v + DB - 1 < n) read(std::integral_constant<int, v + DB - 1>{});
            wait_lgkmcnt<(left * (2 + NB) < 15 ? left * (2 + NB) : 15)>();
            landed(ga[v % DB][0]);
            landed(ga[v % DB][1]);
            static_for<NB>([&](auto B) { landed(gb[v % DB][decltype(B)::value]); });
#pragma unroll
            for (int b = 0; b < NB; b++) {
                Mma16<bf16_t>::run(acc2[b][0], ga[v % DB][0], gb[v % DB][b]);
                Mma16<bf16_t>::run(acc2[b][1], ga[v % DB][1], gb[v % DB][b]);
            }
        });
    };
    auto stage_landed = [&](auto N) {
        wait_vmcnt<decltype(N)::value>();
        wait_lgkmcnt<0>();
        __builtin_amdgcn_s_barrier();
    };
    if constexpr (NSW == 5) {                              // all of w2 lies in the ring; its last stage was asked for last
        stage_landed(std::integral_constant<int, 2>{});
        taps(std::integral_constant<int, 0>{}, std::integral_constant<int, 8>{}, rs);
        stage_landed(std::integral_constant<int, 0>{});
        taps(std::integral_constant<int, 8>{}, std::integral_constant<int, 9>{}, rs + 4 >= NSW ? rs + 4 - NSW : rs + 4);
    } else {
        static_assert(NSW == 5 || NSW == 3, "stages in flight");
        static_for<5>([&](auto J) {
            constexpr int j = decltype(J)::value;
            stage_landed(std::integral_constant<int, (j == 0 ? 2 : j < 4 ? 1 : 0) * 2>{});
            if constexpr (j > 0 && j < 3) issue_w();       // to where stage j - 1 was
            taps(std::integral_constant<int, 2 * j>{}, std::integral_constant<int, j < 4 ? 2 * j + 2 : 9>{}, rs);
            rs = rs + 1 == NSW ? 0 : rs + 1;
        });
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
            *reinterpret_cast<float4 *>(&red[(kq * WPB * NB + wpb * NB + b) * 2 + i][lg2 * LSTR + lr2 * 4]) =
                make_float4(acc2[b][i][0], acc2[b][i][1], acc2[b][i][2], acc2[b][i][3]);
    __syncthreads();
    const float *aff2 = reinterpret_cast<const float *>(lds + AFF0) + 2 * DN_MID;
    bf16_t *__restrict__ yg = static_cast<bf16_t *>(d.y);
    const float lim = d.act == SOL_ACT_RELU ? 0.f : __builtin_nanf("");
    for (int it = tid2; it < bp * 4; it += 512) {           // 8 channels of one pixel
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

template <int PA, int CA, int WPA, int KSB, int DX, int NSW, int DW>
sol_status launch_dense_cfg(const DenseLaunch &d, int bp, hipStream_t st) {
    DenseArgs a{d, bp, ceil_div(d.N * d.H * d.W, bp), d.C / 64, FastDiv((uint32_t)d.W), FastDiv((uint32_t)d.H)};
    const int grid = ((a.ntiles + 7) / 8) * 8;
    hipLaunchKernelGGL((conv_dense_kernel<PA, CA, WPA, KSB, DX, NSW, DW>), dim3(grid), dim3(512), 0, st, a);
    SOL_HIP(hipGetLastError());
    return SOL_OK;
}
// Patch rows of the variants, and the microseconds of one workgroup apart from the launch: base + chunk * (C / 64).  Fitted to
// 7x7 .. 56x56 images of 64 .. 992 channels; one image or 64, as long as the tiles do not outnumber the CUs.
struct DenseVariant { int rows; float base, chunk; };
constexpr DenseVariant kVariant[] = {{64, 3.5f, 0.40f}, {96, 4.3f, 0.52f}, {128, 5.0f, 0.55f}, {192, 5.6f, 0.73f}, {256, 6.8f, 0.95f}, {384, 10.1f, 1.30f}};
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
    // weighted with the time of a round.  (14x14, 640 channels, 64 images: 64 rows 17.4 us, 96 rows 11.9, 128 rows 12.6.)
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
// launches (the 1x1 convolution on conv_pre) -> one, us, launches and events included, 64 images: W = 56, C = 64: 62 -> 40; 88, 256:
// 219 -> 175; 88, 512: 283 -> 249; 104, 64: 220 -> 181; 104, 128: 251 -> 211; 104, 256: 297 -> 269; 104, 512: 384 -> 370; 112, 128: 294 -> 267;
// 112, 256: 341 -> 334; 112, 512: 438 -> 459; 128, 64: 335 -> 362; 128, 512: 561 -> 730.  The line lies where no prefix loses; the narrow ones
// between 104 and 112 the auto-tuner finds.  A prefix that ends inside
// a chunk of 64 channels costs the 1x1 convolution on its own about three times as much, and the line lies further out:
// 144, 224: 1372 -> 917; 160, 224: 1673 -> 1674; 176, 224: 2015 -> 3972; 4 images, 144, 992: 336 -> 144; 160, 992: 424 -> 239.  One round of
// workgroups is about as fast as two launches at any width (one image, 144, 64: 29 -> 21; 84, 64: 17 -> 17; only strips such as
// 2 x 130 pixels, 12 -> 19, are not, which the auto-tuner finds).
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
        //                               PA CA WPA KSB DX NSW DW
        case 0: return launch_dense_cfg<2, 2, 2, 4, 4, 5, 3>(d, bp, st);
        case 1: return launch_dense_cfg<3, 2, 2, 4, 4, 5, 3>(d, bp, st);
        case 2: return launch_dense_cfg<4, 2, 2, 4, 4, 5, 3>(d, bp, st);
        case 3: return launch_dense_cfg<3, 4, 4, 2, 2, 5, 2>(d, bp, st);
        case 4: return launch_dense_cfg<4, 4, 4, 2, 2, 5, 2>(d, bp, st);
        default: return launch_dense_cfg<6, 4, 4, 2, 2, 3, 2>(d, bp, st);
    }
}

}  // namespace sol

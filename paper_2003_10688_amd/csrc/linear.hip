// Linear layer for small batches:  y[m][o] = act( scale[o] * sum_i x[m][i] w[o][i] + shift[o] + res[m][o] ).
//
// With a batch of a few dozen rows the GEMM has one or two pixel tiles, so the convolution kernels, which
// parallelise over output tiles, leave most of the chip idle and walk the whole reduction in one workgroup.
// Here a workgroup owns 32 rows x 32 output features and its eight waves split the reduction between them;
// MFMA fragments (16 bytes of consecutive reduction elements of one row) are loaded straight from global
// memory into registers, sixteen steps in flight per wave (the kernel is latency-bound: for 2048 inputs that is
// the whole reduction in one round trip) -- x is tiny and
// L2-resident -- and the eight partial accumulators are added through LDS in a fixed order behind one barrier.
#include "conv_common.h"

namespace sol {

template <typename T>
__global__ void __launch_bounds__(512) linear_kernel(const ConvArgs a) {
    constexpr int EPC = 16 / (int)sizeof(T);       // reduction elements per fragment
    constexpr int UN = 16, NWV = 8;                // k-steps in flight per wave; waves per workgroup
    __shared__ float red[NWV][32][33];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 31, lh = lane >> 5;
    const int n0 = blockIdx.x * 32, m0 = blockIdx.y * 32;
    const int M = a.P, K = a.C, N = a.Cout;
    const T *__restrict__ xg = static_cast<const T *>(a.x);
    const T *__restrict__ wg = static_cast<const T *>(a.w);

    const bool wok = n0 + lr < N, xok = m0 + lr < M;
    const T *wp = wg + (size_t)(wok ? n0 + lr : 0) * a.Kp;
    const T *xp = xg + (size_t)(xok ? m0 + lr : 0) * K;
    const uint4 zero = make_uint4(0, 0, 0, 0);

    f32x16_t acc;
#pragma unroll
    for (int e = 0; e < 16; e++) acc[e] = 0.f;

    const int nsteps = (K + 2 * EPC - 1) / (2 * EPC);   // one step = 2*EPC reduction elements (both lane halves); K % EPC == 0
    for (int s0 = wave * UN; s0 < nsteps; s0 += NWV * UN) {
        // Every lane loads every step, from a clamped address (the start of a valid row), and what it must not use is
        // replaced by zeros after the last load is issued: a load behind a condition, or a use of its value between
        // the loads, makes the compiler wait for it before it issues the next one.
        uint4 fa[UN], fb[UN];
        auto k_of = [&](int u) { return (s0 + u) * 2 * EPC + lh * EPC; };   // < K, or: past the end / ragged last step
#pragma unroll
        for (int u = 0; u < UN; u++) {
            const int k = k_of(u), kk = k < K ? k : 0;
            fa[u] = *reinterpret_cast<const uint4 *>(wp + kk);
            fb[u] = *reinterpret_cast<const uint4 *>(xp + kk);
        }
        __builtin_amdgcn_sched_barrier(0);             // all 2 * UN loads are in flight before the first value is needed
#pragma unroll
        for (int u = 0; u < UN; u++) {
            const bool ok = k_of(u) < K;
            Mma<T>::run(acc, (ok && wok) ? fa[u] : zero, (ok && xok) ? fb[u] : zero);
        }
    }

    // accumulator register e of lane l: feature 8*(e/4) + 4*(l/32) + e%4, row l%32.  Every wave parks its partial
    // block, then each of the first 256 threads adds the eight partials of 4 outputs in wave order.
#pragma unroll
    for (int e = 0; e < 16; e++) red[wave][lr][8 * (e / 4) + 4 * lh + e % 4] = acc[e];
    __syncthreads();

    if (tid >= 256) return;
    const int row = tid >> 3, f0 = (tid & 7) * 4;
    const int m = m0 + row;
    if (m >= M) return;
    T *__restrict__ yg = static_cast<T *>(a.y);
    const T *__restrict__ resg = static_cast<const T *>(a.res);
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const int o = n0 + f0 + e;
        if (o >= N) break;
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < NWV; w++) t += red[w][row][f0 + e];
        t = t * (a.scale ? a.scale[o] : 1.f) + (a.shift ? a.shift[o] : 0.f);
        if (resg) t += Elem<T>::load(resg + (size_t)m * N + o);
        if (a.act == SOL_ACT_RELU) t = __builtin_fmaxf(t, 0.f);
        Elem<T>::store(yg + (size_t)m * a.ldy + o, t);
    }
}

// unpadded 1x1 "convolution" over a [rows,1,1,C] tensor with few rows, rows a whole number of 16-byte fragments.  The
// kernel reads x as P dense rows: with padding a [n,1,1,C] input has more output pixels than input rows (the padding
// pixels hold act(shift + residual)), which the gather kernels handle.
bool linear_kernel_applies(const ConvArgs &a, int dt) {
    const int frag = 16 / (int)dtype_size(dt);     // a fragment is 16 bytes of one row: rows must be whole fragments
    return a.R == 1 && a.S == 1 && a.H == 1 && a.W == 1 && a.ph == 0 && a.pw == 0 && a.Ho == 1 && a.Wo == 1 && a.P == a.N &&
           a.pool == 0 && a.P <= 1024 && a.C % frag == 0;
}

sol_status launch_linear(const ConvArgs &a, int dt, hipStream_t st) {
    const dim3 grid(ceil_div(a.Cout, 32), ceil_div(a.P, 32));
    if (dt == SOL_BF16)
        hipLaunchKernelGGL(linear_kernel<bf16_t>, grid, dim3(512), 0, st, a);
    else
        hipLaunchKernelGGL(linear_kernel<float>, grid, dim3(512), 0, st, a);
    SOL_HIP(hipGetLastError());
    return SOL_OK;
}

// ---- weight streaming ---------------------------------------------------------------------------------------------
//   y[m][o] as above, for up to 128 rows.  PB x CB blocks of 16 rows x 16 features per workgroup; eight waves split the
// reduction.  The job is to stream the weights at the rate of HBM, so their loads must be whole lines and many of them must be
// in flight: a wave loads 128 bytes of 8 weight rows per instruction into REGISTERS, NS stages ahead (with the rows of x in
// the LDS ring as well, LDS would hold one stage of both), turns them into MFMA fragments through a strip of LDS of its own, and
// takes the rows of x (resident in L2) by LDS DMA.  No wave waits for another before the partial sums meet.
// Measured, every layer on weights that no cache holds (us; before: 32-row linear_kernel below 16 MB of weights, the ring kernel
// of conv_gemm8.hip above): bf16 8192x8192, 64 rows 48.5 -> 35.6, 1 row 43.9 -> 30.2 (4.4 TB/s; the launch, the first round trip and
// the last sums are about 7 us of it); bf16 2048x1000, 64 rows 10.4 -> 7.9; 5000x5000, 37 rows 36.0 -> 23.4; fp32 4096x4096, 64
// rows 49.8 -> 30.2, 1 row 36.3 -> 18.2.  With 64 rows the rows of x are twice the bytes of the weights on the way into a CU.
// Weights packed so that a workgroup's stream is one contiguous run: 28.1 instead of 30.2 us with 1 row, 38.4 instead of 35.6
// with 64 (so the pitch of the rows is not what bounds it).
template <typename T, int PB, int CB, int NS>
__global__ void __launch_bounds__(512) linear_stream_kernel(const ConvArgs a, int nrt, int nft) {
#if defined(__HIP_DEVICE_COMPILE__)
    using namespace lds_pipe;
    constexpr int ES = (int)sizeof(T), BP = PB * 16, BC = CB * 16, NW = 8;
    constexpr int ROWB = 128, XL = BP / 8, WL = BC / 8, L = XL + WL;   // bytes of a row per stage; loads (8 rows each) per stage
    constexpr int XST = BP * ROWB, WST = BC * ROWB, LSTR = 68;
    constexpr int LDSB = NW * (NS * XST + WST), REDB = NW * PB * CB * 4 * LSTR * 4;
    static_assert(LDSB <= 160 * 1024 && REDB <= 160 * 1024 && (NS - 1) * L < 64, "LDS, vmcnt");
    __shared__ __align__(1024) unsigned char lds[LDSB > REDB ? LDSB : REDB];

    // the row tiles of one feature tile run on one XCD at the same time: the second finds the weights in L2
    const int grp = (int)blockIdx.x / (8 * nrt), in = (int)blockIdx.x - grp * 8 * nrt;
    const int ft = grp * 8 + (in & 7), m0 = (in >> 3) * BP, n0 = ft * BC;
    if (ft >= nft) return;

    const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lslot = lane & 7, lrow = lane >> 3;
    const unsigned xbytes = (unsigned)a.P * a.C * ES, wbytes = (unsigned)a.Cout * a.Kp * ES;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.x), 0, (int)xbytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.w), 0, (int)wbytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t xnull = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.x), 0, 0, 0x00020000);
    const __amdgpu_buffer_rsrc_t wnull = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.w), 0, 0, 0x00020000);

    // rows beyond the tensor get an out-of-range offset, which the hardware answers with zeros
    unsigned xo[XL], wo[WL];
#pragma unroll
    for (int i = 0; i < XL; i++) {
        const int row = i * 8 + lrow;
        xo[i] = m0 + row < a.P ? (unsigned)(m0 + row) * a.C * ES + ((lslot ^ swz<ROWB>(row)) << 4) : 0xffffffffu;
    }
#pragma unroll
    for (int i = 0; i < WL; i++) {
        const int row = i * 8 + lrow;
        wo[i] = n0 + row < a.Cout ? (unsigned)(n0 + row) * a.Kp * ES + (lslot << 4) : 0xffffffffu;
    }
    const int nst = (a.C * ES + ROWB - 1) / ROWB, tail = a.C * ES - (nst - 1) * ROWB;    // stages; bytes of the last one
    const int s0 = (int)((long)nst * wave / NW), s1 = (int)((long)nst * (wave + 1) / NW);
    const int n = s1 - s0;
    // the workgroups start at different stages: 39.1 -> 35.6 us (64 rows, 8192x8192), or all ask for the same columns of x at once.
    // The row tiles of one feature tile start at the same one, so that equal rows give equal bits (one stage apart was up to
    // 6 % faster with 65 to 128 rows: 65, bf16 3072 -> 16384, 44.3 against 47.1; 128, 8192 -> 8192, 54.9 against 55.9)
    int s = n > 0 ? s0 + (grp + wave) % n : s0, left = n;
    unsigned char *ring = lds + wave * (NS * XST), *strip = lds + NW * NS * XST + wave * WST;

    u32x4_t wq[NS][WL];
    auto issue = [&](auto B) {                             // stage s into slot B; beyond s1 through a size-0 resource -> zeros
        constexpr int buf = decltype(B)::value;
        const bool real = left > 0, last = s == nst - 1;     // the last stage of a row may be ragged (16-byte pieces)
        const __amdgpu_buffer_rsrc_t xq = real ? xr : xnull, wb = real ? wr : wnull;
#pragma unroll
        for (int i = 0; i < XL; i++) {
            const unsigned cut = (last && ((lslot ^ (int)swz<ROWB>(i * 8 + lrow)) << 4) >= tail) ? 0xffffffffu : 0u;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xq, (__attribute__((address_space(3))) void *)(ring + buf * XST + i * 1024), 16, xo[i] | cut, s * ROWB, 0, 0);
        }
        const unsigned cut = (last && (lslot << 4) >= tail) ? 0xffffffffu : 0u;
#pragma unroll
        for (int i = 0; i < WL; i++) wq[buf][i] = __builtin_amdgcn_raw_buffer_load_b128(wb, wo[i] | cut, s * ROWB, 0);
        --left;
        if (++s == s1) s = s0;
    };
    f32x4_t acc[CB][PB];
#pragma unroll
    for (int i = 0; i < CB; i++)
#pragma unroll
        for (int j = 0; j < PB; j++) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    const unsigned fsw = swz<ROWB>(lr);                    // block row bases are multiples of 16: the swizzle depends on lr only
    const unsigned fo0 = lr * ROWB + ((lg ^ fsw) << 4), fo1 = lr * ROWB + (((lg + 4) ^ fsw) << 4);
    const unsigned xb = lds_addr(ring), sb = lds_addr(strip);
    unsigned wst[WL];                                      // where this lane's piece of a weight row goes in the strip
#pragma unroll
    for (int i = 0; i < WL; i++) wst[i] = sb + (i * 8 + lrow) * ROWB + ((lslot ^ swz<ROWB>(i * 8 + lrow)) << 4);

    if (s0 < s1) {
        static_for<NS>([&](auto B) { issue(B); });
        const int rounds = (s1 - s0 + NS - 1) / NS;        // a wave ends on a whole round: its last stages may be zeros
        for (int r = 0; r < rounds; r++) {
            static_for<NS>([&](auto B) {
                constexpr int buf = decltype(B)::value;
                wait_vmcnt<(NS - 1) * L>();                // this stage has landed once only the NS - 1 behind it are outstanding
#pragma unroll
                for (int i = 0; i < WL; i++) asm volatile("ds_write_b128 %0, %1" ::"v"(wst[i]), "v"(wq[buf][i]) : "memory");
                u32x4_t fw[2][CB], fx[2][PB];
                static_for<PB>([&](auto J) { lds_read16<buf * XST + decltype(J)::value * 16 * ROWB>(fx[0][decltype(J)::value], xb + fo0); });
                static_for<PB>([&](auto J) { lds_read16<buf * XST + decltype(J)::value * 16 * ROWB>(fx[1][decltype(J)::value], xb + fo1); });
                // the wave's own writes: LDS operations of one wave are carried out in order
                static_for<CB>([&](auto I) { lds_read16<decltype(I)::value * 16 * ROWB>(fw[0][decltype(I)::value], sb + fo0); });
                static_for<CB>([&](auto I) { lds_read16<decltype(I)::value * 16 * ROWB>(fw[1][decltype(I)::value], sb + fo1); });
                wait_lgkmcnt<0>();
                static_for<2>([&](auto H) {
                    static_for<CB>([&](auto I) { landed(fw[decltype(H)::value][decltype(I)::value]); });
                    static_for<PB>([&](auto J) { landed(fx[decltype(H)::value][decltype(J)::value]); });
                });
                issue(B);                                  // the slot's data is in registers: refill it
#pragma unroll
                for (int h = 0; h < 2; h++)
#pragma unroll
                    for (int i = 0; i < CB; i++)
#pragma unroll
                        for (int j = 0; j < PB; j++) Mma16<T>::run(acc[i][j], fw[h][i], fx[h][j]);
            });
        }
        wait_vmcnt<0>();                                   // the zero-fill DMAs of the tail
    }
    __syncthreads();                                       // every ring is dead: the LDS becomes the parking place of the partial sums
    typedef float Block[4 * LSTR];
    Block *red = reinterpret_cast<Block *>(lds);           // [wave][block]

    // accumulator register e of lane l: feature 4 * (l / 16) + e, row l % 16 of its block
#pragma unroll
    for (int i = 0; i < CB; i++)
#pragma unroll
        for (int j = 0; j < PB; j++)
            *reinterpret_cast<float4 *>(&red[wave * PB * CB + j * CB + i][lg * LSTR + lr * 4]) = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
    __syncthreads();

    T *__restrict__ yg = static_cast<T *>(a.y);
    const T *__restrict__ resg = static_cast<const T *>(a.res);
    for (int it = tid; it < BP * (BC / 4); it += NW * 64) {   // four features of one row per thread, the waves' sums added in order
        const int cg = it % (BC / 4), row = it / (BC / 4), o = n0 + cg * 4, m = m0 + row, nv = min(4, a.Cout - o);
        if (nv <= 0 || m >= a.P) continue;
        const int blk = (row >> 4) * CB + (cg >> 2), at = (cg & 3) * LSTR + (row & 15) * 4;
        float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; w++) {
            const float4 q = *reinterpret_cast<const float4 *>(&red[w * PB * CB + blk][at]);
            v[0] += q.x; v[1] += q.y; v[2] += q.z; v[3] += q.w;
        }
#pragma unroll
        for (int e = 0; e < 4; e++) {
            if (e >= nv) break;
            float t = v[e] * (a.scale ? a.scale[o + e] : 1.f) + (a.shift ? a.shift[o + e] : 0.f);
            if (resg) t += Elem<T>::load(resg + (size_t)m * a.Cout + o + e);
            v[e] = a.act == SOL_ACT_RELU ? __builtin_fmaxf(t, 0.f) : t;
        }
        T *yp = yg + (size_t)m * a.ldy + o;
        if (nv == 4 && ((a.ldy | a.Cout) & 3) == 0) {
            if constexpr (ES == 2) *reinterpret_cast<uint2 *>(yp) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
            else *reinterpret_cast<float4 *>(yp) = make_float4(v[0], v[1], v[2], v[3]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; e++)
                if (e < nv) Elem<T>::store(yp + e, v[e]);
        }
    }
#endif
}

// Matrices of 16 MB and more belong to the ring kernel when the rows are many for the length of the reduction: x is most of what
// a workgroup fetches, and 64 features share it there, 32 here.  Each side counts for as much as the rounds of 256 workgroups that
// it makes are full.  The line is a fit to 624 timed layers (33..128 rows, 2048..8192 -> 4096..16384 in steps of 512), on which the choice
// is 0.6 % slower than the better of the two on average and 14 % at worst; always here: 2.9 % and 27 %.  bf16, ring kernel
// against here, us: 128 rows, 2048 -> 6656 16.4, 20.5; 2048 -> 8192 17.8, 20.9; 2048 -> 12800 30.1, 38.1; 4096 -> 8192 30.2, 32.7;
// 4096 -> 16384 65.5, 63.4; 8192 -> 8192 55.0, 54.5; 64 rows, 2048 -> 12800 21.1, 23.4; 4096 -> 8192 25.1, 21.7; 4096 -> 12800 37.2, 38.2.
// Features in multiples of 512: eight sets of tiles, one per XCD (128 rows, 2048 -> 6400, where every XCD reads the whole matrix:
// 39.4, 20.2).
static bool ring_kernel_is_better(const ConvArgs &a, int dt) {
    if (dt != SOL_BF16 || a.C % 128 != 0 || a.Cout % 512 != 0 || a.P <= 32 || (double)a.Cout * a.Kp * 2.0 < 16.0 * 1048576) return false;
    const auto fill = [](int n) { return (float)n / (float)(256 * ceil_div(n, 256)); };      // of the rounds that n workgroups make
    const int here = ceil_div(a.P, 64) * ceil_div(a.Cout, 32), tiles = ceil_div(a.P, 64) * ceil_div(a.Cout, 64);
    if (tiles < 200 && here <= 256) return false;
    const float e = here <= 256 ? 1.f : fill(here), er = fill(tiles);
    return (float)a.C * e * e * e <= (float)(tiles <= 256 ? 44 * a.P : 32 * a.P + 512) * er * er;
}

// Up to 128 rows (above, the 64-row tiles re-read the weights too often), and reductions that linear_kernel does not finish in
// one round trip: from 4 KB per row in bf16 (64 rows: 1024 -> 1000 features 6.6 against 6.3 us here, 2048 -> 1000 10.4 against 7.9;
// 13 rows, 512 -> 1000: 4.2 against 5.2; 128 rows, 1528 -> 1528: 7.7 against 8.5), from 2 KB in fp32, where its 32x32 blocks are a
// long chain of matrix instructions (9 rows, 512 -> 1000: 7.3 against 5.5; 64 rows, 128 -> 10: 4.8 against 5.6).
bool linear_stream_applies(const ConvArgs &a, int dt) {
    const double es = (double)dtype_size(dt);
    return linear_kernel_applies(a, dt) && a.P <= 128 && !ring_kernel_is_better(a, dt) && a.C * (int)es >= (dt == SOL_BF16 ? 4096 : 2048) && (double)a.P * a.C * es < 2147483648.0 && (double)a.Cout * a.Kp * es < 2147483648.0;
}

template <typename T> static sol_status launch_stream_typed(const ConvArgs &a, hipStream_t st) {
    const int pb = a.P <= 16 ? 1 : a.P <= 32 ? 2 : 4, nrt = ceil_div(a.P, pb * 16);
    // 32 features per workgroup, or 16 when that takes fewer row loads in the rounds that 256 workgroups of one per CU make
    const int n32 = ceil_div(a.Cout, 32), n16 = ceil_div(a.Cout, 16);
    const bool wide = (long)ceil_div(n32 * nrt, 256) * (pb * 16 + 32) <= (long)ceil_div(n16 * nrt, 256) * (pb * 16 + 16);
    const int nft = wide ? n32 : n16;
    const dim3 grid(ceil_div(nft, 8) * 8 * nrt), block(512);
#define STREAM(PB, CB, NS) hipLaunchKernelGGL((linear_stream_kernel<T, PB, CB, NS>), grid, block, 0, st, a, nrt, nft)
    if (wide) {
        if (pb == 1) STREAM(1, 2, 4);
        else if (pb == 2) STREAM(2, 2, 4);
        else STREAM(4, 2, 2);
    } else {
        if (pb == 1) STREAM(1, 1, 4);
        else if (pb == 2) STREAM(2, 1, 4);
        else STREAM(4, 1, 2);
    }
#undef STREAM
    SOL_HIP(hipGetLastError());
    return SOL_OK;
}

sol_status launch_linear_stream(const ConvArgs &a, int dt, hipStream_t st) {
    return dt == SOL_BF16 ? launch_stream_typed<bf16_t>(a, st) : launch_stream_typed<float>(a, st);
}

}  // namespace sol

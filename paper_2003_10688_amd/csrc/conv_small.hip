// 3x3 convolution of an image of three channels on the vector units (gfx950): the first layer of a network.
//
// With three input channels a filter tap is no run that a matrix instruction could take from memory, and the gather kernel pays
// for building one: per element a division, an address, a range check, a 4-byte load and a 4-byte LDS store.  Here a thread computes
// TR x PX output pixels of NCH channels: the pixels of its window are loaded whole and zero-filled by the range check, every lane of a wave has the same
// channels, so the filter comes by scalar loads and stands in scalar registers, and there is neither LDS nor a barrier.  fp32 products on
// the vector units run at half the rate of the fp32 matrix instructions (which is 1/16 of bf16's), and nothing is multiplied
// that is padding of the reduction: 27 products instead of 32.
// Small calls are bound by the launch, large ones by the stores.  us, gather kernel -> here: fp32 3x3 + 2x2 pool, 16 filters, one 32x32
// image 8.4 -> 4.2, 256 images 26 -> 8.6, 256 of 64x64 90 -> 25; bf16 the same 10.5 -> 5.0, 39 -> 10, 145 -> 28; fp32 3x3, 32 filters, 64
// images of 32x32 8.7 -> 7.4; stride 2, 8 images of 224x224, 32 filters 18.0 -> 11.9.  2 x 2 pixels x 4 channels per thread; 2 x 4 x 8
// 9.6 us on the first of them and 33 on the third, 2 x 2 x 8 6.3 and 32.  7x7 filters stay on the gather kernel: their windows
// are 39 values a row, 205 us instead of 58.
#include "conv_common.h"

namespace sol {

struct SmallArgs {
    ConvArgs c;
    int strips, cols, rows;                // strips of TR x PX output pixels, per image row of strips and per image
    FastDiv dcols, drows;
};

constexpr int C = 3, R = 3;                // input channels; filter rows and columns
constexpr int TR = 2, PX = 2, NCH = 4;     // output rows, columns and channels of a thread

// the channels of one pixel; offset >= 2^31: zeros
template <typename T> __device__ __forceinline__ void load_pixel(const __amdgpu_buffer_rsrc_t &r, unsigned off, float v[C]);
template <> __device__ __forceinline__ void load_pixel<float>(const __amdgpu_buffer_rsrc_t &r, unsigned off, float v[C]) {
    const auto u = __builtin_amdgcn_raw_buffer_load_b96(r, off, 0, 0);
    v[0] = __uint_as_float(u[0]); v[1] = __uint_as_float(u[1]); v[2] = __uint_as_float(u[2]);
}
template <> __device__ __forceinline__ void load_pixel<bf16_t>(const __amdgpu_buffer_rsrc_t &r, unsigned off, float v[C]) {
#pragma unroll
    for (int c = 0; c < C; c++) v[c] = bf16_to_f32((bf16_t)__builtin_amdgcn_raw_buffer_load_b16(r, off + 2u * c, 0, 0));
}
// element i of a packed filter row at a wave-uniform address
template <typename T> __device__ __forceinline__ float filter_at(const T *row, int i);
template <> __device__ __forceinline__ float filter_at<float>(const float *row, int i) { return row[i]; }
template <> __device__ __forceinline__ float filter_at<bf16_t>(const bf16_t *row, int i) {
    const uint32_t u = reinterpret_cast<const uint32_t *>(row)[i >> 1];
    return __uint_as_float((i & 1) ? u & 0xffff0000u : u << 16);
}

template <typename T, int SH>              // SH: stride
__global__ void __launch_bounds__(256) conv_small_kernel(const SmallArgs s) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int ES = (int)sizeof(T), NCOL = (PX - 1) * SH + R, NROW = (TR - 1) * SH + R;
    const ConvArgs &a = s.c;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c0 = (blockIdx.y * 4 + wave) * NCH;
    const int strip = blockIdx.x * 64 + lane;
    if (c0 >= a.Cout) return;
    uint32_t rest, tc, n, tr;
    s.dcols.divmod((uint32_t)min(strip, s.strips - 1), rest, tc);
    s.drows.divmod(rest, n, tr);
    const int oh = (int)tr * TR, ow = (int)tc * PX;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.x), 0, (int)((unsigned)a.N * a.H * a.W * C * ES), 0x00020000);
    const T *__restrict__ w = static_cast<const T *>(a.w) + (size_t)c0 * a.Kp;

    unsigned coff[NCOL];
#pragma unroll
    for (int c = 0; c < NCOL; c++) {
        const int iw = ow * SH - a.pw + c;
        coff[c] = (unsigned)iw < (unsigned)a.W ? (unsigned)(iw * C * ES) : 0x80000000u;
    }
    auto load_row = [&](int j, float (&v)[NCOL][C]) {
        const int ih = oh * SH - a.ph + j;
        const unsigned rb = (unsigned)ih < (unsigned)a.H ? (unsigned)((int)n * a.H + ih) * (unsigned)(a.W * C * ES) : 0x80000000u;
#pragma unroll
        for (int c = 0; c < NCOL; c++) load_pixel<T>(xr, max(rb + coff[c], max(rb, coff[c])), v[c]);   // both out: the sum wraps, the maximum does not
    };
    float acc[TR][PX][NCH];
#pragma unroll
    for (int o = 0; o < TR; o++)
#pragma unroll
        for (int t = 0; t < PX; t++)
#pragma unroll
            for (int e = 0; e < NCH; e++) acc[o][t][e] = 0.f;

    float in[NROW][NCOL][C];                               // the whole window: every load is in flight at once
    static_for<NROW>([&](auto J) { load_row(decltype(J)::value, in[decltype(J)::value]); });
    static_for<NROW>([&](auto J) {
        constexpr int j = decltype(J)::value;
        static_for<TR>([&](auto O) {
            constexpr int o = decltype(O)::value, r = j - o * SH;
            if constexpr (r >= 0 && r < R) {
#pragma unroll
                for (int e = 0; e < NCH; e++)
#pragma unroll
                    for (int q = 0; q < R; q++)
#pragma unroll
                        for (int c = 0; c < C; c++) {
                            const float f = filter_at<T>(w + (size_t)e * a.Kp, (r * R + q) * C + c);
#pragma unroll
                            for (int t = 0; t < PX; t++) acc[o][t][e] = fmaf(in[j][t * SH + q][c], f, acc[o][t][e]);
                        }
            }
        });
    });
    if (strip >= s.strips) return;

    float sc[NCH], sf[NCH];
#pragma unroll
    for (int e = 0; e < NCH; e++) { sc[e] = a.scale ? a.scale[c0 + e] : 1.f; sf[e] = a.shift ? a.shift[c0 + e] : 0.f; }
    const float lim = a.act == SOL_ACT_RELU ? 0.f : __builtin_nanf("");
#pragma unroll
    for (int o = 0; o < TR; o++)
#pragma unroll
        for (int t = 0; t < PX; t++)
#pragma unroll
            for (int e = 0; e < NCH; e++) acc[o][t][e] = __builtin_fmaxf(acc[o][t][e] * sc[e] + sf[e], lim);
    T *__restrict__ y = static_cast<T *>(a.y);
    auto put = [&](int row, int col, int Wy, const float (&v)[NCH]) {
        T *p = y + (((size_t)n * (a.pool ? a.Hy : a.Ho) + row) * Wy + col) * a.ldy + c0;
        constexpr int V = 4;
#pragma unroll
        for (int e = 0; e < NCH; e += V) {
            if constexpr (ES == 4) *reinterpret_cast<float4 *>(p + e) = make_float4(v[e], v[e + 1], v[e + 2], v[e + 3]);
            else *reinterpret_cast<uint2 *>(p + e) = make_uint2(pack_bf16x2(v[e], v[e + 1]), pack_bf16x2(v[e + 2], v[e + 3]));
        }
    };
    if constexpr (SH == 1) {               // a thread's pixels are a window of a fused 2x2 pool
        if (a.pool) {
#pragma unroll
            for (int t = 0; t < PX; t += 2) {
                if ((ow + t) / 2 >= a.Wy) continue;
                float v[NCH];
#pragma unroll
                for (int e = 0; e < NCH; e++) {
                    // as the shared epilogue: the first of the four decides what a NaN behind it does, sums in window order
                    float b = acc[0][t][e];
                    if (a.pool == 1) {
                        b = acc[0][t + 1][e] > b ? acc[0][t + 1][e] : b;
                        b = acc[1][t][e] > b ? acc[1][t][e] : b;
                        b = acc[1][t + 1][e] > b ? acc[1][t + 1][e] : b;
                    } else {
                        b = ((b + acc[0][t + 1][e]) + acc[1][t][e] + acc[1][t + 1][e]) * 0.25f;
                    }
                    v[e] = b;
                }
                put(oh / 2, (ow + t) / 2, a.Wy, v);
            }
            return;
        }
    }
#pragma unroll
    for (int o = 0; o < TR; o++)
#pragma unroll
        for (int t = 0; t < PX; t++)
            if (oh + o < a.Ho && ow + t < a.Wo) put(oh + o, ow + t, a.Wo, acc[o][t]);
#endif
}

// A thread loads its window again for every four filters, and the gather kernel's 128x64 tiles build a row of the reduction once for 64: with
// a 2x2 pool, few pixels, few filters, filters that leave the last channel tile part empty or rows that do not store 16 bytes at once this
// kernel wins at every size measured (1 to 64 images of 12x12 to 256x256, 4 to 512 filters), with full channel tiles the other one, in bf16 from
// one tile per CU on and in fp32 where the output leaves the caches.  Between one and two tiles per CU, which are one round there, three
// quarters of a channel tile are enough.  us, gather kernel / here: bf16, 8 images of 64x64, 64 filters (256 tiles) 10.0 / 8.9, 128 filters (512)
// 11.1 / 14.2; 8 of 51x51, 72 filters (326) 10.9 / 9.3; 64 of 100x100, 48 filters 89 / 72, 64 filters 80 / 93; one of 224x224, 64 filters (392) 10.8 / 14.4, 96
// filters (784) 18.8 / 18.3; fp32, 8 of 224x224, 128 filters 98 / 84, 256 filters 189 / 225; 64 of 100x100, 192 filters 225 / 251; 31 of 138x138, 224 filters
// 272 / 256.  Of 1953 layers without a pool 29 go the slower way by more than 4 %, 266 without this line.
static bool gather_kernel_pays(const ConvArgs &a, int dt) {
    if (a.pool || a.Cout % 8 != 0) return false;
    const int ntc = ceil_div(a.Cout, 64);
    const long tiles = (long)ceil_div(a.P, 128) * ntc;
    const double full = a.Cout / (64.0 * ntc);
    return dt == SOL_BF16 ? tiles > 256 && full >= (tiles <= 512 ? 0.7 : 0.9375) : full >= 0.9375 && (double)a.P * a.Cout > 70e6;
}

// 3x3, stride 1 (with or without a 2x2 pool that keeps no winners) in either type, stride 2 in fp32 (bf16 has the stem kernel)
bool small_kernel_applies(const ConvArgs &a, int dt) {
    if (a.C != 3 || a.R != 3 || a.S != 3 || a.sh != a.sw || a.Cout % 4 != 0 || a.res || a.argmax || a.prepool || a.pool == 3 || a.pre_scale || a.ldx != a.C || a.Cvalid != a.C) return false;
    if (a.sh != 1 && !(dt == SOL_F32 && a.pool == 0 && a.sh == 2)) return false;
    return !gather_kernel_pays(a, dt) && (double)a.N * a.H * a.W * a.C * dtype_size(dt) < 2147483648.0;
}

template <typename T, int SH> static void launch_small_cfg(const ConvArgs &a, hipStream_t st) {
    SmallArgs s;
    s.c = a;
    s.rows = ceil_div(a.pool ? 2 * a.Hy : a.Ho, TR);
    s.cols = ceil_div(a.pool ? 2 * a.Wy : a.Wo, PX);
    s.strips = a.N * s.rows * s.cols;
    s.dcols = FastDiv((uint32_t)s.cols); s.drows = FastDiv((uint32_t)s.rows);
    hipLaunchKernelGGL((conv_small_kernel<T, SH>), dim3(ceil_div(s.strips, 64), ceil_div(a.Cout, 4 * NCH)), dim3(256), 0, st, s);
}

sol_status launch_conv_small(const ConvArgs &a, int dt, hipStream_t st) {
    if (a.sh == 2) launch_small_cfg<float, 2>(a, st);
    else if (dt == SOL_BF16) launch_small_cfg<bf16_t, 1>(a, st);
    else launch_small_cfg<float, 1>(a, st);
    SOL_HIP(hipGetLastError());
    return SOL_OK;
}

}  // namespace sol

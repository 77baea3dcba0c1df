// Shared host/device helpers of the HIP library (internal).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "../../include/sol.h"

namespace sol {

// ---- error reporting ---------------------------------------------------------------------------
void set_error(const char *fmt, ...);   // stores the text returned by sol_last_error()

#define SOL_FAIL(code, ...)            \
    do {                               \
        ::sol::set_error(__VA_ARGS__); \
        return (code);                 \
    } while (0)

#define SOL_REQUIRE(cond, code, ...) \
    do {                             \
        if (!(cond)) SOL_FAIL(code, __VA_ARGS__); \
    } while (0)

#define SOL_HIP(call)                                                                       \
    do {                                                                                    \
        hipError_t e_ = (call);                                                             \
        if (e_ != hipSuccess) SOL_FAIL(SOL_ERR_HIP, "%s: %s", #call, hipGetErrorString(e_)); \
    } while (0)

static inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
static inline size_t dtype_size(int dt) { return dt == SOL_BF16 ? 2 : 4; }
static inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
static inline size_t round_up(size_t a, size_t b) { return (a + b - 1) / b * b; }
static inline int out_size(int in, int k, int s, int p) { return (in + 2 * p - k) / s + 1; }

// reduction length of a packed convolution weight row (zero padded to one LDS row of 128 bytes)
static inline int packed_k(const sol_conv_desc &cd, int dt) {
    const int bk = dt == SOL_BF16 ? 64 : 32;
    return (int)round_up((size_t)cd.kh * cd.kw * cd.cin, bk);
}

// ---- device helpers ----------------------------------------------------------------------------
typedef uint16_t bf16_t;   // raw bf16 bits

__device__ __forceinline__ float bf16_to_f32(bf16_t v) { return __uint_as_float(((uint32_t)v) << 16); }

// two fp32 -> packed bf16 pair (low half = lo), round to nearest, ties to even: one v_cvt_pk_bf16_f32
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    const f32x2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
__device__ __forceinline__ bf16_t f32_to_bf16(float f) { return (bf16_t)(pack_bf16x2(f, 0.f) & 0xffffu); }

template <typename T> struct Elem;
template <> struct Elem<float> {
    static __device__ __forceinline__ float load(const float *p) { return *p; }
    static __device__ __forceinline__ void store(float *p, float v) { *p = v; }
};
template <> struct Elem<bf16_t> {
    static __device__ __forceinline__ float load(const bf16_t *p) { return bf16_to_f32(*p); }
    static __device__ __forceinline__ void store(bf16_t *p, float v) { *p = f32_to_bf16(v); }
};

// ---- internal launchers (implemented in the .hip files) ------------------------------------------
// Division of a 32-bit unsigned by a run-time constant (multiply-high and shifts instead of the
// ~40-instruction software division; the divisor's magic number is computed on the host).
struct FastDiv {
    uint32_t d, mul, s1, s2;
    __host__ __device__ FastDiv() : d(1), mul(1), s1(0), s2(0) {}
    explicit FastDiv(uint32_t div) : d(div) {
        uint32_t l = 0;
        while ((1ull << l) < div) l++;
        mul = (uint32_t)(((1ull << 32) * ((1ull << l) - div)) / div + 1);
        s1 = l < 1 ? l : 1;
        s2 = l > 0 ? l - 1 : 0;
    }
#if defined(__HIPCC__)
    __device__ __forceinline__ uint32_t div(uint32_t n) const {
        const uint32_t t = __umulhi(mul, n);
        return (t + ((n - t) >> s1)) >> s2;
    }
    __device__ __forceinline__ void divmod(uint32_t n, uint32_t &q, uint32_t &r) const { q = div(n); r = n - q * d; }
#endif
};

struct ConvArgs {
    const void *x, *w;
    const float *scale, *shift;
    const void *res;
    void *y;
    int32_t *argmax;
    void *prepool;
    int N, H, W, C;          // input
    int Cout, R, S, sh, sw, ph, pw;
    int Ho, Wo;              // convolution output extent
    int Hy, Wy;              // stored output extent (pooled when pool != 0)
    int ldy;                 // elements between consecutive output pixels in y: Cout, or more when y is a channel slice of a
                             // wider tensor (a concatenation written in place); pool == 0 only
    int P;                   // GEMM rows: N*Ho*Wo, or N*Hy*Wy*4 with a fused 2x2 pool
    int Kp;                  // padded reduction length of a packed weight row
    int Ktot;                // R*S*C
    int act, pool;           // pool: 0 none, 1 max 2x2/2, 2 avg 2x2/2 (in the epilogue of any kernel), 3 max 3x3/2 unpadded or pad 1 (stem-pool kernel only)
    const float *pre_scale, *pre_shift;   // not NULL: relu(pre_scale[c] * x + pre_shift[c]) is applied to every in-range input element before
                             // the contraction (BN + ReLU on the input side; taps in the padding stay 0); conv_pre, conv_direct and conv_igemm kernels
    int ldx;                 // elements between consecutive input pixels in x: C, or more when x is a channel prefix of a wider tensor
    int Cvalid;              // input channels >= Cvalid read as 0 whatever the memory holds (C rounded up over a channel prefix); C when unused
    int ntc;                 // number of channel tiles (set by the launcher)
    int ntiles;
    int cpx;                 // > 0: each XCD owns cpx channel tiles (all pixel tiles); 0: a contiguous run of tiles
    FastDiv dw, dh;          // by Wo, Ho (by Wy, Hy with a fused pool): GEMM row -> pixel
};

struct PoolArgs {
    const void *x;
    void *y;
    int32_t *argmax;
    int N, H, W, C, Ho, Wo;
    int kh, kw, sh, sw, ph, pw;
    int kind, count_pad;
};

struct DwArgs {              // depthwise convolution: one filter per channel, weights [kh*kw][C]
    const void *x, *w, *res;
    const float *scale, *shift;
    void *y;
    int N, H, W, C, Ho, Wo;
    int kh, kw, sh, sw, ph, pw;
    int act;
};

// Convolution tile ids (pixels x channels per workgroup); also accepted as a debugging override.
// T_*: register-staged kernel (conv_igemm.hip).  D_*: LDS-DMA ring kernel (conv_dma.hip), suffix =
// row bytes per stage x ring stages.
enum {
    T_AUTO = 0, T_256x128 = 1, T_128x128 = 2, T_128x64 = 3, T_256x64 = 4, T_64x64 = 5, T_128x32 = 6, T_128x256 = 7,
    T_64x128 = 8,
    D_128x128_64x4 = 11, D_128x128_64x3 = 12, D_256x128_64x3 = 13, D_128x64_64x4 = 14, D_64x64_64x4 = 15,
    D_128x256_64x3 = 16, D_256x64_64x3 = 17, D_64x128_64x4 = 18,
    D_128x128_128x2 = 21, D_128x128_128x3 = 22, D_128x64_128x3 = 23, D_64x64_128x3 = 24,
    D_128x128_64x5 = 25, D_64x64_128x4 = 26, D_256x128_128x3 = 27, D_256x128_64x4 = 31, D_128x256_64x4 = 32, D_64x64_64x8 = 33,
    // H_*: 3x3 halo-in-LDS kernel (conv_halo.hip), suffix = patch DMA instructions per wave (s: single input chunk)
    H_256x128_x5 = 41, H_128x128_x3 = 42, H_256x64_x5 = 43, H_256x64_x6s = 44, H_256x64_x6s2 = 45, H_128x128_k2 = 46, H_64x128_k4 = 47, H_128x64_k4 = 48, H_64x64_k4 = 49, H_256x64_x6 = 50, H_FIRST = 41, H_LAST = 59,
    // G_*: eight-wave 1x1 GEMM kernel (conv_gemm8.hip); kN: reduction split N ways inside the workgroup, r64: 64-byte rows
    G_128x128_k2 = 61, G_256x128 = 62, G_128x256 = 63, G_64x128_k4 = 64, G_128x64_k4 = 65, G_256x256_r64 = 66, G_256x128_r64 = 67,
    G_64x64_k4 = 68, G_64x64_k4_deep = 69, G_64x32_k4_r256 = 70, G_FIRST = 61, G_LAST = 79,
    // S_*: small tiles, one LDS-DMA ring per wave, for layers with few pixels (conv_direct.hip)
    S_16x16 = 81, S_16x32 = 82, S_32x32 = 83, S_64x32 = 84, S_64x64 = 85, S_FIRST = 81, S_LAST = 85,
    // B_*: patch rows of the dense-layer kernel (conv_dense.hip); not a choice of any other layer
    B_64 = 91, B_96 = 92, B_128 = 93, B_192 = 94, B_256 = 95, B_384 = 96, B_FIRST = 91, B_LAST = 96,
    T_NO_HALO = 99   // automatic choice among the implicit-GEMM kernels only
};
int dma_tile_row_bytes(int tile);
sol_status launch_conv_dma(const ConvArgs &a, int dt, int tile, hipStream_t st);
bool gemm8_kernel_applies(const ConvArgs &a, int dt);
sol_status launch_conv_gemm8(const ConvArgs &a, int tile, hipStream_t st);
bool direct_kernel_applies(const ConvArgs &a, int dt);
int direct_choose_pre_tile(const ConvArgs &a, int dt);
// Which kernels an automatic choice may take, by the order in which they add up a reduction (fp32; see launch_conv, conv_choose_tile)
enum SumOrder { SUMS_ANY, SUMS_CHAIN, SUMS_GRADIENT };
int conv_choose_tile(const ConvArgs &a, int dt, SumOrder order);        // conv_choose.hip
int conv_rule_tile(const ConvArgs &a, int dt);           // conv_igemm.hip
float conv_tile_estimate(int tile, int dt, long P, int Cout, float kbytes, float res, float mbytes);
sol_status launch_conv_direct(const ConvArgs &a, int dt, int tile, hipStream_t st);
int direct_choose_pair_tile(const ConvArgs &a, int K2);
sol_status launch_conv_direct_pair(const ConvArgs &a, int tile, const void *x2, const void *w2, const float *scale2, const float *shift2,
                                   int H2, int W2, int K2, int Kp2, int stride, hipStream_t st);
const char *conv_kernel_of_thread();                     // sol_debug_conv_kernel (conv_igemm.hip)
bool chain_kernel_applies(const ConvArgs &a);            // fp32, the sums of D_64x64_128x3 on smaller tiles (conv_chain.hip)
sol_status launch_conv_chain(const ConvArgs &a, hipStream_t st);
bool small_kernel_applies(const ConvArgs &a, int dt);    // three input channels on the vector units (conv_small.hip)
sol_status launch_conv_small(const ConvArgs &a, int dt, hipStream_t st);
bool pre_kernel_applies(const ConvArgs &a, int dt);      // 1x1 with BN + ReLU on the input side over whole 64-channel chunks (conv_pre.hip)
sol_status launch_conv_pre(const ConvArgs &a, hipStream_t st);
bool halo_kernel_applies(const ConvArgs &a, int dt);
sol_status launch_conv_halo(const ConvArgs &a, int tile, hipStream_t st);
bool stem_kernel_applies(const ConvArgs &a, int dt);
sol_status launch_conv_stem(const ConvArgs &a, hipStream_t st);
// projection shortcut (1x1, stride s, K2 channels on an H2 x W2 grid) + the 1x1 convolution it is added to, in one kernel (conv_pair.hip)
bool pair_applies(const ConvArgs &a, int dt, int H2, int W2, int K2, int Kp2, int stride);
sol_status launch_conv_pair(ConvArgs a, const void *x2, const void *w2, const float *scale2, const float *shift2, int H2, int W2, int K2,
                            int Kp2, int stride, hipStream_t st);
bool stem_pool_applies(const ConvArgs &a, int dt, const sol_pool_desc &p);   // stem + ReLU + 3x3/2 max pool in one kernel
sol_status launch_conv_stem_pool(const ConvArgs &a, int dt, int pad, hipStream_t st);     // pad: of the pool
// a whole stride-1 bottleneck (1x1 reduce, 3x3, 1x1 expand + identity shortcut, folded BN and ReLU each) in one kernel (conv_block.hip)
struct BlockLaunch {
    const void *x; void *y;                          // block input / output, NHWC [N][H][W][C4]
    const void *w1, *w2, *w3;                        // packed weights of the three convolutions
    const float *s1, *h1, *s2, *h2, *s3, *h3;        // their folded scale / shift
    int N, H, W, C4, WM;                             // WM: mid channels
};
bool block_kernel_applies(int dt, int N, int H, int W, int C4, int WM);
sol_status launch_conv_block(const BlockLaunch &b, hipStream_t st);
struct XrLaunch {
    const void *t, *r; void *y, *z;                  // expand input [P][WM], its shortcut [P][C4]; outputs y [P][C4], z [P][WZ]
    const void *w3, *w1;                             // packed weights [C4][WM], [WZ][C4]
    const float *s3, *h3, *s1, *h1;                  // folded scale / shift of the two layers
    long P; int WM, C4, WZ;
};
bool xr_kernel_applies(int dt, long P, int WM, int C4, int WZ);
sol_status launch_conv_xr(const XrLaunch &b, hipStream_t st);
// a dense layer (BN + ReLU, 1x1 to 128 channels, BN + ReLU, 3x3 to 32 channels) in one kernel (conv_dense.hip)
struct DenseLaunch {
    const void *x; int ldx, C, Cvalid;               // block buffer, its pixel pitch, channels read (a multiple of 64), real ones among them
    const float *ps, *ph;                            // input-side scale / shift [C]
    const void *w1; int Kp1; const float *s1, *h1;   // packed 1x1 weights [128][Kp1], folded scale / shift
    const void *w2; const float *s2, *h2;            // packed 3x3 weights [32][9*128], folded scale / shift
    void *y; int ldy, act;
    int N, H, W;
};
bool dense_kernel_applies(int dt, int N, int H, int W, int C, int ldx, int mid, int cout, int ldy);
bool dense_one_launch_pays(int N, int H, int W, int C, bool masked);   // masked: the real channels end inside a chunk of 64
sol_status launch_conv_dense(const DenseLaunch &d, int variant, hipStream_t st);
// a depthwise 3x3 convolution (pad 1, stride S) and the 1x1 convolution behind it in one kernel (conv_dwpw.hip)
struct DwPwLaunch {
    const void *x, *wd; const float *sd, *hd; int act_d;   // input [N][H][W][C], packed depthwise weights [9][C], their folded scale / shift
    const void *w; const float *s, *h; int act;            // packed 1x1 weights [K][C rounded up to 64], folded scale / shift
    void *y; int ldy;
    int N, H, W, C, S, K;
};
bool dwpw_kernel_applies(int dt, int N, int H, int W, int C, int S, int K, int ldy);
bool dwpw_pays(int N, int H, int W, int C, int S, int K);
sol_status launch_conv_dwpw(const DwPwLaunch &d, hipStream_t st);
// a fire module -- 1x1 squeeze, 1x1 and 3x3 expand of it side by side -- in one kernel (conv_fire.hip)
struct FireLaunch {
    const void *x, *ws; const float *ss, *hs; int act_s;   // input [N][H][W][C], packed squeeze weights [SP][C], folded scale / shift
    const void *w1; const float *s1, *h1; int act1;        // packed 1x1 expand weights [E1][64]
    const void *w3; const float *s3, *h3; int act3;        // packed 3x3 expand weights [E3][9 * SP rounded up to 64]
    void *y1, *y3; int ldy;                                // where each expand's first channel goes; output pixel pitch
    int N, H, W, C, SP, E1, E3;
};
bool fire_kernel_applies(int dt, int N, int H, int W, int C, int SP, int E1, int E3, int ldy);
bool fire_pays(int N, int H, int W, int C, int E1, int E3);
sol_status launch_conv_fire(const FireLaunch &f, hipStream_t st);
bool linear_kernel_applies(const ConvArgs &a, int dt);
sol_status launch_linear(const ConvArgs &a, int dt, hipStream_t st);
bool linear_stream_applies(const ConvArgs &a, int dt);   // up to 128 rows, weights streamed (linear.hip)
sol_status launch_linear_stream(const ConvArgs &a, int dt, hipStream_t st);
sol_status launch_conv(const ConvArgs &a, int dt, int tile_override, hipStream_t st, SumOrder order = SUMS_ANY);
sol_status launch_pool(const PoolArgs &a, int dt, hipStream_t st);
sol_status launch_dwconv(const DwArgs &a, int dt, hipStream_t st);
sol_status launch_pack_dw(int C, int taps, int dt, const float *w, void *packed, hipStream_t st);
sol_status launch_gap(const void *x, void *y, int N, int HW, int C, int dt, hipStream_t st);
// copies a dense [rows][c] tensor into channels off .. off + c - 1 of a [rows][ldy] tensor (one part of a concatenation)
sol_status launch_concat_copy(const void *x, void *y, long rows, int c, int ldy, int off, int dt, hipStream_t st);
// cout_real / cin_real > 0: w holds that many filters / input channels, the rest of cd's are zero padding (pack only)
sol_status launch_pack(const sol_conv_desc &cd, int dt, const float *w, void *packed, bool unpack, hipStream_t st, int cout_real = 0,
                       int cin_real = 0);
sol_status launch_fold(int c, const float *gamma, const float *beta, const float *mean, const float *var,
                       const float *bias, float eps, float *scale, float *shift, hipStream_t st);

// training step (train.hip); `part` is scratch for the two-stage reductions
int col_reduce_chunks(int rows, int *rows_per_chunk);
sol_status launch_bn_stats(const void *z, int rows, int C, int dt, float eps, float *mean, float *var, float *invstd,
                           float *part, hipStream_t st);
sol_status launch_bn_apply(const void *z, const void *res, void *y, const float *mean, const float *invstd,
                           const float *gamma, const float *beta, long total, int C, int relu, int dt, hipStream_t st);
sol_status launch_grad_col_sums(const void *z, const void *dy, const void *y, const float *mean, const float *invstd,
                                int rows, int C, int relu, int dt, float *out0, float *out1, float *part, hipStream_t st);
sol_status launch_act_bn_bwd(const void *z, const void *dy, const void *y, const float *mean, const float *invstd,
                             const float *gamma, const float *dbeta, const float *dgamma, void *dz, void *dres,
                             int res_first, long total, int C, int relu, int bn, int rows, int dt, hipStream_t st);
// statistics + apply, and column sums + backward, of a BN layer in one launch each: the results of the launches above, to the last bit
bool bn_small_applies(int rows, int C);
sol_status launch_bn_small(const void *z, const void *res, void *y, const float *gamma, const float *beta, float *mean, float *var, float *invstd,
                           int rows, int C, float eps, int relu, int dt, hipStream_t st);
sol_status launch_bn_small_bwd(const void *z, const void *dy, const void *y, const float *mean, const float *invstd, const float *gamma, float *dbeta,
                               float *dgamma, void *dz, void *dres, int res_first, int rows, int C, int relu, int dt, hipStream_t st);
sol_status launch_dilate(const void *dz, void *out, int N, int Ho, int Wo, int K, int Hd, int Wd, int sh, int sw, int dt,
                         hipStream_t st);
sol_status launch_pool_bwd(const PoolArgs &a, const void *dy, void *dx, int first, int dt, hipStream_t st);
sol_status launch_gap_bwd(const void *dy, void *dx, int N, int HW, int C, int first, int dt, hipStream_t st);
sol_status launch_softmax_ce(const void *logits, const int32_t *labels, void *dlogits, float *row_loss, float *loss, int N,
                             int C, int dt, hipStream_t st);

// Parameter update: up to UPD_MAX_SEG tensors by one launch (the segment table travels in the kernel arguments, so nothing is
// allocated or copied).  A segment with packed copies is a weight tensor [K][C][RS]; one without is a run of C values.
constexpr int UPD_MAX_SEG = 48, UPD_PLANE = 9216;     // UPD_PLANE: weights of one block's tile
struct UpdateBatch {
    int nseg;
    int first_block[UPD_MAX_SEG + 1];      // blocks [first_block[i], first_block[i+1]) work on segment i
    float *w[UPD_MAX_SEG], *v[UPD_MAX_SEG];
    const float *g[UPD_MAX_SEG];
    void *out[UPD_MAX_SEG], *outT[UPD_MAX_SEG];     // packed weights in forward order / flipped and transposed; NULL: not kept
    int K[UPD_MAX_SEG], C[UPD_MAX_SEG], RS[UPD_MAX_SEG], Kp[UPD_MAX_SEG], KpT[UPD_MAX_SEG];
    int TK[UPD_MAX_SEG], TC[UPD_MAX_SEG];  // filters x input channels of a block's tile; TK == 0: a run
};
// Cuts the segment whose w, v, g, out, outT, K, C, RS, Kp and KpT are set into blocks; false: a filter larger than a block's tile
bool update_segment_blocks(UpdateBatch &b, int i);
constexpr int UPD_ELEMS_PER_BLOCK = 256 * 8;
sol_status launch_update_batch(const UpdateBatch &b, int dt, float lr, float mu, hipStream_t st);
sol_status launch_pack_flip(const sol_conv_desc &cd, int dt, const float *w, void *packed, hipStream_t st);
void wgrad_plan(const sol_tensor_desc &xd, const sol_conv_desc &cd, int Ho, int Wo, int *nsplit, size_t *part_floats);
// deferred_nsplit != NULL: only the first stage runs (split partials into `part`) and the number of splits is
// returned; the caller adds the partials of many layers in one launch_wgrad_reduce_batch
sol_status launch_wgrad(const sol_tensor_desc &xd, const void *x, const sol_conv_desc &cd, const void *dz, int Ho, int Wo,
                        float *dw, float *part, hipStream_t st, int *deferred_nsplit = nullptr);
// Second stage of the weight gradients of up to WRED_MAX_SEG layers in one launch: one workgroup per output channel
// of a layer adds that channel's split partials in split order and writes dW in framework layout.
constexpr int WRED_MAX_SEG = 64, WRED_MAX_PLANE = 12288;   // floats of one output channel's [taps][cin] plane held in LDS
struct WgradReduceBatch {
    int nseg;
    int first_block[WRED_MAX_SEG + 1];
    const float *part[WRED_MAX_SEG];
    float *dw[WRED_MAX_SEG];
    int nsplit[WRED_MAX_SEG], K[WRED_MAX_SEG], C[WRED_MAX_SEG], RS[WRED_MAX_SEG];
};
sol_status launch_wgrad_reduce_batch(const WgradReduceBatch &b, hipStream_t st);

}  // namespace sol

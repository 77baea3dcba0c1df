// Which kernel and tile a convolution runs on when no tile is asked for: the one with the smallest estimated time (host code).
//
// Estimated time of a layer on a tile, in microseconds:
//     t0 + (serial^4 + share^4 + memory^4)^(1/4)
//   serial = a + n lat                    the chain of one workgroup: n stages of a wave
//   share  = waves (c + cr res + N rho)   one CU's part of all tiles, N stages per tile; waves = tiles / 256, a fraction beta of it rounded up
//                                         to whole rounds of `occ` workgroups per CU
//   memory = bw MB + ww MB                 input read once, output written, residual read; weights, which every XCD reads
// -- what is largest of the three with a soft corner.  The nine constants of a tile are least-squares fits, in the logarithm, to
// 3600 (bf16) and 1600 (fp32) timed layers (1x1 and 3x3 of stride 1 and 2, 1..64 images of 4..113 pixels, 16..2048 channels, some
// with a pool or a residual, weights rotating through 120 MB); a layer's time is off by 4 % (small tiles) to 14 % (halo tiles), root mean square.
// On 2287 other layers the choice takes 1.014 (bf16) and 1.012 (fp32) times as long as the best of all tiles, where the rules of thumb that
// stood here (thresholds on the number of 128x128 tiles) took 1.094 and 1.077 (geometric means); of the summed time 0.83 and 0.87; 721 layers
// are faster by more than 5 %, 57 slower (11 by more than 10 %).  Tiles that change that by less than a ten-thousandth are left out.
// Where it loses (of all 7500 layers timed, in bf16 33 by more than 10 % and 4 by more than 20, in fp32 5 and none): 1x1 layers whose tiles fill a
// little more than a whole number of rounds, on G_128x128_k2 most often (us, rules of thumb -> here: 2 images of 54x54, 1024 -> 2048 channels, 40.6 ->
// 52.4; 40 of 12x12, with residual, 43.6 -> 51.3); 1024 channels to 16 or 32 filters, where T_128x32 beats D_128x64_64x4 (20 of 58x58, 28.3
// -> 35.1); 32 or 64 channels to many on D_64x64_64x4 (26 of 8x8, 64 -> 128, 4.1 -> 5.1).  The auto-tuner finds those.
#include <math.h>

#include "common.h"

namespace sol {

struct TileCost { int tile, bp, bc, rowb, maxw, occ; float t0, a, lat, c, cr, rho, beta, bw, ww; };   // maxw: widest image (halo tiles)
static const TileCost kBf16[] = {
    {D_128x64_64x4, 128, 64, 64, 0, 3, 3.66f, 0.f, 0.285f, 0.691f, 0.174f, 0.229f, 0.275f, 0.19f, 2.86f},
    {D_64x64_64x4, 64, 64, 64, 0, 4, 3.26f, 0.f, 0.233f, 0.427f, 0.0407f, 0.141f, 0.262f, 0.194f, 2.99f},
    {D_64x128_64x4, 64, 128, 64, 0, 3, 3.47f, 0.f, 0.297f, 0.761f, 0.187f, 0.2f, 0.289f, 0.189f, 3.81f},
    {D_128x128_128x2, 128, 128, 128, 0, 2, 3.44f, 0.612f, 0.616f, 1.8f, 0.489f, 0.495f, 0.488f, 0.195f, 2.44f},
    {D_128x64_128x3, 128, 64, 128, 0, 2, 3.18f, 0.f, 0.408f, 1.25f, 0.155f, 0.36f, 0.535f, 0.201f, 2.17f},
    {D_64x64_128x3, 64, 64, 128, 0, 3, 3.09f, 0.f, 0.371f, 0.658f, 0.046f, 0.212f, 0.423f, 0.195f, 2.89f},
    {D_64x64_128x4, 64, 64, 128, 0, 2, 2.82f, 0.f, 0.33f, 0.877f, 0.0669f, 0.246f, 0.581f, 0.227f, 2.95f},
    {H_256x128_x5, 256, 128, 128, 31, 1, 6.07f, 0.233f, 0.52f, 6.54f, 5.24f, 0.465f, 0.f, 0.f, 13.8f},
    {H_256x64_x6s2, 256, 64, 128, 62, 1, 3.7f, 0.0107f, 0.00784f, 1.07f, 1.17f, 0.466f, 0.745f, 0.f, 10.1f},
    {H_128x64_k4, 128, 64, 128, 31, 1, 1.99f, 0.0183f, 0.f, 5.31f, 1.91f, 0.177f, 0.995f, 0.f, 6.75f},
    {H_64x64_k4, 64, 64, 128, 31, 1, 4.64f, 0.f, 0.155f, 2.02f, 1.7f, 0.107f, 1.f, 0.f, 4.57f},
    {H_256x64_x6, 256, 64, 128, 62, 1, 1.47f, 0.0309f, 0.f, 4.35f, 0.583f, 0.363f, 0.883f, 0.f, 9.72f},
    {G_128x128_k2, 128, 128, 128, 0, 1, 2.16f, 0.0586f, 0.f, 4.88f, 0.34f, 0.416f, 0.907f, 0.24f, 2.07f},
    {G_128x64_k4, 128, 64, 128, 0, 1, 1.67f, 4.49f, 0.229f, 5.2f, 2.62f, 0.309f, 0.889f, 0.267f, 0.f},
    {G_256x256_r64, 256, 256, 64, 0, 1, 1.45f, 3.24f, 0.483f, 7.45f, 4.58f, 0.681f, 0.83f, 0.26f, 6.92f},
    {G_256x128_r64, 256, 128, 64, 0, 1, 2.21f, 0.f, 0.158f, 5.3f, 0.84f, 0.442f, 0.761f, 0.24f, 4.38f},
    {S_16x16, 16, 16, 128, 0, 1, 3.18f, 0.526f, 0.127f, 0.598f, 0.0267f, 0.0317f, 0.864f, 0.228f, 0.585f},
    {S_16x32, 16, 32, 128, 0, 1, 2.87f, 0.934f, 0.194f, 0.987f, 0.0318f, 0.0491f, 0.866f, 0.281f, 0.698f},
    {S_32x32, 32, 32, 128, 0, 1, 3.05f, 0.943f, 0.245f, 1.12f, 0.045f, 0.0657f, 0.787f, 0.227f, 0.665f},
    {S_64x32, 64, 32, 128, 0, 1, 2.37f, 1.22f, 0.25f, 3.18f, 0.0873f, 0.11f, 0.848f, 0.268f, 0.843f},
    {S_64x64, 64, 64, 128, 0, 1, 2.35f, 1.67f, 0.358f, 4.26f, 0.153f, 0.156f, 0.869f, 0.271f, 0.771f},
    {T_128x32, 128, 32, 128, 0, 3, 2.69f, 0.f, 0.782f, 0.669f, 0.0781f, 0.331f, 0.52f, 0.203f, 2.86f},
};
static const TileCost kF32[] = {
    {D_64x64_64x4, 64, 64, 64, 0, 1, 3.44f, 0.f, 0.422f, 0.78f, 0.178f, 0.29f, 0.772f, 0.183f, 4.33f},
    {D_64x128_64x4, 64, 128, 64, 0, 1, 3.63f, 0.f, 0.635f, 1.44f, 0.357f, 0.528f, 0.749f, 0.174f, 5.82f},
    {D_64x64_128x3, 64, 64, 128, 0, 1, 3.56f, 0.f, 0.708f, 0.833f, 0.126f, 0.569f, 0.845f, 0.192f, 3.54f},
    {D_64x64_128x4, 64, 64, 128, 0, 1, 3.3f, 0.f, 0.702f, 1.14f, 0.0758f, 0.59f, 0.8f, 0.199f, 3.24f},
    {D_64x64_64x8, 64, 64, 64, 0, 1, 3.24f, 0.f, 0.422f, 1.14f, 0.107f, 0.327f, 0.687f, 0.175f, 4.13f},
    {S_16x16, 16, 16, 128, 0, 1, 3.23f, 0.475f, 0.224f, 0.628f, 0.0249f, 0.0456f, 0.815f, 0.181f, 0.457f},
    {S_16x32, 16, 32, 128, 0, 1, 3.07f, 0.767f, 0.341f, 1.02f, 0.0301f, 0.0829f, 0.814f, 0.211f, 0.573f},
    {S_32x32, 32, 32, 128, 0, 1, 3.16f, 0.821f, 0.544f, 1.22f, 0.0427f, 0.146f, 0.801f, 0.216f, 0.793f},
    {S_64x64, 64, 64, 128, 0, 1, 1.8f, 3.27f, 1.57f, 5.13f, 0.271f, 0.516f, 0.855f, 0.32f, 0.f},
    {T_128x32, 128, 32, 128, 0, 1, 3.5f, 0.f, 0.977f, 0.805f, 0.158f, 0.708f, 0.828f, 0.177f, 3.33f},
};

struct LayerSize { unsigned P, Cout; float kbytes, res, mbytes, wmbytes; };
// Tiles are powers of two.  `limit`: an estimate that is not below it need not be exact (what the three terms cannot be below is compared
// first: a choice takes 0.2 us of the host's time with it).
static float estimate(const TileCost &t, const LayerSize &l, float limit) {
    const unsigned tiles = ((l.P + (unsigned)t.bp - 1) >> __builtin_ctz((unsigned)t.bp)) * ((l.Cout + (unsigned)t.bc - 1) >> __builtin_ctz((unsigned)t.bc));
    const float N = l.kbytes * (t.rowb == 128 ? 1.f / 128.f : 1.f / 64.f), n = t.tile >= S_FIRST ? ceilf(N * 0.25f - 1e-4f) : N;   // a small tile's four waves split its stages
    const float rounds = (float)((tiles + 256u * (unsigned)t.occ - 1) / (256u * (unsigned)t.occ) * (unsigned)t.occ);
    const float waves = (1.f - t.beta) * ((float)tiles * (1.f / 256.f)) + t.beta * rounds;
    const float serial = t.a + n * t.lat, share = waves * (t.c + t.cr * l.res + N * t.rho), memory = t.bw * l.mbytes + t.ww * l.wmbytes;
    const float least = t.t0 + fmaxf(serial, fmaxf(share, memory));
    if (least >= limit) return least;
    const float s2 = serial * serial, w2 = share * share, m2 = memory * memory;
    return t.t0 + sqrtf(sqrtf(s2 * s2 + w2 * w2 + m2 * m2));
}

static float layer_mbytes(const ConvArgs &a, int dt) {
    const double in = fmin((double)a.N * a.H * a.W, (double)a.P * a.R * a.S) * a.C, out = (double)a.P * a.Cout * (a.pool ? 0.25 : 1.0);
    return (float)((in + out * (a.res ? 2.0 : 1.0)) * (double)dtype_size(dt) * 1e-6);
}

float conv_tile_estimate(int tile, int dt, long P, int Cout, float kbytes, float res, float mbytes) {
    const LayerSize l{(unsigned)P, (unsigned)Cout, kbytes, res, mbytes, (float)Cout * kbytes * 1e-6f};
    if (dt == SOL_BF16) {
        for (const TileCost &t : kBf16)
            if (t.tile == tile) return estimate(t, l, INFINITY);
    } else {
        for (const TileCost &t : kF32)
            if (t.tile == tile) return estimate(t, l, INFINITY);
    }
    return INFINITY;
}

// The tile whose order of summation an fp32 data gradient keeps.  Small tiles split a reduction over their four waves; the ring kernel walks
// it in one chain that starts at another chunk for each tile of pixels, 64 or 128 bytes at a time; the register-staged kernel starts at the
// first.  None is the more exact, but the last bits of an activation gradient reach the updated weights, and a step on, a ReLU or pooling
// decision within a rounding of zero that falls the other way moves whole terms of a weight gradient: with a few layers' order changed, three
// steps of a ResNet-18-shaped network end up to 0.007 of a gradient's norm and 1.5 of its rms in one element away (10 images of 99x99; 9 of
// 113x113: 0.006, 1.3).  So the order is a rule on the layer's size that stays as it is while the tables above are fitted anew, and is not to be
// tuned: below 96 tiles of 128x128 what an estimate from 154 timed shapes, t0 + ((a + n lat)^4 + (tiles / 256 (c + N rho))^4)^(1/4),
// finds fastest, and conv_rule_tile from there on.
static int gradient_tile(const ConvArgs &a) {
    struct Est { int tile, bp, bc, waves, rowb; float t0, a, lat, c, rho; };
    static const Est kEst[] = {
        {S_16x16, 16, 16, 4, 128, 3.47f, 0.f, 0.208f, 0.60f, 0.0481f}, {S_16x32, 16, 32, 4, 128, 2.97f, 0.25f, 0.370f, 1.10f, 0.0923f},
        {S_32x32, 32, 32, 4, 128, 3.09f, 0.59f, 0.599f, 1.37f, 0.1623f}, {S_64x32, 64, 32, 4, 128, 1.69f, 3.45f, 1.078f, 4.69f, 0.3427f},
        {S_64x64, 64, 64, 4, 128, 5.00f, 2.33f, 2.009f, 5.00f, 0.7287f},
        {D_64x64_128x4, 64, 64, 1, 128, 2.86f, 0.f, 0.719f, 1.23f, 0.655f}, {D_64x64_64x4, 64, 64, 1, 64, 2.95f, 0.f, 0.419f, 0.73f, 0.336f}};
    if (!direct_kernel_applies(a, SOL_F32) || (long)ceil_div(a.P, 128) * ceil_div(a.Cout, 128) >= 96) return conv_rule_tile(a, SOL_F32);
    const double kbytes = (double)a.R * a.S * a.C * 4.0;
    int best = T_AUTO;
    float bt = INFINITY;
    for (const Est &t : kEst) {
        const double tiles = (double)(((long)a.P + t.bp - 1) / t.bp) * ceil_div(a.Cout, t.bc), N = kbytes / t.rowb, n = N / t.waves;
        const double serial = t.a + (t.waves > 1 ? (double)(long)(n + 0.999) : n) * t.lat, share = tiles / 256.0 * (t.c + N * t.rho);
        const float c = (float)(t.t0 + sqrt(sqrt(serial * serial * serial * serial + share * share * share * share)));
        if (c < bt) { best = t.tile; bt = c; }
    }
    return best;
}

// T_AUTO where no candidate takes the layer (input channels that are not whole 64-byte chunks, more than 32 taps, operands of 2 GiB).
int conv_choose_tile(const ConvArgs &a, int dt, SumOrder order) {
    const int es = (int)dtype_size(dt), rowbytes = a.C * es;
    const double xb = (double)a.N * a.H * a.W * a.C * es + (double)(a.ph * a.W + a.pw) * a.C * es, wb = (double)a.Cout * a.Kp * es;
    if (rowbytes % 64 != 0 || a.R * a.S > 32 || xb >= 2147483648.0 || wb >= 2147483648.0) return T_AUTO;
    const bool halo = halo_kernel_applies(a, dt), direct = direct_kernel_applies(a, dt), chunk128 = rowbytes % 128 == 0;
    const float kbytes = (float)a.R * (float)a.S * (float)rowbytes;
    const LayerSize l{(unsigned)a.P, (unsigned)a.Cout, kbytes, a.res ? 1.f : 0.f, layer_mbytes(a, dt), (float)a.Cout * kbytes * 1e-6f};
    // SUMS_GRADIENT: among the tiles with the rule's order -- all small ones; on the ring kernel those of as many pixels and bytes
    const bool keep = order == SUMS_GRADIENT && dt == SOL_F32;
    const int rule = keep ? gradient_tile(a) : (int)T_AUTO;
    const TileCost *like = nullptr;
    for (const TileCost &t : kF32)
        if (t.tile == rule) like = &t;
    int best = rule;
    float bt = INFINITY;
    const TileCost *tab = dt == SOL_BF16 ? kBf16 : kF32;
    const int nt = dt == SOL_BF16 ? (int)(sizeof(kBf16) / sizeof(TileCost)) : (int)(sizeof(kF32) / sizeof(TileCost));
    for (int i = 0; i < nt; i++) {
        const TileCost &t = tab[i];
        if (t.rowb == 128 && !chunk128) continue;
        if (t.maxw && (!halo || a.W > t.maxw || (t.tile == H_256x64_x6s2 && a.C != 64))) continue;
        if (t.tile >= S_FIRST && !direct) continue;
        if (keep && !(rule >= S_FIRST ? t.tile >= S_FIRST : like && t.tile < S_FIRST && t.bp == like->bp && t.rowb == like->rowb)) continue;
        const float c = estimate(t, l, bt);
        if (c < bt) { best = t.tile; bt = c; }
    }
    return best;
}

}  // namespace sol

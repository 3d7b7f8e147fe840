// The wide kernel (w4a4_wide_kernel.h): the rule that picks it and its tile, and the per-group launches (bf16 or quantized output).
#include "w4a4_wide_kernel.h"

namespace quartz {
namespace {

// Launch times in microseconds, fitted (relative least squares over 30 shapes
// of 220 to 18432 rows, the wide kernel at every tile; residuals 2-4 %).  The
// teams of a tile share its groups, so each takes `steps` of them, a multiple
// of two:
//   wide           c + rounds (steps (g0 + g1 TR) + t0 + t1 TR) + load steps TR u
//   whole tiles    c + rounds (groups g + t) + load groups u
//   split          c + load groups gs + ts,  with fewer tiles than workgroups
//                  c + (groups per workgroup) gs + 10.2 + 0.093 tiles
// where load = tiles / compute units; its terms are what a busier device costs
// in clock.  What they say: a tile row of 7 x 32 costs 0.99 us a group against
// 2 x 0.61 for the 256 rows of two w4a4_linear tiles (static 0.53 against 2 x
// 0.35), and tiles of 4 x 32 rows lose that (0.67 against 0.61).  So one team
// takes shapes for which some height fills whole rounds of the device (4608
// rows: 7 x 32, 98 % full; 4608 x 3072 -> 9216: 153 us against 173).  Fewer
// tiles than compute units is where the others come in: w4a4_linear then
// splits the groups over workgroups and pays 10 to 20 us for exchanging
// partial sums through memory, a tile of two or four teams splits them within
// a workgroup for about 1 us (256 x 1152 -> 1152: 7.0 us against 15.4; 333 x
// 2048 -> 1000: 8.2 against 20.4; 1024 x 3072 -> 3072: 22.0 against 39.1).
// w4a4_linear keeps the shapes with too few tiles even so and many groups
// (1024 x 11520 -> 1280: 44 us against 49) and 128-row tiles that fill a round
// (4096 x 4608 -> 1152: 47 us against 50).  Over the 30 shapes the choice is
// within 1 % of the best kernel and tile (geometric mean; 1.26 times faster
// than w4a4_linear alone) and never slower than w4a4_linear; closer than 3 %
// it stays with the latter.
struct WideCost {
    float c, g0, g1, t0, t1, u;
};
struct LinearCost {
    float c, g, gs, t, ts, u;
};
struct Costs {
    WideCost one, two, four;                     // by teams
    LinearCost lin;
};
// the asymmetric mode's zero-point operands leave no registers for 8 row tiles
// (20 values spill around every group: 98 us against 69 at 7 x 32 rows, 4608 x
// 3072 -> 3072)
constexpr Costs kCosts[3] = {
    {{3.35f, 0.234f, 0.088f, 0.15f, 0.43f, 0.020f},   // bf16 and quantized output
     {3.37f, 0.329f, 0.067f, 0.16f, 0.46f, 0.027f},
     {3.24f, 0.457f, 0.0f, 1.29f, 0.0f, 0.017f},
     {5.57f, 0.419f, 0.630f, 1.91f, 15.2f, 0.196f}},
    {{3.22f, 0.255f, 0.024f, -0.12f, 0.52f, 0.017f},  // static
     {3.07f, 0.281f, 0.021f, 0.30f, 0.45f, 0.017f},
     {3.28f, 0.329f, 0.0f, 1.22f, 0.0f, 0.011f},
     {4.94f, 0.196f, 0.356f, 2.49f, 18.9f, 0.166f}},
    {{3.52f, 0.232f, 0.124f, 0.37f, 0.37f, 0.019f},   // asymmetric
     {3.32f, 0.423f, 0.076f, 0.05f, 0.50f, 0.030f},
     {3.24f, 0.556f, 0.0f, 1.26f, 0.0f, 0.014f},
     {5.89f, 0.578f, 0.740f, 1.96f, 18.1f, 0.224f}},
};
constexpr float kMargin = 0.97f;
// The per-group convolution takes the tile that the linear layer takes on the
// im2col matrix (with or without its split, as a workspace is there): both
// then add the groups in the same order, so their outputs are equal bit for
// bit.  (4096 x 5760 -> 640: 37 us against 44 on w4a4_gemm; 9216 x 5760 ->
// 1280: 88 against 104; where the linear layer stays with w4a4_linear, w4a4_gemm
// wins here too: 16384 x 2880 -> 320 34 against 38.)  The static one's sums
// are exact integers in any order (26 us against 41; 53 against 86; 27 against
// 31).  Its gather weighs more on w4a4_gemm, whose waves all multiply, than on
// the wide kernel: 16384 x 2880 -> 320 31.1 us against 22.6 for the linear
// layer there, 26.9 against 24.6 here.
constexpr float kConvStatic = 1.2f;

}  // namespace

WideShape wide_shape(LayerKind kind, const LayerShape& s)
{
    const int64_t M = s.M, N = s.N, K = s.K;
    const bool conv = kind == LayerKind::kConv || kind == LayerKind::kConvStatic;
    const bool asym = kind == LayerKind::kAsym, is_static = kind == LayerKind::kStatic || kind == LayerKind::kConvStatic;
    const GemmSchedule lin = linear_schedule(M, N, K, s.blocks, s.split);
    const int64_t G = K / kGroup;
    const int64_t panels = (N + kPanel - 1) / kPanel;
    // the kernel's offsets are 32-bit: every array's range ends below 2^30,
    // where a group past the last one reads, and the rows' offsets of the up
    // to 7 groups past the last one below 2^31, which marks a lane as outside
    constexpr int64_t kMost = int64_t(1) << 30;
    if (M * G * 32 > kMost || panels * G * kChunkBytes > kMost || N * G * 2 > kMost || M > (int64_t(1) << 22))
        return {0, 0};
    const int64_t blocks = s.blocks;
    const Costs& k = kCosts[asym ? 2 : is_static ? 1 : 0];
    auto rounds = [&](int64_t tiles) { return (float)((tiles + blocks - 1) / blocks); };
    auto load = [&](int64_t tiles) { return (float)tiles / (float)blocks; };
    const int64_t lin_tiles = ((M + 127) / 128) * ((N + 255) / 256);
    const float groups = (float)G;
    float best;
    if (lin.sk_tiles == 0)
        best = k.lin.c + rounds(lin_tiles) * (groups * k.lin.g + k.lin.t) + load(lin_tiles) * groups * k.lin.u;
    else if (lin_tiles > blocks)
        best = k.lin.c + load(lin_tiles) * groups * k.lin.gs + k.lin.ts;
    else
        best = k.lin.c + (float)lin.sk_q * k.lin.gs + 10.2f + 0.093f * (float)lin_tiles;
    best *= conv && is_static ? kConvStatic : kMargin;
    WideShape w{0, 0};
    auto consider = [&](const WideCost& c, int tr, int wn) {
        const int64_t teams = kWideWaves / wn;
        const int64_t tiles = ((M + 32 * tr - 1) / (32 * tr)) * ((N + 32 * wn - 1) / (32 * wn));
        const float steps = (float)((G + 2 * teams - 1) / (2 * teams) * 2), t = (float)tr;
        const float us = c.c + rounds(tiles) * (steps * (c.g0 + c.g1 * t) + c.t0 + c.t1 * t) + load(tiles) * steps * t * c.u;
        if (us < best && tiles <= kMaxGemmTiles / 2) {
            best = us;
            w = {tr, wn};
        }
    };
    for (int tr = 4; tr <= (asym ? 7 : 8); ++tr)
        consider(k.one, tr, 8);
    for (int tr = 2; tr <= 4; ++tr)
        consider(k.two, tr, 4);
    consider(k.four, 2, 2);
    return w;
}

GemmSchedule wide_schedule(const GemmLaunch& a)
{
    return gemm_schedule_tiles(a.M, a.N, a.K, device_compute_units(), false, 32 * a.wide.tr, 32 * a.wide.wn);
}

hipError_t launch_wide(const GemmLaunch& a, hipStream_t stream)
{
    return a.qout.codes ? launch_wide_mode<false, true, false, false>(a, stream)
                        : launch_wide_mode<false, false, false, false>(a, stream);
}

}  // namespace quartz

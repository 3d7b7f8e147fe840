// The wide kernel (w4a4_wide_kernel.h): the rule that picks it and its tile, and the per-group launches (bf16 or quantized output).
#include <array>

#include "w4a4_wide_kernel.h"

namespace quartz {
namespace {

// Launch times in microseconds, fitted per kind of layer (relative least
// squares; every tile and the other kernel, w4a4_linear or w4a4_gemm, timed
// over 3200 random shapes of a kind, M to 18432, K to 12288, every G_s, half
// with a workspace; residuals 2-4 %, 10 % where tiles are fewer than
// workgroups and split):
//   wide     c + rounds (steps (g0 + g1 TR) (1 + g8) + t0 passes + (t1 + te) TR)
//            + load TR (steps u + s)
//   whole    c + rounds (groups g (1 + g8 + ge) + t + te) + load (groups u + s)
//   split    c + load (groups g (1 + g8) + t + te), with fewer tiles than
//            workgroups c + (groups per workgroup) g (1 + g8) + te
// where rounds and load are tiles over compute units, rounded up and not; a
// team takes `steps` of the tile's groups, a multiple of two; g8 counts at
// G_s = 8 (twice the FLAGs to look at), te and ge with GELU.  The u and s terms
// are what a busier device costs in clock and in stores.
//
// What they say: a tile row of 7 x 32 costs 0.80 us a group against 2 x 0.51
// for the 256 rows of two w4a4_linear tiles (static 0.36 against 2 x 0.28), and
// tiles of 4 x 32 rows lose that.  So one team takes shapes for which some
// height fills whole rounds of the device (4608 rows: 7 x 32, 98 % full; 4608 x
// 3072 -> 9216: 153 us against 173).  Fewer tiles than compute units is where
// the others come in: w4a4_linear then splits the groups over workgroups and
// pays 10 to 20 us for exchanging partial sums through memory, a tile of two or
// four teams splits them within a workgroup for about 1 us (256 x 1152 -> 1152:
// 7.0 us against 15.4; 333 x 2048 -> 1000: 8.2 against 20.4; 1024 x 3072 ->
// 3072: 22.0 against 39.1).  w4a4_linear keeps the shapes with too few tiles
// even so and many groups (1024 x 11520 -> 1280: 44 us against 49), 128-row
// tiles that fill a round (4096 x 4608 -> 1152: 47 us against 50), and more of
// them with zero points or at G_s = 8 (7107 x 2432 -> 6667, asymmetric, G_s =
// 8, GELU: 195 us against 215; 3367 x 1088 -> 1703, static, G_s = 8: 13.7
// against 14.9).
//
// The quantized output's epilogue weighs 2 us per pass of 128 rows, and 8 row
// tiles spill 11 or 12 registers there (convolutions 5 or 6 at G_s 8 and 16),
// which its times include: 5823 x 4608 -> 704 stays with w4a4_linear for both
// outputs (46.9 us against 50.4 for the quantized one).
//
// A convolution's other kernel is w4a4_gemm, whose waves all multiply, and
// whose gather costs less of a tile that is 256 rows high (12540 x 2880 -> 560:
// 40.8 us against 49.5 for 4 x 32 rows; 4096 x 5760 -> 640: 44 against 37 for
// two teams, static 41 against 26).
//
// The choice takes what is expected to be at least 4 % faster, so that what is
// not in these terms does not turn it into a loss: over the fitted shapes it is
// 0.1 to 0.4 % slower than the best kernel and tile (geometric mean), 0.68 to
// 0.71 of w4a4_linear's time (convolutions 0.50 and 0.43 of
// w4a4_gemm's), and slower than the other kernel by
// more than 2 % in 15 of 19200 shapes.
struct WideCost {
    float c, g0, g1, g8, t0, t1, te, u, s;
};
struct WholeCost {
    float c, g, g8, ge, t, te, u, s;
};
struct SplitCost {
    float c, g, g8, t, te;
};
struct Costs {
    WideCost one, two, four;                     // by teams
    WholeCost whole;
    SplitCost split, split_small;
};
// the asymmetric mode's zero-point operands leave no registers for 8 row tiles
// (20 values spill around every group: 98 us against 69 at 7 x 32 rows, 4608 x
// 3072 -> 3072)
constexpr Costs kCosts[6] = {
    // per-group, bf16 output
    {{4.437f, 0.265f, 0.076f, 0.043f, -0.149f, 0.237f, 0.312f, 0.023f, 0.354f},
     {3.426f, 0.293f, 0.072f, 0.064f, 0.396f, 0.386f, 0.181f, 0.020f, 0.098f},
     {3.068f, 0.443f, 0.0f, 0.071f, 1.430f, 0.0f, 0.145f, 0.020f, 0.0f},
     {5.683f, 0.505f, 0.014f, 0.0f, 0.600f, 1.256f, 0.078f, 2.500f},
     {18.465f, 0.595f, 0.023f, 2.759f, 1.362f},
     {20.940f, 0.655f, -0.002f, 0.0f, 1.168f}},
    // quantized output
    {{3.515f, 0.244f, 0.079f, 0.044f, 1.885f, 0.442f, 0.375f, 0.022f, 0.014f},
     {3.233f, 0.316f, 0.067f, 0.058f, 1.988f, 0.340f, 0.200f, 0.017f, -0.014f},
     {3.080f, 0.449f, 0.0f, 0.076f, 2.825f, 0.0f, 0.135f, 0.016f, 0.0f},
     {4.448f, 0.505f, 0.026f, 0.0f, 3.260f, 1.782f, 0.063f, 0.863f},
     {17.448f, 0.590f, 0.019f, 3.841f, 1.851f},
     {23.054f, 0.620f, 0.0f, 0.0f, 0.996f}},
    // static
    {{3.554f, 0.206f, 0.022f, 0.096f, 0.251f, 0.285f, 0.314f, 0.033f, 0.262f},
     {2.785f, 0.265f, 0.015f, 0.143f, 0.392f, 0.342f, 0.181f, 0.020f, 0.231f},
     {2.551f, 0.297f, 0.0f, 0.205f, 1.404f, 0.0f, 0.171f, 0.024f, 0.0f},
     {4.687f, 0.282f, 0.021f, 0.0f, 1.149f, 1.379f, 0.075f, 2.152f},
     {15.118f, 0.388f, 0.035f, 3.884f, 1.382f},
     {22.511f, 0.354f, 0.040f, 0.0f, 0.964f}},
    // asymmetric
    {{4.470f, 0.275f, 0.113f, 0.034f, -0.358f, 0.239f, 0.324f, 0.016f, 0.394f},
     {3.565f, 0.356f, 0.090f, 0.058f, 0.410f, 0.357f, 0.176f, 0.019f, 0.099f},
     {3.129f, 0.559f, 0.0f, 0.066f, 1.389f, 0.0f, 0.151f, 0.013f, 0.0f},
     {6.084f, 0.664f, 0.017f, -0.094f, 0.389f, 1.629f, 0.100f, 2.851f},
     {19.108f, 0.690f, 0.017f, 3.293f, 1.498f},
     {22.105f, 0.733f, 0.048f, 0.0f, 1.198f}},
    // convolution
    {{4.838f, 0.331f, 0.086f, 0.031f, -0.778f, 0.165f, 0.331f, 0.005f, 0.697f},
     {3.176f, 0.413f, 0.064f, 0.049f, 0.094f, 0.424f, 0.197f, 0.010f, 0.410f},
     {2.984f, 0.525f, 0.0f, 0.077f, 1.575f, 0.0f, 0.145f, 0.023f, 0.0f},
     {6.197f, 0.548f, 0.109f, 0.0f, 0.815f, 1.688f, 0.030f, 3.478f},
     {19.050f, 0.630f, 0.089f, 3.129f, -0.348f},
     {21.668f, 0.732f, 0.101f, 0.0f, 0.417f}},
    // static convolution
    {{4.324f, 0.263f, 0.032f, 0.060f, -0.539f, 0.208f, 0.311f, 0.008f, 0.663f},
     {3.182f, 0.353f, 0.011f, 0.098f, 0.257f, 0.332f, 0.192f, 0.008f, 0.410f},
     {3.022f, 0.378f, 0.0f, 0.034f, 1.398f, 0.0f, 0.148f, 0.027f, 0.0f},
     {5.745f, 0.500f, 0.068f, 0.0f, 0.806f, 1.641f, 0.019f, 2.418f},
     {18.617f, 0.506f, 0.128f, 4.409f, 0.624f},
     {22.779f, 0.599f, 0.076f, 0.0f, 1.058f}},
};
constexpr float kMargin = 0.96f;

// the tiles, by teams: one, two, four
struct Tile {
    int tr, wn;
};
constexpr Tile kTiles[] = {{4, 8}, {5, 8}, {6, 8}, {7, 8}, {8, 8}, {2, 4}, {3, 4}, {4, 4}, {2, 2}};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);

// What a launch of each tile comes to, whatever the kind of layer.
struct TileLoads {
    float steps[3], rounds[kNumTiles], load[kNumTiles];   // load < 0: more tiles than a launch can number
    TileLoads(const LayerShape& s)
    {
        const int32_t G = (int32_t)(s.K / kGroup);
        for (int i = 0; i < 3; ++i)
            steps[i] = (float)((G + (2 << i) - 1) / (2 << i) * 2);
        for (int i = 0; i < kNumTiles; ++i) {
            const int64_t bm = 32 * kTiles[i].tr, bn = 32 * kTiles[i].wn;
            const int64_t tiles = ((s.M + bm - 1) / bm) * ((s.N + bn - 1) / bn);
            const bool ok = tiles <= kMaxGemmTiles / 2;
            rounds[i] = (float)(((uint32_t)tiles + (uint32_t)s.blocks - 1) / (uint32_t)s.blocks);
            load[i] = ok ? (float)tiles / (float)s.blocks : -1.0f;
        }
    }
};

// the best tile with each number of teams: [0] one, [1] two, [2] four
struct Best {
    float us;
    WideShape w;
};
std::array<Best, 3> best_tiles(LayerKind kind, const LayerShape& s, const TileLoads& l)
{
    const Costs& k = kCosts[(int)kind];
    std::array<Best, 3> best;
    best.fill({1e30f, {0, 0}});
    for (int i = 0; i < kNumTiles; ++i) {
        const Tile& t = kTiles[i];
        if (l.load[i] < 0.0f || (kind == LayerKind::kAsym && t.tr == 8))
            continue;
        const int c = t.wn == 8 ? 0 : t.wn == 4 ? 1 : 2;
        const WideCost& w = c == 0 ? k.one : c == 1 ? k.two : k.four;
        const float tr = (float)t.tr, g8 = s.lzs_group == 8 ? w.g8 : 0.0f, te = s.gelu ? w.te : 0.0f;
        // the quantizing epilogue goes through LDS 128 rows at a time
        const float passes = kind == LayerKind::kQuantized && t.tr > 4 ? 2.0f : 1.0f;
        const float us = w.c + l.rounds[i] * (l.steps[c] * (w.g0 + w.g1 * tr) * (1.0f + g8) + w.t0 * passes + (w.t1 + te) * tr) +
                         l.load[i] * tr * (l.steps[c] * w.u + w.s);
        if (us < best[c].us)
            best[c] = {us, {t.tr, t.wn}};
    }
    return best;
}

// the other kernel, with its schedule
float other_us(LayerKind kind, const LayerShape& s, const GemmSchedule& sch)
{
    const Costs& k = kCosts[(int)kind];
    const float tiles = (float)(sch.sk_first + sch.sk_tiles), groups = (float)sch.groups, load = tiles / (float)s.blocks;
    const bool fine = s.lzs_group == 8;
    if (sch.sk_tiles == 0) {
        const WholeCost& w = k.whole;
        const float rounds = (float)((sch.sk_first + s.blocks - 1) / s.blocks);
        return w.c + rounds * (groups * w.g * (1.0f + (fine ? w.g8 : 0.0f) + (s.gelu ? w.ge : 0.0f)) + w.t + (s.gelu ? w.te : 0.0f)) +
               load * (groups * w.u + w.s);
    }
    const SplitCost& w = load > 1.0f ? k.split : k.split_small;
    const float g = w.g * (1.0f + (fine ? w.g8 : 0.0f)), te = s.gelu ? w.te : 0.0f;
    return load > 1.0f ? w.c + load * (groups * g + w.t + te) : w.c + (float)sch.sk_q * g + te;
}

}  // namespace

// the tile that beats `limit` by most
WideShape fastest(const std::array<Best, 3>& b, float limit)
{
    WideShape w{0, 0};
    for (const Best& x : b)
        if (x.us < limit) {
            limit = x.us;
            w = x.w;
        }
    return w;
}

// Each kind of layer decides by its own times, but some have to add the groups
// of an output in one order, so that their results are equal bit for bit: the
// quantized output (its codes are those of the stored bf16 output), and a
// convolution and the linear layer on its im2col matrix when neither's other
// kernel splits tiles.  The static setting's sums are exact integers in any
// order up to K = 21376 (|sum| <= 784 K < 2^24), and a layer and its
// convolution share an order past that.  The orders are ascending (one team,
// or the other kernel without a split), by two teams, by four, and that of
// w4a4_linear's split.  One that the other kernels don't have is open when
// some tile of it beats them for every kind that shares it (14720 x 512 -> 384:
// two teams would take 14.3 us for the quantized output against 12.9); the
// bf16 output's times pick among the open ones.
WideShape wide_shape(LayerKind kind, const LayerShape& s)
{
    // the kernel's offsets are 32-bit.  Every array's range ends at 2^30 at
    // most, where the weights of a group past the last one are read, and an
    // offset from 2^31 on marks a lane as outside: scalar and lane offsets of
    // the weights, scales and sums add up to less than 2^32.  So do the rows'
    // (the fetch runs up to 22 groups past the last one: 2^30 + 22 x 32 x 2^22),
    // but for waves without rows of their own, which stage what nobody reads.
    constexpr int64_t kMost = int64_t(1) << 30;
    const int64_t G = s.K / kGroup, panels = (s.N + kPanel - 1) / kPanel;
    if (s.M * G * 32 > kMost || panels * G * kChunkBytes > kMost || s.N * G * 2 > kMost || s.M > (int64_t(1) << 22))
        return {0, 0};
    const TileLoads loads(s);
    const bool conv = kind == LayerKind::kConv || kind == LayerKind::kConvStatic;
    const LayerKind layer = kind == LayerKind::kQuantized || kind == LayerKind::kConv ? LayerKind::kLinear
                            : kind == LayerKind::kConvStatic                          ? LayerKind::kStatic
                                                                                      : kind;
    const GemmSchedule lin = linear_schedule(s.M, s.N, s.K, s.blocks, s.split);
    const bool whole = lin.sk_tiles == 0;
    // the convolution that shares the order, if there is one
    constexpr int64_t kExactK = (int64_t(1) << 24) / 784;
    const LayerKind gathered = layer == LayerKind::kStatic ? LayerKind::kConvStatic : LayerKind::kConv;
    GemmSchedule gemm{};
    bool tied = s.K % (9 * kGroup) == 0 && layer != LayerKind::kAsym && (layer != LayerKind::kStatic || s.K > kExactK);
    if (tied || conv)
        gemm = gemm_schedule(s.M, s.N, s.K, s.blocks, s.split);
    tied = tied && whole && gemm.sk_tiles == 0;

    const std::array<Best, 3> own = best_tiles(kind, s, loads);
    const float own_other = kMargin * other_us(kind, s, conv ? gemm : lin);
    if (conv && !tied)
        return fastest(own, own_other);
    const std::array<Best, 3> y = kind == layer ? own : best_tiles(layer, s, loads);
    const float y_other = kind == layer ? own_other : kMargin * other_us(layer, s, lin);
    bool open[3];
    for (int c = 0; c < 3; ++c)
        open[c] = y[c].us < y_other;
    auto shared_with = [&](LayerKind k, const GemmSchedule& sch) {
        const std::array<Best, 3> b = k == kind ? own : best_tiles(k, s, loads);
        const float limit = k == kind ? own_other : kMargin * other_us(k, s, sch);
        for (int c = 0; c < 3; ++c)
            open[c] = open[c] && b[c].us < limit;
    };
    if (layer == LayerKind::kLinear && s.N % kGroup == 0)
        shared_with(LayerKind::kQuantized, lin);
    if (tied)
        shared_with(gathered, gemm);
    int order = whole ? 0 : -1;                  // the other kernel's
    float best = whole ? std::min(y[0].us, y_other) : y_other;
    for (int c = whole ? 1 : 0; c < 3; ++c)
        if (open[c] && y[c].us < best) {
            best = y[c].us;
            order = c;
        }
    if (order < 0 || (order == 0 && whole && own[0].us >= own_other))
        return {0, 0};
    return own[order].w;
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

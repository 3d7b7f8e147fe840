// The wide linear kernel (w4a4_wide_kernel.h): the rule that picks it and its
// tile height, and the per-group launches (bf16 or quantized output).
#include "w4a4_wide_kernel.h"

namespace quartz {
namespace {

// Launch times in microseconds, fitted (relative least squares over 30 shapes
// of 220 to 18432 rows, the wide kernel at every tile height; residuals 2-4 %,
// static 3-6 %), with groups rounded up to even for the wide kernel:
//   wide           c + rounds (groups (g0 + g1 TR) + t0 + t1 TR) + load groups TR u
//   whole tiles    c + rounds (groups g + t) + load groups u
//   split          c + load groups gs + ts,  with fewer tiles than workgroups
//                  c + (groups per workgroup) gs + 8 + 0.14 tiles
// where load = tiles / compute units; its terms are what a busier device costs
// in clock.  What they say: a tile row of 7 x 32 costs 0.99 us a group against
// 2 x 0.61 for the 256 rows of two w4a4_linear tiles (static 0.53 against 2 x
// 0.35); tiles of 4 x 32 rows lose that (0.67 against 0.61), and a split launch
// pays about 20 us for exchanging partial sums.  So the wide kernel takes
// shapes for which some height fills whole rounds of the device (4608 rows: 7
// x 32, 98 % full; 4608 x 3072 -> 9216: 153 us against 173) and w4a4_linear
// the ones with too few tiles, or with 128-row tiles that fill a round (4096
// x 4608 -> 1152: 47 us against 50).  Over the 30 shapes the choice is within
// 0.5 % of the better kernel's best height (geometric mean) and never slower
// than w4a4_linear; closer than 3 % it stays with the latter.
struct WideCost {
    float c, g0, g1, t0, t1, u;
    int max_tr;
};
struct LinearCost {
    float c, g, gs, t, ts, u;
};
struct Costs {
    WideCost wide;
    LinearCost lin;
};
// the asymmetric mode's zero-point operands leave no registers for 8 row tiles
// (20 values spill around every group: 98 us against 69 at 7 x 32 rows, 4608 x
// 3072 -> 3072)
constexpr Costs kCosts[4] = {
    {{4.35f, 0.244f, 0.080f, -0.11f, 0.43f, 0.026f, 8}, {5.84f, 0.432f, 0.596f, 1.89f, 18.2f, 0.176f}},   // bf16 output
    {{3.83f, 0.237f, 0.087f, -0.33f, 1.36f, 0.016f, 8}, {5.13f, 0.485f, 0.626f, 4.62f, 21.3f, 0.110f}},   // quantized
    {{4.43f, 0.232f, 0.022f, 0.05f, 0.46f, 0.021f, 8}, {5.46f, 0.208f, 0.355f, 2.48f, 17.9f, 0.143f}},    // static
    {{4.50f, 0.235f, 0.116f, -0.07f, 0.43f, 0.025f, 7}, {5.89f, 0.606f, 0.719f, 1.96f, 19.7f, 0.192f}},   // asymmetric
};
constexpr float kMargin = 0.97f;

}  // namespace

int wide_row_tiles(GemmLaunch& a, WideMode mode)
{
    const int64_t M = a.M, N = a.N, G = a.K / kGroup;
    const int64_t panels = (N + kPanel - 1) / kPanel;
    // the kernel's offsets are 32-bit, and every array's range ends below the
    // offset that marks a lane as outside (2^31)
    constexpr int64_t kMost = int64_t(1) << 30;
    if (M * G * 32 > kMost || panels * G * kChunkBytes > kMost || N * G * 2 > kMost || a.ldy * 2 * kWideMaxRows > kMost)
        return 0;
    const int64_t blocks = device_compute_units();
    const int64_t tiles_n = (N + WBN - 1) / WBN;
    // a quantized output equals quantizing the bf16 output bit for bit, so
    // where w4a4_linear would split (another order of the fp32 sums) the two
    // modes decide alike
    const bool split = a.sch.sk_tiles > 0;
    const Costs& k = kCosts[split && mode == WideMode::kQuantized ? (int)WideMode::kPlain : (int)mode];
    auto rounds = [&](int64_t tiles) { return (float)((tiles + blocks - 1) / blocks); };
    auto load = [&](int64_t tiles) { return (float)tiles / (float)blocks; };
    const int64_t lin_tiles = (M + 127) / 128 * tiles_n;
    const float groups = (float)G, steps = (float)((G + 1) / 2 * 2);
    float best;
    if (!split)
        best = k.lin.c + rounds(lin_tiles) * (groups * k.lin.g + k.lin.t) + load(lin_tiles) * groups * k.lin.u;
    else if (lin_tiles > blocks)
        best = k.lin.c + load(lin_tiles) * groups * k.lin.gs + k.lin.ts;
    else
        best = k.lin.c + (float)a.sch.sk_q * k.lin.gs + 8.0f + 0.14f * (float)lin_tiles;
    best *= kMargin;
    int tr = 0;
    for (int t = kWideMinTR; t <= k.wide.max_tr; ++t) {
        const int64_t tiles = (M + 32 * t - 1) / (32 * t) * tiles_n;
        const float us = k.wide.c + rounds(tiles) * (steps * (k.wide.g0 + k.wide.g1 * (float)t) + k.wide.t0 + k.wide.t1 * (float)t) +
                         load(tiles) * steps * (float)t * k.wide.u;
        if (us < best && tiles <= kMaxGemmTiles / 2) {
            best = us;
            tr = t;
        }
    }
    if (tr > 0)
        a.sch = gemm_schedule_tiles(M, N, a.K, (int)blocks, false, 32 * tr, WBN);
    return tr;
}

hipError_t launch_wide(const GemmLaunch& a, int tr, hipStream_t stream)
{
    return a.qout.codes ? launch_wide_mode<false, true>(a, tr, stream)
                        : launch_wide_mode<false, false>(a, tr, stream);
}

}  // namespace quartz

// The W4A4 linear layer in tall tiles or by teams of waves: every mode of
// w4a4_linear_kernel.h (per-group with a bf16 or quantized output, the LDM
// setting, the asymmetric mode) and the 3 x 3 convolution as an implicit GEMM.
// A tile is always whole, no workspace.  With one team the arithmetic and its
// order (each output's 64-groups in ascending order) are w4a4_linear_kernel's
// unsplit ones, and the results equal them bit for bit.
//
// What bounds these layers is the issue of vector instructions next to the
// MFMAs: on this chip a wave-slot of one 32 x 32 tile costs about half of its
// MFMA cycles (96 with the scale tile, 64 without) plus 3.4 cycles per vector
// instruction (microbenchmark, two waves per SIMD), and with every compute
// unit busy the clock falls from 2.4 to 2.0 GHz.  (Counters, 4608 x 12288 ->
// 3072: MFMAs in 56 % of the cycles, vector instructions in 63 %, one of them or
// both in 83 %; static 57, 46 and 79 %.)  So the layout minimises instructions
// per output:
//  * One workgroup of 8 waves, two per SIMD with 256 registers each, owns a
//    tile of TR x 32 rows (TR = 4 to 8) by 256 columns: each wave all rows of
//    its own 32 columns (WN = 8, one team).  A weight word is then decoded
//    once per tile (the 64 x 64 waves of w4a4_linear decode it twice) and an
//    activation once per 256 columns and up to 256 rows.  There are no decode
//    waves: each wave stages 32 rows of the group two ahead between its MFMAs,
//    and its weight words and scales go from memory to its registers without
//    LDS.  Per group and 256 x 32 outputs 197 vector instructions (counted,
//    epilogue included, 4608 x 12288 -> 3072; 128 of them the dequantization
//    FMAs) against 224 in w4a4_linear.
//  * TR is picked per launch (wide_shape) so that the tiles fill whole
//    rounds of the device: 4608 rows are 21 tiles of 224, and with 12, 36 or
//    48 column tiles 98 % of one, three or four rounds.
//  * Fewer tiles than compute units are made smaller instead, and their groups
//    shared: with WN = 4 (TR 2 to 4) or WN = 2 (TR = 2) the 8 / WN teams of WN
//    waves take the groups of a tile in turn, each staging its own rows, and
//    add their sums through LDS at the end (in the order of the teams, each row
//    tile by the team that stores it).  The device is filled without a trip
//    through memory and its synchronization, 10 to 20 us in w4a4_linear.
//  * Addresses cost one scalar add per array and group: one buffer range over
//    each whole array, a constant lane offset and one scalar offset (both are
//    covered by the range check).
//  * Four LDS stages of activations, two rounds of two groups, one barrier a
//    round; the rows of a round are staged during the one before it, from
//    loads issued two groups earlier.
// Measured against w4a4_linear, launch only: 4608 x 3072 -> 9216 153 us
// (173), static 89 (119), asymmetric 202 (207); 4608 x 12288 -> 3072 208 (226),
// static 106 (131); 3400 x 1280 -> 5120 39 (50), static 26 (43); two teams:
// 1024 x 3072 -> 3072 22.0 (39.1), 4096 x 5760 -> 640 34 (41), static 23 (32),
// as a convolution 37 (44 in w4a4_gemm), static 26 (41); four: 333 x 2048 ->
// 1000 8.2 (20.4), 256 x 1152 -> 1152 7.0 (15.4).
// Tried and dropped: two LDS stages with 64-column waves (2 x 4 waves of 128 x
// 64, weights decoded twice: 5 % slower), a barrier every group (3 %), the
// product transposed so that a lane holds consecutive columns (its stores
// without LDS reach 32 bytes of a row each: 4-7 % slower).
#pragma once

#include "w4a4_gemm_kernel.h"

namespace quartz {
namespace {

constexpr int kWideWaves = 8;
constexpr int kWideThreads = 64 * kWideWaves;
constexpr int kWideStages = 4;

// STATIC, QOUT, ASYM: as in w4a4_linear_kernel; CONV: the rows are gathered
// from the feature map (ConvGeom).  tiles: output tiles, walked
// b, b + gridDim.x, ... by workgroup b.
template <int GS, int TR, int WN, bool STATIC, bool QOUT, bool ASYM, bool CONV>
__global__ __launch_bounds__(kWideThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void w4a4_wide_kernel(
    const uint8_t* __restrict__ codes, const uint8_t* __restrict__ flags,
    const uint16_t* __restrict__ scales, const uint8_t* __restrict__ w_packed,
    const uint16_t* __restrict__ bias, uint16_t* __restrict__ y, int64_t M, int64_t N, int64_t K,
    int64_t ldy, int32_t tiles, int32_t tiles_n, float act_scale, bool gelu, QuantOut qout,
    const int8_t* __restrict__ zeros, const int16_t* __restrict__ wsums, ConvGeom conv)
{
    constexpr int KS = kWideWaves / WN;          // teams, which share the groups in turn
    constexpr int BMW = TR * 32, BNW = WN * 32;  // tile rows and columns
    static_assert(TR <= WN, "a team stages its own rows");
    static_assert(!QOUT || WN % 2 == 0, "quantized output in groups of 64 columns");
    constexpr int kAPlane = WN * 32 * 32;        // of one team
    constexpr int kTeamA = 2 * kAPlane;
    constexpr int kAStage = KS * kTeamA;
    constexpr int kSStage = 256 * 4;
    constexpr int kS0 = kWideStages * kAStage;
    constexpr int kZ0 = kS0 + kWideStages * kSStage;
    constexpr int kT0 = kZ0 + (ASYM ? kWideStages * kSStage : 0);
    __shared__ __attribute__((aligned(16))) uint8_t lds[kT0 + kWideWaves * kTransposeBytes];
    uint8_t* const Ts = lds + kT0;

    constexpr int FB = 64 / GS;                  // flag bytes per (group, row)
    const int tid = threadIdx.x;
    const int uwave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = (int)(K / 64);
    const uint32_t panels = (uint32_t)((N + kPanel - 1) / kPanel);
    const int lane = tid & 63, l32 = tid & 31, khalf = (tid >> 5) & 1;
    const int team = uwave / WN, wn = uwave % WN;

    // ---------------------------------------------------------------- fetch
    // Rows past M and columns past the packed panels read their neighbours or,
    // past the end of an array, zero; they only feed outputs that are never
    // stored.  The fetch runs two rounds (of two groups) ahead of the
    // multiplication for the rows and one to two for the weights, across
    // tile boundaries; past the last tile it fetches groups nobody uses.
    const int32_t stride = (int32_t)gridDim.x;
    const int dm = stride / tiles_n, dn = stride - dm * tiles_n;
    int f_tile = (int)blockIdx.x, f_tm = f_tile / tiles_n, f_tn = f_tile - f_tm * tiles_n;
    const int rounds = (G + 2 * KS - 1) / (2 * KS);
    int f_round = 0, f_g = 0;                    // the fetched round of the tile, and its first group for this team
    const uint32_t rowsG = (uint32_t)(M * (CONV ? conv.cg : G));
    const Rsrc ra = make_rsrc(codes, rowsG * 32u), rf = make_rsrc(flags, rowsG * (uint32_t)FB);
    const Rsrc rs = make_rsrc(scales, STATIC ? 0u : rowsG * 2u);
    const Rsrc rb = make_rsrc(w_packed, panels * (uint32_t)G * kChunkBytes);
    const Rsrc rw = make_rsrc(wsums, ASYM ? (uint32_t)(N * G) * 2u : 0u);
    const Rsrc rz = make_rsrc(zeros, ASYM ? rowsG : 0u);
    const uint32_t uM = (uint32_t)M;
    uint32_t f_r = 0;                            // (group, row) index of the wave's first staged row
    uint32_t f_w = 0, f_w2 = 0;                  // byte offset of the wave's weight columns; the fetched round's
    uint32_t f_z = 0, f_z2 = 0;
    // Groups past the tile's last one (an odd count, or fewer than the teams
    // take a round) multiply zeros: the rows, scales and sums of group G and
    // after lie past the end of their arrays, and the weights, whose next
    // panel follows, get an offset past theirs.  (Zero activations alone would
    // not do: an infinite weight scale there would make a NaN of them.)
    constexpr uint32_t kPast = 0x40000000u;      // past the end of every array
    auto weights_at = [&](int u) { return f_g + u * KS < G ? f_w2 + (uint32_t)(u * KS) * kChunkBytes : kPast; };
    // CONV: this lane's output pixel, and its row and column in the image
    int c_m = 0, c_h = 0, c_w = 0;
    auto set_offsets = [&] {
        const uint32_t col0 = (uint32_t)f_tn * BNW + (uint32_t)wn * 32u;
        f_r = (uint32_t)team * uM + (uint32_t)f_tm * BMW + (uint32_t)wn * 32u;
        f_w2 = ((col0 >> 6) * (uint32_t)G + (uint32_t)team) * kChunkBytes;
        if constexpr (ASYM)
            f_z2 = ((uint32_t)team * (uint32_t)N + col0) * 2u;
        f_round = 0;
        f_g = team;
        if constexpr (CONV) {
            c_m = f_tm * BMW + wn * 32 + (lane >> 1);
            const uint32_t q = (uint32_t)c_m / (uint32_t)conv.W;
            c_w = c_m - (int)q * conv.W;
            c_h = (int)(q % (uint32_t)conv.H);
        }
    };
    auto next_round = [&] {
        ++f_round;
        f_g += 2 * KS;
        f_w2 += 2 * KS * kChunkBytes;
        if constexpr (ASYM)
            f_z2 += 4 * KS * (uint32_t)N;
        if (f_round == rounds && f_tile + stride < tiles) {
            f_tile += stride;
            f_tm += dm;
            f_tn += dn;
            if (f_tn >= tiles_n) {
                f_tn -= tiles_n;
                ++f_tm;
            }
            set_offsets();
        }
    };
    struct RawA {
        uint4 a;
        typename std::conditional<GS == 8, uint32_t, typename std::conditional<GS == 16, uint16_t, uint8_t>::type>::type f;
        uint16_t s;                              // (raw 8- and 16-bit values: widened in place they would be
        uint8_t z;                               // widened, and waited for, where they are loaded)
    };
    struct RawW {
        uint4 w;
        uint16_t s, sum;
    };
    constexpr uint32_t kOut = 0x80000000u;       // outside every range
    // rows: this lane stages half lane & 1 of row lane >> 1 of the wave's 32
    // rows (waves past the tile's rows stage zeros nobody reads)
    const bool stager = wn < TR;
    const uint32_t offa = stager ? (uint32_t)lane * 16u : kOut;
    const uint32_t offf = !stager ? kOut : GS == 8 ? (uint32_t)lane * 4u : GS == 16 ? (uint32_t)lane * 2u : GS == 32 ? (uint32_t)lane : (uint32_t)lane >> 1;
    const uint32_t offs = stager ? (uint32_t)(lane >> 1) * 2u : kOut;
    const uint32_t offz = stager ? (uint32_t)(lane >> 1) : kOut;
    // columns: lane l32 of k half khalf; the scales' upper half-wave reads zero
    const uint32_t offw = (uint32_t)(wn & 1) * 1024u + (uint32_t)l32 * 32u + (uint32_t)khalf * 16u;
    const uint32_t offws = khalf ? kOut : (uint32_t)(kChunkCodeBytes + (wn & 1) * 64 + l32 * 2);
    const uint32_t offsum = khalf ? kOut : (uint32_t)l32 * 2u;
    auto fetch_a = [&](RawA& r, int u) {
        if constexpr (CONV) {
            // the channel block's plane at the pixel that the group's tap
            // shifts this lane's output pixel to, nothing outside the image
            const uint32_t g = (uint32_t)(f_g + u * KS);
            const uint32_t tap = conv.cg == 1 ? g : __umulhi(g, conv.div_magic);
            const int dh = (int)(tap / 3u) - 1, dw = (int)(tap % 3u) - 1;
            const uint32_t plane = (g - tap * (uint32_t)conv.cg) * uM;
            const bool in = stager & ((uint32_t)c_m < uM) & ((uint32_t)(c_h + dh) < (uint32_t)conv.H) &
                            ((uint32_t)(c_w + dw) < (uint32_t)conv.W) & (tap < 9u);
            const uint32_t row = (uint32_t)(c_m + dh * conv.W + dw), half = (uint32_t)lane & 1u;
            r.a = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                                ra, (int)(in ? row * 32u + half * 16u : kOut), (int)(plane * 32u), 0));
            const int fo = (int)(in ? row * (uint32_t)FB + (GS < 64 ? half * (uint32_t)(FB / 2) : 0u) : kOut);
            const int fp = (int)(plane * (uint32_t)FB);
            if constexpr (GS == 8)
                r.f = __builtin_amdgcn_raw_buffer_load_b32(rf, fo, fp, 0);
            else if constexpr (GS == 16)
                r.f = __builtin_amdgcn_raw_buffer_load_b16(rf, fo, fp, 0);
            else
                r.f = __builtin_amdgcn_raw_buffer_load_b8(rf, fo, fp, 0);
            if constexpr (!STATIC)
                r.s = __builtin_amdgcn_raw_buffer_load_b16(rs, (int)(in ? row * 2u : kOut), (int)(plane * 2u), 0);
            return;
        }
        r.a = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(ra, (int)offa, (int)(f_r * 32u), 0));
        if constexpr (GS == 8)
            r.f = __builtin_amdgcn_raw_buffer_load_b32(rf, (int)offf, (int)(f_r * 8u), 0);
        else if constexpr (GS == 16)
            r.f = __builtin_amdgcn_raw_buffer_load_b16(rf, (int)offf, (int)(f_r * 4u), 0);
        else
            r.f = __builtin_amdgcn_raw_buffer_load_b8(rf, (int)offf, (int)(f_r * (uint32_t)FB), 0);
        if constexpr (!STATIC)
            r.s = __builtin_amdgcn_raw_buffer_load_b16(rs, (int)offs, (int)(f_r * 2u), 0);
        if constexpr (ASYM)
            r.z = __builtin_amdgcn_raw_buffer_load_b8(rz, (int)offz, (int)f_r, 0);
        f_r += KS * uM;
    };
    auto fetch_w = [&](RawW& r) {
        r.w = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rb, (int)offw, (int)f_w, 0));
        if constexpr (!STATIC)
            r.s = __builtin_amdgcn_raw_buffer_load_b16(rb, (int)offws, (int)f_w, 0);
        if constexpr (ASYM)
            r.sum = __builtin_amdgcn_raw_buffer_load_b16(rw, (int)offsum, (int)f_z, 0);
        if constexpr (ASYM)
            f_z += 2u * KS * (uint32_t)N;
    };

    // 16-byte chunk p of k half h of row r lives in plane p at
    // r * 32 + (h ^ r2 ^ r3) * 16
    auto a_slot = [](int r, int h) { return (uint32_t)(r * 32 + ((h ^ (r >> 2) ^ (r >> 3)) & 1) * 16); };
    // LDS addresses; the ones that are written run two stages ahead, and each
    // moves by two stages a round
    uint32_t a_st = (uint32_t)(team * kTeamA) + a_slot(wn * 32 + (lane >> 1), lane & 1);
    uint32_t s_st = (uint32_t)(kS0 + (tid >> 1) * 4);
    uint32_t a_rd = (uint32_t)(team * kTeamA) + a_slot(l32, khalf);
    uint32_t s_rd = (uint32_t)(kS0 + team * WN * 128 + l32 * 4);
    auto word = [&](const RawA& r, int w) {
        const uint32_t a[4] = {r.a.x, r.a.y, r.a.z, r.a.w};
        constexpr int kWordsPerFlag = GS / 8;
        Fp8Table t;
        switch (w / kWordsPerFlag) {
        case 0: t = fp8_table_raw<0>(r.f, 0u); break;
        case 1: t = fp8_table_raw<1>(r.f, 0u); break;
        case 2: t = fp8_table_raw<2>(r.f, 0u); break;
        default: t = fp8_table_raw<3>(r.f, 0u); break;
        }
        return decode_nibbles_fp8(a[w], t);
    };
    uint2 o0;
    auto stage_part = [&](const RawA& r, int st, int q) {
        const uint2 o1 = word(r, q);
        if (q & 1)
            *reinterpret_cast<uint4*>(lds + st * kAStage + (q >> 1) * kAPlane + a_st) = make_uint4(o0.x, o0.y, o1.x, o1.y);
        o0 = o1;
        if (q == 3) {
            if constexpr (!STATIC)
                *reinterpret_cast<uint32_t*>(lds + st * kSStage + s_st) = r.s;
            if constexpr (ASYM)                  // -z, exact in fp16
                *reinterpret_cast<uint32_t*>(lds + (kZ0 - kS0) + st * kSStage + s_st) =
                    __builtin_bit_cast(uint16_t, (_Float16)(short)(-(int)(int8_t)r.z));
        }
    };

    // ---------------------------------------------------------------- math
    typedef int v2i __attribute__((ext_vector_type(2)));
    typedef _Float16 v4h __attribute__((ext_vector_type(4)));
    v16f acc[TR];
    v8i af[2], bf;
    v2i sa_op[2], za_op[2], sw_op, ws_op;
    const v16f zero = {};
    // rows 32 i .. of the group in stage st (relative to a_rd), buffer p
    auto load_a = [&](int p, int i, int st) {
        const uint8_t* src = lds + st * kAStage + a_rd + i * 1024;
        const uint4 l = *reinterpret_cast<const uint4*>(src);
        const uint4 h = *reinterpret_cast<const uint4*>(src + kAPlane);
        af[p] = v8i{(int)l.x, (int)l.y, (int)l.z, (int)l.w, (int)h.x, (int)h.y, (int)h.z, (int)h.w};
        if constexpr (!STATIC)
            sa_op[p][0] = *reinterpret_cast<const int*>(lds + st * kSStage + s_rd + i * 128);
        if constexpr (ASYM)
            za_op[p][0] = *reinterpret_cast<const int*>(lds + (kZ0 - kS0) + st * kSStage + s_rd + i * 128);
    };
    auto decode_w = [&](const RawW& r) {
        const uint2 w0 = decode_weight_fp8(r.w.x), w1 = decode_weight_fp8(r.w.y);
        const uint2 w2 = decode_weight_fp8(r.w.z), w3 = decode_weight_fp8(r.w.w);
        bf = v8i{(int)w0.x, (int)w0.y, (int)w1.x, (int)w1.y, (int)w2.x, (int)w2.y, (int)w3.x, (int)w3.y};
        asm volatile("" : "+v"(bf));
        if constexpr (!STATIC)
            sw_op[0] = r.s;
        if constexpr (ASYM)                      // W * 2^-9 (the unit of the weight operands), exact
            ws_op[0] = __builtin_bit_cast(uint16_t, (_Float16)((_Float16)(short)r.sum * (_Float16)(1.0f / kWeightUnitInv)));
    };
    auto scale_tile = [&](int p) {
        return __builtin_amdgcn_mfma_f32_32x32x8f16(__builtin_bit_cast(v4h, sa_op[p]),
                                                    __builtin_bit_cast(v4h, sw_op), zero, 0, 0, 0);
    };
    auto mfma_p = [&](int p) {
        v16f c = zero;
        if constexpr (ASYM)
            c = __builtin_amdgcn_mfma_f32_32x32x8f16(__builtin_bit_cast(v4h, za_op[p]),
                                                     __builtin_bit_cast(v4h, ws_op), zero, 0, 0, 0);
        return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(af[p], bf, c, 0, 0, 0, 0, 0, 0);
    };
    auto fma_tile = [&](v16f& a, const v16f& p, const v16f& s) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
            a[r] = fmaf(p[r], s[r], a[r]);
        asm volatile("" : "+v"(a));              // not sunk out of its slot
    };
    auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    RawA rawa[2];
    RawW raww[2];
    v16f pc, sc;
    int c_tm = f_tm, c_tn = f_tn;

    // Group u of a round (2r + u): multiply it (LDS stage a_rd + u), stage
    // group 2r + u + 2, fetch the rows of 2r + u + 4 and the weights of
    // 2r + u + 3.
    auto step = [&](auto uc) {
        constexpr int u = decltype(uc)::value;
        constexpr int D = STATIC ? 1 : 0;        // the products of STATIC are issued one slot later
        // rows are read kAhead slots before their product, into the buffer that
        // the row two before them has left; the first read of the next round
        // comes after the round's one barrier: the rows staged in both of its
        // steps are then visible, and the reads of this round's rows done
        constexpr int kAhead = TR > 2 ? 3 : 2;
        constexpr int kFirst = TR - kAhead + D;  // the slot of that read
        constexpr int kSlots = kFirst < 1 ? 1 : kFirst < 4 ? kFirst : 4;   // slots the staging is spread over
#pragma unroll
        for (int t = 0; t < TR; ++t) {
            v16f pn;
            if constexpr (STATIC) {
                acc[t] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(af[(u * TR + t) & 1], bf, acc[t], 0, 0, 0, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            } else {
                pn = mfma_p((u * TR + t + 1) & 1);
                __builtin_amdgcn_sched_barrier(0);
                fma_tile(acc[t], pc, sc);
                __builtin_amdgcn_sched_barrier(0);
                sc = scale_tile((u * TR + t + 1) & 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            auto stage_slot = [&] {
#pragma unroll
                for (int w = 0; w < 4; ++w)
                    if (t == (w * kSlots) / 4)
                        stage_part(rawa[u], u, w);
            };
            if (t == kFirst) {
                if (kFirst == 0)
                    stage_slot();
                if (u == 1) {
                    barrier();
                    a_rd ^= 2 * kAStage;
                    s_rd = kS0 + ((s_rd - kS0) ^ (2 * kSStage));
                }
            }
            constexpr int ahead = kAhead - D;
            if (t + ahead < TR)
                load_a((u * TR + t + ahead) & 1, t + ahead, u);
            else
                load_a((u * TR + t + ahead) & 1, t + ahead - TR, 1 - u);
            if (kFirst > 0 || t > 0)
                stage_slot();
            if (t == (3 * kSlots) / 4)
                fetch_a(rawa[u], u);
            if (t == TR - 2 + D) {
                decode_w(raww[1 - u]);
                fetch_w(raww[1 - u]);
            }
            __builtin_amdgcn_sched_barrier(0);
            pc = pn;
        }
    };

    // ---------------------------------------------------------------- output
    // Lane l32 holds column l32 of the wave's 32, rows 32 i + 8 (r / 4) +
    // 4 khalf + r % 4 of the tile in register r of acc[i].
    uint16_t bias_bits = 0, cscale_bits = 0;
    auto load_columns = [&] {
        const int64_t col0 = (int64_t)c_tn * BNW + wn * 32;
        const Rsrc rbias = make_rsrc(bias, bias ? (uint32_t)(N * 2) : 0u);
        bias_bits = __builtin_amdgcn_raw_buffer_load_b16(rbias, (int)((col0 + l32) * 2), 0, 0);
        if constexpr (STATIC)
            // the channel scales, from the scale slot of group 0 of the panel
            cscale_bits = __builtin_amdgcn_raw_buffer_load_b16(
                rb, (int)((uint32_t)(col0 >> 6) * (uint32_t)G * kChunkBytes + kChunkCodeBytes + (wn & 1) * 64 + l32 * 2), 0, 0);
    };
    typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef float v4f __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) v4f lds_v4f;
    // Teams: each tile's partial sums go through LDS to the team that owns it
    // (row tile i: team i % KS), which adds them in team order.
    constexpr int TL = (TR + KS - 1) / KS;       // row tiles a wave writes out
    v16f red[KS > 1 ? TL : 1];
    auto reduce_teams = [&] {
        auto slot = [&](int i, int t) {
            const int owner = i % KS, rank = t < owner ? t : t - 1;
            return (lds_u8*)(Ts + ((i * (KS - 1) + rank) * WN + wn) * 4096 + lane * 16);
        };
#pragma unroll
        for (int i = 0; i < TR; ++i)
            if (team != i % KS)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *(lds_v4f*)(slot(i, team) + q * 1024) = v4f{acc[i][4 * q], acc[i][4 * q + 1], acc[i][4 * q + 2], acc[i][4 * q + 3]};
        barrier();
#pragma unroll
        for (int i = 0; i < TR; ++i)
            if (team == i % KS) {
                v16f sum;
#pragma unroll
                for (int t = 0; t < KS; ++t)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        v4f x = {acc[i][4 * q], acc[i][4 * q + 1], acc[i][4 * q + 2], acc[i][4 * q + 3]};
                        if (t != i % KS)
                            x = *(lds_v4f*)(slot(i, t) + q * 1024);
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            sum[4 * q + e] = t == 0 ? x[e] : sum[4 * q + e] + x[e];
                    }
                red[i / KS] = sum;
            }
        barrier();
    };
    auto store_tile = [&](auto gelu_c) {
        v16f (&out)[KS > 1 ? TL : TR] = [&]() -> v16f (&)[KS > 1 ? TL : TR] {   // out[j]: row tile j KS + team
            if constexpr (KS > 1)
                return red;
            else
                return acc;
        }();
        // opaque copies, so that nothing here is computed before the branches
        // above (or before the tile loop) and kept in registers until now
        int lane_ = lane;
        asm volatile("" : "+v"(lane_));
        const int l32 = lane_ & 31, khalf = lane_ >> 5;
        float b = __uint_as_float((uint32_t)bias_bits << 16);
        // STATIC: act_scale * s_w[n] times the 2^9 of the weight unit
        const float cs = STATIC ? act_scale * (float)__builtin_bit_cast(_Float16, cscale_bits) * kWeightUnitInv : kWeightUnitInv;
        auto fresh = [&] { asm volatile("" : "+v"(b)); };
        auto pack2 = [&](int j, int r, auto gelu_c2) {   // rows r, r + 1
            float v0 = fmaf(out[j][r], cs, b), v1 = fmaf(out[j][r + 1], cs, b);
            if constexpr (decltype(gelu_c2)::value) {
                v0 = gelu_tanh(v0);
                v1 = gelu_tanh(v1);
            }
            const f2 pair = {v0, v1};
            return __builtin_bit_cast(uint32_t, __builtin_convertvector(pair, bf2));
        };
        const int64_t m0 = (int64_t)c_tm * BMW;
        const int64_t m_end = min(M, m0 + BMW);
        const int64_t col_base = (int64_t)c_tn * BNW + wn * 32;
        if constexpr (QOUT) {
            // 128 rows at a time: the waves write their columns into regions
            // of 64 rows x 64 columns (quantize_rows_out's layout), then one
            // wave takes each region
#pragma unroll
            for (int h = 0; h < (TR + 3) / 4; ++h) {
                auto write = [&](auto g) {
                    fresh();
#pragma unroll
                    for (int j = KS > 1 ? 0 : 4 * h; j < (KS > 1 ? TL : min(4 * h + 4, TR)); ++j) {
                        const int i = j * KS + team;
                        if (KS > 1 && i >= TR)
                            continue;
                        lds_u8* const tb = (lds_u8*)(Ts + ((wn >> 1) * 2 + ((i >> 1) & 1)) * kTransposeBytes + (i & 1) * 4096);
#pragma unroll
                        for (int r = 0; r < 16; r += 2) {
                            const uint32_t pk = pack2(j, r, g);
                            const int row = 8 * (r >> 2) + (r & 3);                  // + 4 khalf, in the 32 rows
                            const uint32_t cb = (uint32_t)((wn & 1) * 64 + l32 * 2);
                            const uint32_t x = (uint32_t)((row >> 1) & 7) << 4;      // the chunk swizzle of rows row, row + 1
                            const uint32_t at = (uint32_t)(row * 128 + khalf * 512) + ((cb ^ x) ^ (uint32_t)(khalf * 32));
                            *(lds_u16*)(tb + at) = (uint16_t)pk;
                            *(lds_u16*)(tb + at + 128) = (uint16_t)(pk >> 16);
                        }
                    }
                };
                if (col_base < N) {
                    if (gelu)
                        write(std::integral_constant<bool, true>());
                    else
                        write(std::integral_constant<bool, false>());
                }
                barrier();
                if (uwave < WN)
                    quantize_rows_out((lds_u8*)(Ts + uwave * kTransposeBytes), lane_, m0 + h * 128 + (uwave & 1) * 64,
                                      (int64_t)c_tn * BNW + (uwave >> 1) * 64, m_end, M, N, qout);
                barrier();
            }
            return;
        }
        if (col_base >= N)
            return;                              // wave-uniform
        const uint32_t row_bytes = (uint32_t)ldy * 2u;
        // the 32 rows of row tile i: rows past M fall outside the range
        auto tile_range = [&](int i) {
            const int64_t row0 = m0 + i * 32;
            const int64_t rows = max((int64_t)0, min(m_end - row0, (int64_t)32));
            return make_rsrc(y + row0 * ldy + col_base, (uint32_t)rows * row_bytes);
        };
        if (col_base + 32 <= N && ((reinterpret_cast<uintptr_t>(y) | (uint64_t)row_bytes) & 15u) == 0) {
            // through the wave's own LDS region, 4 row tiles at a time: line
            // 16 j + r holds register r of row tile j (two 64-byte row
            // segments, one per half-wave)
            lds_u8* const tw = (lds_u8*)(Ts + uwave * kTransposeBytes);
            fresh();
#pragma unroll
            for (int h = 0; h < (TL + 3) / 4; ++h) {
#pragma unroll
                for (int j = 4 * h; j < min(4 * h + 4, TL); ++j)
#pragma unroll
                    for (int r = 0; r < 16; r += 2) {
                        const uint32_t pk = pack2(j, r, gelu_c);
                        lds_u8* const at = tw + ((j - 4 * h) * 16 + r) * 128 + lane_ * 2;
                        *(lds_u16*)at = (uint16_t)pk;
                        *(lds_u16*)(at + 128) = (uint16_t)(pk >> 16);
                    }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
                for (int q = 0; q < 2 * min(4, TL - 4 * h); ++q) {
                    const int i = (4 * h + q / 2) * KS + team;
                    if (KS > 1 && i >= TR)
                        continue;
                    const Rsrc out_r = tile_range(i);
                    const uint32_t line = (uint32_t)(8 * (q & 1)) + ((uint32_t)lane_ >> 3), c = (uint32_t)lane_ & 7u;
                    const v4u v = *(lds_v4u*)(tw + (q / 2) * 2048u + line * 128u + c * 16u);
                    const uint32_t row = (line >> 2) * 8u + (c >> 2) * 4u + (line & 3u);
                    __builtin_amdgcn_raw_buffer_store_b128(v, out_r, (int)(row * row_bytes + (c & 3u) * 16u), 0, 0);
                }
                asm volatile("" ::: "memory");
            }
            return;
        }
        const uint32_t voff = col_base + l32 < N ? (uint32_t)l32 * 2u + (uint32_t)(khalf * 4) * row_bytes : kOut;
        fresh();
#pragma unroll
        for (int j = 0; j < TL; ++j) {
            const int i = j * KS + team;
            if (KS > 1 && i >= TR)
                continue;
            const Rsrc out_r = tile_range(i);
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const uint32_t pk = pack2(j, r, gelu_c);
                const uint32_t row0 = (uint32_t)(8 * (r >> 2) + (r & 3));
                __builtin_amdgcn_raw_buffer_store_b16((uint16_t)pk, out_r, (int)(voff + row0 * row_bytes), 0, 0);
                __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(pk >> 16), out_r, (int)(voff + (row0 + 1) * row_bytes), 0, 0);
            }
        }
    };

    // prologue: groups 0 and 1 staged, the rows of groups 2 and 3 and the
    // weights of groups 1 and 2 in flight (of this team's groups)
    sa_op[0] = sa_op[1] = za_op[0] = za_op[1] = sw_op = ws_op = v2i{0, 0};
    set_offsets();
    f_z = f_z2;
    fetch_a(rawa[0], 0);
    fetch_a(rawa[1], 1);
    f_w = weights_at(0);
    fetch_w(raww[0]);
    f_w = weights_at(1);
    fetch_w(raww[1]);
#pragma unroll
    for (int q = 0; q < 4; ++q)
        stage_part(rawa[0], 0, q);
#pragma unroll
    for (int q = 0; q < 4; ++q)
        stage_part(rawa[1], 1, q);
    a_st ^= 2 * kAStage;
    s_st = kS0 + ((s_st - kS0) ^ (2 * kSStage));
    next_round();
    f_z = f_z2;
    fetch_a(rawa[0], 0);
    fetch_a(rawa[1], 1);
    decode_w(raww[0]);
    f_w = weights_at(0);
    fetch_w(raww[0]);
    barrier();
    for (int tile = (int)blockIdx.x; tile < tiles; tile += stride) {
        load_columns();
#pragma unroll
        for (int i = 0; i < TR; ++i)
            acc[i] = zero;
        load_a(0, 0, 0);
        load_a(1, 1, 0);
        if constexpr (!STATIC) {
            pc = mfma_p(0);
            sc = scale_tile(0);
            if constexpr (TR > 2)
                load_a(0, 2, 0);
        }
        for (int left = rounds; left > 0; --left) {
            f_w = weights_at(1);
            next_round();
            step(std::integral_constant<int, 0>());
            f_w = weights_at(0);
            f_z = f_z2;
            step(std::integral_constant<int, 1>());
            // arrived with the first group's loads: waited for here, not with
            // the fetches in flight at the tile's end
            asm volatile("" : "+v"(bias_bits), "+v"(cscale_bits));
            a_st ^= 2 * kAStage;
            s_st = kS0 + ((s_st - kS0) ^ (2 * kSStage));
        }
        if constexpr (KS > 1)
            reduce_teams();
        if (gelu && !QOUT)                       // (QOUT looks at gelu itself)
            store_tile(std::integral_constant<bool, true>());
        else
            store_tile(std::integral_constant<bool, false>());
        if constexpr (KS > 1)
            barrier();                           // the regions are the next tile's slots
        c_tm += dm;
        c_tn += dn;
        if (c_tn >= tiles_n) {
            c_tn -= tiles_n;
            ++c_tm;
        }
    }
}

template <bool STATIC, bool QOUT, bool ASYM, bool CONV>
hipError_t launch_wide_mode(const GemmLaunch& a, hipStream_t stream)
{
    const WideShape& w = a.wide;
    const GemmSchedule sch = wide_schedule(a);
    const dim3 grid((unsigned)sch.blocks), block(kWideThreads);
    auto go = [&](auto gs, auto tr, auto wn) {
        w4a4_wide_kernel<decltype(gs)::value, decltype(tr)::value, decltype(wn)::value, STATIC, QOUT, ASYM, CONV>
            <<<grid, block, 0, stream>>>(a.codes, a.flags, a.scales, a.w_packed, a.bias, a.y, a.M, a.N,
                                         a.K, a.ldy, sch.sk_first, sch.tiles_n, a.act_scale,
                                         a.epilogue == 1, a.qout, a.zeros, a.wsums, a.conv);
    };
    using std::integral_constant;
    auto with_tile = [&](auto gs) {
        const integral_constant<int, 8> wide;
        const integral_constant<int, 4> half;
        const integral_constant<int, 2> quarter;
        if (w.wn == 2)
            return go(gs, quarter, quarter);
        if (w.wn == 4)
            switch (w.tr) {
            case 2: return go(gs, quarter, half);
            case 3: return go(gs, integral_constant<int, 3>(), half);
            default: return go(gs, half, half);
            }
        switch (w.tr) {
        case 4: return go(gs, half, wide);
        case 5: return go(gs, integral_constant<int, 5>(), wide);
        case 6: return go(gs, integral_constant<int, 6>(), wide);
        case 7: return go(gs, integral_constant<int, 7>(), wide);
        default:
            if constexpr (!ASYM)                 // wide_shape stops at 7 there
                return go(gs, wide, wide);
        }
    };
    switch (a.lzs_group) {
    case 8: with_tile(integral_constant<int, 8>()); break;
    case 16: with_tile(integral_constant<int, 16>()); break;
    case 32: with_tile(integral_constant<int, 32>()); break;
    default: with_tile(integral_constant<int, 64>()); break;
    }
    return hipGetLastError();
}

}  // namespace
}  // namespace quartz

// Fused LZS attention (the attention setting of the hardware appendix,
// Table 8) for head dimensions 64 and 128: the scores never leave registers.
//
// Per head, O = softmax(S) V with S = Q~ K~^T / sqrt(d); Q~, K~ quantized per
// token along d, V~^T per channel along the keys and the binary32 softmax
// output P per query row in 64-key groups, all by Eq. 1 and Eq. 2, and both
// products exact per-group integer products with the fp16 group scales
// applied in fp32 (the same quantities the unfused path materializes).
//
// The quantized P of a 64-key group needs the row's final max and sum (its
// group scale is fp16(max P / 127) of the normalized values), so each query
// row is swept twice:
//   pass 1  S of every 64-key chunk and the sum of exp against a reference
//           near the row's maximum;
//   pass 2  S again, P = exp(S - reference) / sum in binary32, the group scale,
//           Stage-1 codes, FLAG per subgroup and the truncated LZS values
//           d = c 2^FLAG, which go straight into the PV matrix product.
// The codes are rne(e R) with e = exp(S - reference) and R = (1 / sum) (1 / s),
// rounded once (a fused multiply-add) where the unfused path rounds P and P r
// first, so a code can differ from that path's only where P r lies within an
// ulp of a rounding boundary.
// One wave owns 32 queries of one head (or its team's share of their keys);
// the chunks go through LDS, shared by the waves of a block.  The operands
// come from HBM / L2 already decoded to fp8 e4m3 (quantize_operands_kernel:
// every d = c 2^FLAG is exact in e4m3), since every chunk of K~ and V~^T is
// read by all L / 32 query waves of its head and decoding it once is cheaper
// than decoding it L / 32 times.
//
// Layout of the score tiles.  The product runs as S^T = K~ Q~^T on
// v_mfma_f32_32x32x64_f8f6f4 (rows: keys, columns: queries), so lane l holds
// query l % 32 and 16 keys per 32-key tile.  Row rho of key tile t is fed
// with key 32 ((rho >> 2) & 1) + 16 t + 4 (rho >> 3) + (rho & 3) of the
// chunk, which puts keys 32 h + 16 t + r (register r, h = l / 32) in lane l:
// each half-wave holds 32 consecutive keys of every query, so row maxima,
// group maxima and the FLAG subgroups (G_s <= 32) are in-lane reductions and
// a 64-key group takes one exchange between the two half-waves.  The same
// registers, converted to e4m3 and packed in the byte order of the quantized
// V~^T's keys, are the k-slice of the PV product O^T = V~^T P~^T.
#include <algorithm>
#include <cmath>

#include "lzs_device.h"
#include "w4a4_gemm_kernel.h"

namespace quartz {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

// -------------------------------------------------- quantize to fp8 operands
// Q, K (per token along d) and V^T (per channel along the keys) quantized by
// Eq. 1 and Eq. 2 and left as e4m3 values of c 2^FLAG, in one launch: the
// quantizer's codes are decoded in the registers that formed them (word w of a
// group gives bytes 8 w .. 8 w + 7 in the order decode_nibbles_fp8 writes
// them) instead of going through memory as 4-bit codes to a second kernel, and
// three quantizers and three expansions would be six launches (64 us at 32
// heads, L = 4608, d = 128; 20 us at 20 heads, L = 1024, d = 64; this launch 29
// and 6 us).  HBM-bound: 3 bytes in and out per element, 5.9 TB/s there.
//
// A team of 8 lanes takes a group, lane u its elements 8 u .. 8 u + 7; amax: what
// their maximum starts from (a NaN loses to any number: a row whose values are
// all NaN keeps one and saturates its scale, a channel's starts from 0).
template <int GS>
__device__ __forceinline__ uint2 quantize_fp8(const uint4& v, float amax, uint32_t& s16)
{
    constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kMirror = 0x141;   // quad_perm, quad_perm, row_half_mirror
    auto dpp = [](auto c, uint32_t x) {
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(c)::value, 0xF, 0xF, false);
    };
    using std::integral_constant;
    const uint32_t d[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        amax = fmaxf(amax, fabsf(__uint_as_float(d[k] << 16)));
        amax = fmaxf(amax, fabsf(__uint_as_float(d[k] & 0xFFFF0000u)));
    }
    uint32_t m = __float_as_uint(amax);          // (non-negative floats order as their bits)
    m = max(m, dpp(integral_constant<int, kXor1>(), m));
    m = max(m, dpp(integral_constant<int, kXor2>(), m));
    m = max(m, dpp(integral_constant<int, kMirror>(), m));
    const GroupScale gsc = group_scale(__uint_as_float(m));
    s16 = gsc.s16;
    uint32_t p[4];
    mag_pairs8(d, gsc.r, __builtin_amdgcn_ballot_w64(gsc.clamp) != 0, p);
    uint32_t o = pairs_or(p);
    if constexpr (GS >= 16)
        o |= dpp(integral_constant<int, kXor1>(), o);
    if constexpr (GS >= 32)
        o |= dpp(integral_constant<int, kXor2>(), o);
    if constexpr (GS >= 64)
        o |= dpp(integral_constant<int, kMirror>(), o);
    const int fl = lzs_flag(o);
    return decode_nibbles_fp8(lzs_word(p, sign_nibbles(d), fl), fp8_table_raw<0>((uint32_t)fl, 0u));
}

struct AttnOperands {
    const uint16_t *q, *k, *v;                   // bf16 [heads L][d]
    uint8_t *qx, *kx, *vx;                       // e4m3 [heads L][d] twice, [heads d][L]
    uint16_t *qs, *ks, *vs;                      // fp16 [d / 64][heads L] twice, [L / 64][heads d]
};
constexpr int kRowItems = 4;                     // 16-byte pieces per thread and tensor

// The first blocks take 64 keys x 64 channels of V each (through an LDS
// transpose), the others kRowItems 256 pieces of Q or of K.
template <int GS>
__global__ __launch_bounds__(256) void quantize_operands_kernel(AttnOperands a, int64_t heads, int64_t L,
                                                                int64_t d, uint32_t vblocks, uint32_t rblocks)
{
    __shared__ __attribute__((aligned(16))) uint16_t tile[64][64 + 8];
    const int t = threadIdx.x, u = t & 7;
    const uint32_t G = (uint32_t)d / 64, LG = (uint32_t)(L / 64);
    uint32_t b = blockIdx.x;
    if (b < vblocks) {
        const uint32_t cb = b % G, hg = b / G;
        const int64_t h = hg / LG, g = hg % LG;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int key = (t >> 3) + 32 * i;
            const uint4 x = *reinterpret_cast<const uint4*>(a.v + (h * L + g * 64 + key) * d + cb * 64 + 8 * u);
            const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                tile[8 * u + 2 * j][key] = (uint16_t)w[j];
                tile[8 * u + 2 * j + 1][key] = (uint16_t)(w[j] >> 16);
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int ch = (t >> 3) + 32 * i;
            uint32_t s16;
            const uint2 x = quantize_fp8<GS>(*reinterpret_cast<const uint4*>(&tile[ch][8 * u]), 0.0f, s16);
            const int64_t row = h * d + cb * 64 + ch;
            *reinterpret_cast<uint2*>(a.vx + row * L + g * 64 + 8 * u) = x;
            if (u == 0)
                a.vs[g * heads * d + row] = (uint16_t)s16;
        }
        return;
    }
    b -= vblocks;
    const bool is_k = b >= rblocks;
    b -= is_k ? rblocks : 0;
    const uint4* const src = reinterpret_cast<const uint4*>(is_k ? a.k : a.q);
    uint2* const dst = reinterpret_cast<uint2*>(is_k ? a.kx : a.qx);
    uint16_t* const scales = is_k ? a.ks : a.qs;
    const int64_t rows = heads * L, pieces = rows * G * 8;   // (whole teams: pieces % 8 == 0)
    const int64_t p0 = (int64_t)b * (256 * kRowItems) + t;
    uint4 x[kRowItems];
#pragma unroll
    for (int i = 0; i < kRowItems; ++i)
        if (p0 + 256 * i < pieces)
            x[i] = src[p0 + 256 * i];
#pragma unroll
    for (int i = 0; i < kRowItems; ++i) {
        const int64_t p = p0 + 256 * i;
        if (p >= pieces)
            break;
        uint32_t s16;
        dst[p] = quantize_fp8<GS>(x[i], fabsf(__uint_as_float(x[i].x << 16)), s16);
        if (u == 0)
            scales[G == 1 ? p >> 3 : ((p >> 3) & 1) * rows + (p >> 4)] = (uint16_t)s16;
    }
}

__device__ __forceinline__ v8i load32(const uint8_t* p)
{
    const uint4 a = reinterpret_cast<const uint4*>(p)[0];
    const uint4 b = reinterpret_cast<const uint4*>(p)[1];
    return v8i{(int)a.x, (int)a.y, (int)a.z, (int)a.w, (int)b.x, (int)b.y, (int)b.z, (int)b.w};
}

// operand of the scale outer product (fp16 32x32x8, only k = 0 non-zero); the
// key's or channel's word is zero in the upper half-wave, which holds k = 4 ..
__device__ __forceinline__ v16f mfma_outer(int a, int b)
{
    typedef int v2i __attribute__((ext_vector_type(2)));
    typedef _Float16 v4h __attribute__((ext_vector_type(4)));
    const v16f zero = {};
    return __builtin_amdgcn_mfma_f32_32x32x8f16(__builtin_bit_cast(v4h, v2i{a, 0}),
                                                __builtin_bit_cast(v4h, v2i{b, 0}), zero, 0, 0, 0);
}

__device__ __forceinline__ v16f mfma_fp8(const v8i& a, const v8i& b)
{
    const v16f zero = {};
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, zero, 0, 0, 0, 0, 0, 0);
}

// v of this lane and of lane l ^ 32
__device__ __forceinline__ float2 both_halves(float v)
{
    const uint32_t b = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    return {__uint_as_float(r[0]), __uint_as_float(r[1])};
}

// LDS staging of one 64-key chunk, in the order the MFMA lanes read it, so
// that every operand read is one conflict-free ds_read_b128 per 16 bytes:
//   K~   [t][g][j][slot][16 B]: lane (rho, h) of key tile t reads bytes
//        64 g + 32 h + 16 j .. of key kappa(t, rho) (see the header);
//   V~^T [i][j][slot][16 B]: lane (n, h) reads bytes 32 h + 16 j .. of the
//        chunk's 64 keys of channel 32 i + n;
//   slot = 32 h + (rho or n) ^ swz(g, h, j): 8 threads that store consecutive
//   pieces of a row reach 8 different slots mod 8 (without it every piece of a
//   key met in the same banks: 24 % of the kernel's cycles at L = 4608);
//   the key scales [t][g][lane] and the channel scales [i][lane]: words of an
//   fp16 value in lanes 0 .. 31, zeros in the others.
template <int G, int WQ, int S>
struct AttnStage {
    static constexpr int D = 64 * G;
    static constexpr int kV = 64 * D;               // offsets: V~^T,
    static constexpr int kSk = kV + D * 64;         // key scales,
    static constexpr int kSv = kSk + 2 * G * 256;   // channel scales
    static constexpr int kBytes = kSv + D * 8;
    static constexpr int kThreads = 64 * WQ * S;
    static constexpr int kPieces = 4 * D;           // 16-byte pieces of K~, and of V~^T
    static constexpr int kItems = S * kPieces / kThreads;   // per thread, of S chunks
    static_assert(S * kPieces % kThreads == 0 && (kPieces % kThreads == 0 || kThreads % kPieces == 0),
                  "every thread moves as many, and each lies in one chunk");
    // a row of 8 pieces (K~ at d = 128) takes 8 slots, two rows of 4 take the
    // even and the odd ones
    static __device__ constexpr int k_swz(int g, int h, int j) { return G == 2 ? 4 * g + 2 * h + j : 4 * h + 2 * j; }
    static __device__ constexpr int v_swz(int h, int j) { return 4 * h + 2 * j; }
};

// One block: WQ S waves, queries 32 WQ qb .. of head `head`: S teams of WQ
// waves of 32 queries each, which take the chunks in turn (team k chunks k,
// k + S, ..) and share the staged ones; the teams' sums meet after pass 1 and
// their outputs at the end, in LDS.  Block b of the launch is block first + b
// of heads qblocks.  qx / kx: [heads L][64 G] e4m3, qs / ks: [G][heads L]
// fp16; vx: [heads d][L] e4m3 (V^T), vs: [L / 64][heads d] fp16; o: bf16
// [L][ldo], head h at columns h d ...
//
// What bounds it is the issue of vector instructions (per 64-key chunk and
// wave 24 MFMAs at d = 128 beside 582, counted; 64 are exponentials), so both
// passes are written as slots: a slot issues the matrix product of one unit
// (32 rows by 32 queries of one 64-group, with the outer product of its
// scales) and multiplies out the unit before it, whose product ran meanwhile,
// beside a piece of the softmax or of the quantizer; the operands are read
// from LDS a slot ahead.  Pass 2 runs the PV units of the chunk before, then
// the score units of the chunk after the one it quantizes.  At 32 heads, L =
// 4608, d = 128 the kernel took 757 us as one chain of scores, softmax,
// quantizer and PV with a maximum per chunk; 623 in slots, 543 with the
// swizzled staging, 450 with teams for the last quarter of a round (vector
// instructions then issue in 80 % of the whole rounds' cycles, MFMAs in 35 %).
// Tried and dropped: log2(e) / sqrt(d) folded into the score scales (one
// instruction less per score and pass, 1-5 % faster, but a larger error:
// 1.682e-3 against 1.670e-3 of the output's norm).
template <int GS, int G, int WQ, int S>
__global__ __launch_bounds__(64 * WQ * S) __attribute__((amdgpu_waves_per_eu(2, 2))) void lzs_attention_fused_kernel(
    const uint8_t* __restrict__ qx, const uint16_t* __restrict__ qs,
    const uint8_t* __restrict__ kx, const uint16_t* __restrict__ ks,
    const uint8_t* __restrict__ vx, const uint16_t* __restrict__ vs, int64_t heads, int64_t L,
    float kexp, uint16_t* __restrict__ o, int64_t ldo, uint32_t first_block, uint32_t qblocks)
{
    using St = AttnStage<G, WQ, S>;
    constexpr int D = St::D;
    constexpr int TV = D / 32;                 // channel tiles of the PV product
    constexpr int NU = 2 * G;                  // score units of a chunk
    __shared__ __attribute__((aligned(16))) uint8_t smem[2][S][St::kBytes];

    // blocks of one head on one XCD (consecutive block ids go round robin
    // over the 8 XCDs), so its K~ / V~^T chunks are shared in that L2
    const uint32_t total = gridDim.x, bid = blockIdx.x;
    const uint32_t logical = first_block + (total % 8 == 0 ? (bid % 8) * (total / 8) + bid / 8 : bid);
    const int64_t head = logical / qblocks;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int team = wave / WQ, wq = wave % WQ;
    const int64_t qb = (int64_t)(logical % qblocks) * (32 * WQ);
    if (qb >= L)
        return;                                // a ragged head's last blocks
    const int64_t q0 = qb + wq * 32;
    // a wave past the end of a ragged block still loads and waits at the
    // barriers, and computes nothing (wave-uniform)
    const bool active = q0 < L;
    const int lane = tid & 63;
    const int n = lane & 31, h = lane >> 5;
    const int64_t rows = heads * L;
    const int chunks = (int)(L / 64), steps = (chunks + S - 1) / S;

    // ---- cooperative staging of a step's S chunks: thread tid moves pieces
    // tid + 64 WQ S p, in two halves (K~, V~^T) through the same registers
    // K~ piece u: key u / (D / 16), bytes 16 (u % (D / 16)) of its row
    auto rho_of = [](int key) { return 8 * ((key >> 2) & 3) + 4 * (key >> 5) + (key & 3); };
    auto k_lds_off = [&](int u) {
        const int key = u / (D / 16), part = u % (D / 16);
        const int g = part >> 2, hh = (part >> 1) & 1, j = part & 1;
        return (((((key >> 4) & 1) * G + g) * 2 + j) * 64 + (rho_of(key) ^ St::k_swz(g, hh, j)) + 32 * hh) * 16;
    };
    // V~^T piece u: channel u / 4, bytes 16 (u % 4) of its 64-key row
    auto v_lds_off = [](int u) {
        const int ch = u >> 2, hh = (u >> 1) & 1, j = u & 1;
        return St::kV + (((ch >> 5) * 2 + j) * 64 + ((ch & 31) ^ St::v_swz(hh, j)) + 32 * hh) * 16;
    };
    v4u pieces[St::kItems];                    // native vectors: kept in registers
    uint32_t scale = 0;
    auto chunk_of = [&](int step, int k) { return min(step * S + k, chunks - 1); };
    constexpr int T = St::kThreads, kP = St::kPieces;
    auto chunk_of_piece = [&](int p) { return T <= kP ? T * p / kP : T / kP * p + tid / kP; };
    // a step's scales: thread tid the chunk, group or channel tid names
    const int ks_k = tid / (64 * G), ks_i = tid % (64 * G), vs_k = tid / D, vs_i = tid % D;
    static_assert(T >= S * D, "a thread per scale");
    auto load_k = [&](int step) {
#pragma unroll
        for (int p = 0; p < St::kItems; ++p) {
            const int k = chunk_of_piece(p), u = (tid + T * p) % kP;
            pieces[p] = reinterpret_cast<const v4u*>(kx + (head * L + 64 * chunk_of(step, k)) * D)[u];
        }
        if (T == S * D || ks_k < S)
            scale = ks[(ks_i >> 6) * rows + head * L + 64 * chunk_of(step, ks_k) + (ks_i & 63)];
    };
    auto load_v = [&](int step) {
#pragma unroll
        for (int p = 0; p < St::kItems; ++p) {
            const int k = chunk_of_piece(p), u = (tid + T * p) % kP;
            pieces[p] = *reinterpret_cast<const v4u*>(vx + (head * D + (u >> 2)) * L + 64 * chunk_of(step, k) +
                                                          16 * (u & 3));
        }
        if (T == S * D || vs_k < S)
            scale = vs[chunk_of(step, vs_k) * heads * D + head * D + vs_i];
    };
    auto store_k = [&](int b) {
#pragma unroll
        for (int p = 0; p < St::kItems; ++p) {
            const int k = chunk_of_piece(p), u = (tid + T * p) % kP;
            *reinterpret_cast<v4u*>(smem[b][k] + k_lds_off(u)) = pieces[p];
        }
        if (T == S * D || ks_k < S) {
            const int key = ks_i & 63;
            *reinterpret_cast<uint32_t*>(smem[b][ks_k] + St::kSk +
                                         ((((key >> 4) & 1) * G + (ks_i >> 6)) * 64 + rho_of(key)) * 4) = scale;
        }
    };
    auto store_v = [&](int b) {
#pragma unroll
        for (int p = 0; p < St::kItems; ++p) {
            const int k = chunk_of_piece(p), u = (tid + T * p) % kP;
            *reinterpret_cast<v4u*>(smem[b][k] + v_lds_off(u)) = pieces[p];
        }
        if (T == S * D || vs_k < S)
            *reinterpret_cast<uint32_t*>(smem[b][vs_k] + St::kSv + ((vs_i >> 5) * 64 + (vs_i & 31)) * 4) = scale;
    };
    // (loads in flight stay in flight)
    auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    // ---- what the waves share, in order: pass 1 reads step c from buffer
    // c & 1, which step c + 2 then replaces; pass 2 at step c writes K~ of c + 2
    // and V~^T of c into buffer c & 1 and reads K~ of c + 1 and V~^T of c - 1
    // from the other.
    for (int i = tid; i < 2 * S * (2 * G + TV) * 32; i += T) {   // the zeros of the scales' upper lanes
        const int row = i / 32 % (2 * G + TV), b = i / 32 / (2 * G + TV);
        *reinterpret_cast<uint32_t*>(smem[b / S][b % S] + St::kSk + row * 256 + 128 + (i & 31) * 4) = 0;
    }
    auto begin1 = [&] {
        load_k(0);
        store_k(0);
        load_k(1);
        store_k(1);
        barrier();
    };
    auto begin2 = [&] {
        barrier();
        load_k(0);
        store_k(0);
        load_k(1);
        store_k(1);
        load_v(0);
        store_v(1);                            // (stands in for step -1, whose codes are 0)
        barrier();
    };
    // the sums of a team's queries: [team][wq][n] of (nf, l), in the first buffer
    float2* const sums = reinterpret_cast<float2*>(smem[0][0]);
    // a team's partial outputs: row tile i of wave wq, for the team i % S that stores it
    auto partial = [&](int i, int from) {
        const int owner = i % S, rank = from < owner ? from : from - 1;
        return reinterpret_cast<v4f*>(smem[0][0] + ((i * (S - 1) + rank) * WQ + wq) * 4096 + lane * 16);
    };
    static_assert(S == 1 || TV * (S - 1) * WQ * 4096 <= (int)sizeof(smem), "partial outputs fit");
    if (!active) {
        begin1();
        for (int c = 0; c < steps; ++c) {
            load_k(c + 2);
            barrier();
            store_k(c & 1);
        }
        if constexpr (S > 1) {
            barrier();
            barrier();
        }
        begin2();
        barrier();
        for (int c = 0; c < steps; ++c) {
            load_k(c + 2);
            store_k(c & 1);
            load_v(c);
            store_v(c & 1);
            barrier();
        }
        if constexpr (S > 1) {
            barrier();
            barrier();
        }
        return;
    }

    auto lds32 = [&](const uint8_t* s0, const uint8_t* s1) {
        const uint4 a = *reinterpret_cast<const uint4*>(s0);
        const uint4 b = *reinterpret_cast<const uint4*>(s1 + 1024);
        return v8i{(int)a.x, (int)a.y, (int)a.z, (int)a.w, (int)b.x, (int)b.y, (int)b.z, (int)b.w};
    };
    v8i qop[G];
    int sq[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        qop[g] = load32(qx + (head * L + q0 + n) * D + 64 * g + 32 * h);
        sq[g] = qs[g * rows + head * L + q0 + n];
    }

    int k_slot[G][2], v_slot[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        v_slot[j] = (32 * h + (n ^ St::v_swz(h, j))) * 16;
#pragma unroll
        for (int g = 0; g < G; ++g)
            k_slot[g][j] = (32 * h + (n ^ St::k_swz(g, h, j))) * 16;
    }
    // score unit u = t G + g: x[t] gains group g's product
    v8i op;                                    // the next unit's rows and their scales
    int sc_next;
    auto fetch_k = [&](const uint8_t* s, int u) {
        op = lds32(s + u * 2048 + k_slot[u % G][0], s + u * 2048 + k_slot[u % G][1]);
        sc_next = *reinterpret_cast<const int*>(s + St::kSk + u * 256 + lane * 4);
    };
    auto fetch_v = [&](const uint8_t* s, int i) {
        op = lds32(s + St::kV + i * 2048 + v_slot[0], s + St::kV + i * 2048 + v_slot[1]);
        sc_next = *reinterpret_cast<const int*>(s + St::kSv + i * 256 + lane * 4);
    };
    v16f x[2], pc, sc;                         // pc, sc: the pending unit's products
    auto score = [&](auto uc, const v16f& p, const v16f& s) {
        constexpr int t = decltype(uc)::value / G, g = decltype(uc)::value % G;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            x[t][r] = g == 0 ? p[r] * s[r] : fmaf(p[r], s[r], x[t][r]);
        asm volatile("" : "+v"(x[t]));         // not sunk out of its slot
    };
    auto fence = [] { __builtin_amdgcn_sched_barrier(0); };

    // ---- pass 1: per lane the sum of e = 2^(x kexp + nf) over its 32 keys of
    // every chunk.  -nf is an integer near the maximum of x kexp: any
    // reference does that neither overflows nor loses the sum, so it is moved
    // (to a tile's maximum) only when a tile's sum passes 2^12, and no maximum
    // is formed otherwise.
    constexpr float kMost = 4096.0f;
    float nf = 1e30f, l = 0.0f;                // (the first tile's sum is infinite)
    auto tile_sum = [&](auto tc, bool exists) {
        const v16f& v = x[decltype(tc)::value];
        // four independent chains
        auto sum = [&] {
            float s4[4];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float e = __builtin_amdgcn_exp2f(fmaf(v[r], kexp, nf));
                s4[r & 3] = r < 4 ? e : s4[r & 3] + e;
            }
            return (s4[0] + s4[1]) + (s4[2] + s4[3]);
        };
        float s = sum();
        if (__builtin_amdgcn_ballot_w64(s > kMost) && exists) {
            float m = v[0];
#pragma unroll
            for (int r = 1; r < 16; ++r)
                m = fmaxf(m, v[r]);
            const float to = s > kMost ? -__builtin_rintf(m * kexp) : nf;
            l *= __builtin_amdgcn_exp2f(to - nf);
            nf = to;
            s = sum();
        }
        l += exists ? s : 0.0f;
    };
    begin1();
    fetch_k(smem[0][team], 0);
    pc = mfma_fp8(op, qop[0]);
    sc = mfma_outer(sc_next, sq[0]);
    fetch_k(smem[0][team], 1);
    for (int c = 0; c < steps; ++c) {
        const uint8_t* const here = smem[c & 1][team];
        const uint8_t* const next = smem[(c & 1) ^ 1][team];
        const bool exists = S == 1 || c * S + team < chunks;
        load_k(c + 2);
        auto slot = [&](auto uc) {
            constexpr int u = decltype(uc)::value;
            if constexpr (u == NU - 2)
                barrier();                     // all of this chunk is read, the next is there
            const v16f pn = mfma_fp8(op, qop[(u + 1) % G]);
            const int sn = sc_next;
            fence();
            if constexpr (u + 2 < NU)
                fetch_k(here, u + 2);
            else
                fetch_k(next, u + 2 - NU);
            fence();
            score(uc, pc, sc);
            fence();
            sc = mfma_outer(sn, sq[(u + 1) % G]);
            pc = pn;
            fence();
            if constexpr (u % G == G - 1)
                tile_sum(std::integral_constant<int, u / G>(), exists);
            fence();
        };
        slot(std::integral_constant<int, 0>());
        slot(std::integral_constant<int, 1>());
        if constexpr (G == 2) {
            slot(std::integral_constant<int, 2>());
            slot(std::integral_constant<int, 3>());
        }
        store_k(c & 1);
    }
    {
        // the two half-waves' keys of the same query (identical result in both)
        const float2 n2 = both_halves(nf), l2 = both_halves(l);
        nf = fminf(n2.x, n2.y);
        l = l2.x * __builtin_amdgcn_exp2f(nf - n2.x) + l2.y * __builtin_amdgcn_exp2f(nf - n2.y);
    }
    if constexpr (S > 1) {                     // the teams', in their order (identical result in all)
        barrier();
        sums[(team * WQ + wq) * 32 + n] = {nf, l};
        barrier();
        float2 t[S];
#pragma unroll
        for (int k = 0; k < S; ++k) {
            t[k] = sums[(k * WQ + wq) * 32 + n];
            nf = fminf(nf, t[k].x);
        }
        l = 0.0f;
#pragma unroll
        for (int k = 0; k < S; ++k)
            l += t[k].y * __builtin_amdgcn_exp2f(nf - t[k].x);
    }
    const float inv_l = 1.0f / l;

    // ---- pass 2
    v16f acc[TV];
#pragma unroll
    for (int i = 0; i < TV; ++i)
        acc[i] = v16f{};
    begin2();
    auto first = [&](auto uc) {                // the scores of step 0, the last unit left pending
        constexpr int u = decltype(uc)::value;
        fetch_k(smem[0][team], u);
        pc = mfma_fp8(op, qop[u % G]);
        sc = mfma_outer(sc_next, sq[u % G]);
        if constexpr (u + 1 < NU)
            score(uc, pc, sc);
    };
    first(std::integral_constant<int, 0>());
    first(std::integral_constant<int, 1>());
    if constexpr (G == 2) {
        first(std::integral_constant<int, 2>());
        first(std::integral_constant<int, 3>());
    }
    barrier();
    fetch_v(smem[1][team], 0);

    // the quantized probabilities of the chunk before (operand, group scale)
    v8i pop = {};
    int sp = 0;
    v8i pnew;
    int spnew = 0;
    float R = 0.0f;                            // e R: the Stage-1 code before rounding
    int fl[4] = {0, 0, 0, 0};
    auto max8 = [&](int t, int half) {
        const v16f& v = x[t];
        float m = v[8 * half];
#pragma unroll
        for (int r = 1; r < 8; ++r)
            m = fmaxf(m, v[8 * half + r]);
        return m;
    };
    // rne(e R) in the low half (a code is 127 at most but for a group scale
    // that was rounded down)
    auto code_bits = [&](float v) {
        return __float_as_uint(fmaf(__builtin_amdgcn_exp2f(fmaf(v, kexp, nf)), R, kMagic));
    };
    float m8[4];
    auto group_scale_of = [&](bool exists) {
        float xm = fmaxf(fmaxf(m8[0], m8[1]), fmaxf(m8[2], m8[3]));
        const float2 x2 = both_halves(xm);
        xm = fmaxf(x2.x, x2.y);
        // alpha = max of P = e / sum over the 64-key group, the fp16 scale
        // s = alpha / 127 (the IEEE quotient: one correction step), R = 1 / (sum s)
        const float alpha = __builtin_amdgcn_exp2f(fmaf(xm, kexp, nf)) * inv_l;
        const float a0 = alpha * kInv127;
        const _Float16 s16 = (_Float16)fmaf(fmaf(-127.0f, a0, alpha), kInv127, a0);
        const uint32_t sbits = exists ? __builtin_bit_cast(uint16_t, s16) : 0u;
        const float s = (float)s16, r0 = __builtin_amdgcn_rcpf(s);
        R = sbits == 0 ? 0.0f : inv_l * fmaf(r0, fmaf(-s, r0, 1.0f), r0);
        spnew = (int)sbits;
        // FLAG of each subgroup from its largest code (monotone in x)
        auto flag_of = [&](float v) { return lzs_flag(min(code_bits(v) - kMagicBits, 127u)); };
        if constexpr (GS == 8) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                fl[k] = flag_of(m8[k]);
        } else if constexpr (GS == 16) {
            fl[0] = fl[1] = flag_of(fmaxf(m8[0], m8[1]));
            fl[2] = fl[3] = flag_of(fmaxf(m8[2], m8[3]));
        } else {
            const float v = GS == 64 ? xm : fmaxf(fmaxf(m8[0], m8[1]), fmaxf(m8[2], m8[3]));
            fl[0] = fl[1] = fl[2] = fl[3] = flag_of(v);
        }
    };
    // The k-slice of P~^T: dword k of the operand holds keys (relative to
    // the half-wave) 8 (k / 2) + {0, 4, 1, 5} (k even) or {2, 6, 3, 7}
    // (k odd), the byte order of the V~^T rows.  Dwords 2 sub and
    // 2 sub + 1: the codes in pairs, clamped to 127, as bytes, c = q >> FLAG, and the e4m3 value of
    // c 2^FLAG by lookup in the base table with FLAG added to the exponent
    // field of entries 1 .. 7.
    auto quantize8 = [&](int sub) {
        const v16f& v = x[sub >> 1];
        uint32_t q[8];
#pragma unroll
        for (int r = 0; r < 8; ++r)
            q[r] = code_bits(v[8 * (sub & 1) + r]);
        auto pair = [](uint32_t lo, uint32_t hi) {
            const lzs_us2 most = {127, 127};
            return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(
                __builtin_bit_cast(lzs_us2, __builtin_amdgcn_perm(hi, lo, 0x05040100u)), most));
        };
        const uint32_t hi = kTabHi + (uint32_t)fl[sub] * 0x08080808u;
        const uint32_t lo = kTabLo + (uint32_t)fl[sub] * 0x08080800u;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const uint32_t a = pair(q[2 * k], q[2 * k + 4]), b = pair(q[2 * k + 1], q[2 * k + 5]);
            const uint32_t w = __builtin_amdgcn_perm(b, a, 0x06040200u);
            pnew[2 * sub + k] = (int)__builtin_amdgcn_perm(hi, lo, (w >> fl[sub]) & 0x07070707u);
        }
        asm volatile("" : "+v"(pnew));
    };
    auto add_pv = [&](int i) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
            acc[i][r] = fmaf(pc[r], sc[r], acc[i][r]);
        asm volatile("" : "+v"(acc[i]));
    };
    for (int c = 0; c < steps; ++c) {
        const uint8_t* const there = smem[(c & 1) ^ 1][team];
        const bool exists = S == 1 || c * S + team < chunks;
        load_k(c + 2);
        auto slot = [&](auto kc) {
            // units: TV of PV (step c - 1), NU scores (step c + 1)
            constexpr int k = decltype(kc)::value;
            if constexpr (k == (TV + NU) / 2) {
                store_k(c & 1);
                load_v(c);
            }
            if constexpr (k == TV + NU - 1) {
                store_v(c & 1);
                barrier();                     // all of `there` is read, the other buffer is there
            }
            v16f pn;
            if constexpr (k < TV)
                pn = mfma_fp8(op, pop);
            else
                pn = mfma_fp8(op, qop[(k - TV) % G]);
            const int sn = sc_next;
            fence();
            if constexpr (k + 1 < TV)
                fetch_v(there, k + 1);
            else if constexpr (k + 1 < TV + NU)
                fetch_k(there, k + 1 - TV);
            else
                fetch_v(smem[c & 1][team], 0);
            fence();
            if constexpr (k == 0)
                score(std::integral_constant<int, NU - 1>(), pc, sc);
            else if constexpr (k <= TV)
                add_pv(k - 1);
            else
                score(std::integral_constant<int, k - TV - 1>(), pc, sc);
            fence();
            if constexpr (k < TV)
                sc = mfma_outer(sn, sp);
            else
                sc = mfma_outer(sn, sq[(k - TV) % G]);
            pc = pn;
            fence();
            // the quantizer: TV slots for the four pieces; x[t] is free for
            // the next chunk's scores after its two
            if constexpr (k == 0) {
                m8[0] = max8(0, 0);
                m8[1] = max8(0, 1);
                m8[2] = max8(1, 0);
                m8[3] = max8(1, 1);
                group_scale_of(exists);
            } else if constexpr (k <= TV) {
                constexpr int per = 4 / TV;
#pragma unroll
                for (int j = 0; j < per; ++j)
                    quantize8(per * (k - 1) + j);
            }
            fence();
        };
        slot(std::integral_constant<int, 0>());
        slot(std::integral_constant<int, 1>());
        slot(std::integral_constant<int, 2>());
        slot(std::integral_constant<int, 3>());
        if constexpr (G == 2) {
            slot(std::integral_constant<int, 4>());
            slot(std::integral_constant<int, 5>());
            slot(std::integral_constant<int, 6>());
            slot(std::integral_constant<int, 7>());
        }
        pop = pnew;
        sp = spnew;
    }
    // the PV units of the last step (the first one's rows are fetched)
#pragma unroll
    for (int i = 0; i < TV; ++i) {
        if (i > 0)
            fetch_v(smem[(steps - 1) & 1][team], i);
        pc = mfma_fp8(op, pop);
        sc = mfma_outer(sc_next, sp);
        add_pv(i);
    }
    if constexpr (S > 1) {
        barrier();
#pragma unroll
        for (int i = 0; i < TV; ++i)
            if (team != i % S)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    partial(i, team)[64 * q] = v4f{acc[i][4 * q], acc[i][4 * q + 1], acc[i][4 * q + 2], acc[i][4 * q + 3]};
        barrier();
#pragma unroll
        for (int i = 0; i < TV; ++i)
            if (team == i % S) {
                v16f sum;
#pragma unroll
                for (int k = 0; k < S; ++k)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        v4f y = {acc[i][4 * q], acc[i][4 * q + 1], acc[i][4 * q + 2], acc[i][4 * q + 3]};
                        if (k != i % S)
                            y = partial(i, k)[64 * q];
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            sum[4 * q + e] = k == 0 ? y[e] : sum[4 * q + e] + y[e];
                    }
                acc[i] = sum;
            }
    }
    // O^T tile i, register r: channel 32 i + 8 (r / 4) + 4 h + r % 4 of query
    // q0 + n; four consecutive channels per 8-byte store
    typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    uint16_t* orow = o + (q0 + n) * ldo + head * D;
#pragma unroll
    for (int i = 0; i < TV; ++i) {
        if (team != i % S)
            continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const f2 a = {acc[i][4 * j], acc[i][4 * j + 1]};
            const f2 b = {acc[i][4 * j + 2], acc[i][4 * j + 3]};
            const uint2 v = {__builtin_bit_cast(uint32_t, __builtin_convertvector(a, bf2)),
                             __builtin_bit_cast(uint32_t, __builtin_convertvector(b, bf2))};
            *reinterpret_cast<uint2*>(orow + 32 * i + 8 * j + 4 * h) = v;
        }
    }
}

template <int GS, int WQ, int S>
void launch_fused_w(const uint8_t* qx, const uint16_t* qs, const uint8_t* kx, const uint16_t* ks,
                    const uint8_t* vx, const uint16_t* vs, int64_t heads, int64_t L, int64_t d,
                    uint16_t* o, int64_t ldo, int64_t first, int64_t count, int64_t qblocks, hipStream_t stream)
{
    const dim3 grid((unsigned)count), block(64 * WQ * S);
    const float kexp = (float)(1.4426950408889634 / std::sqrt((double)d));
    if (d == 64)
        lzs_attention_fused_kernel<GS, 1, WQ, S><<<grid, block, 0, stream>>>(
            qx, qs, kx, ks, vx, vs, heads, L, kexp, o, ldo, (uint32_t)first, (uint32_t)qblocks);
    else
        lzs_attention_fused_kernel<GS, 2, WQ, S><<<grid, block, 0, stream>>>(
            qx, qs, kx, ks, vx, vs, heads, L, kexp, o, ldo, (uint32_t)first, (uint32_t)qblocks);
}

// Two blocks of 4 waves (128 queries each) fill a compute unit, and take whole
// rounds of the device (one block of 8 waves, whose barriers hold more waves,
// is 2 to 9 % slower at 48 heads, L = 4096).  What is left over is split among
// teams so that it is one shorter round: up to a quarter of one by 4 teams, up
// to a half by 2, up to three quarters by 2 in blocks of 64 queries; more than
// that runs on unsplit.  Measured in us, d = 128, for unsplit / 2 teams of 4
// waves / 2 of 2 / 4 of 2 left-over blocks: 32 heads x 4608, a quarter, 564 /
// 537 / 510 / 491; 12 x 2048, 0.38, 75 / 65 / 68 / 76; 24 x 2048, 0.75, 110 /
// 121 / 103 / 113; 40 x 4608, 0.81, 612 in one launch / 654 / 664 / 688.  Four
// teams want two chunks each: 8 x 256 14.3 with two, 15.0 with four.
template <int GS>
hipError_t launch_fused_gs(const uint8_t* qx, const uint16_t* qs, const uint8_t* kx,
                           const uint16_t* ks, const uint8_t* vx, const uint16_t* vs,
                           int64_t heads, int64_t L, int64_t d, uint16_t* o, int64_t ldo,
                           hipStream_t stream)
{
    const int64_t round = 2 * std::max<int64_t>(1, device_compute_units());
    const int64_t per_head = (L + 127) / 128, blocks = heads * per_head;
    const int64_t over = blocks % round;
    const int64_t rest = 4 * over > 3 * round ? 0 : over, whole = blocks - rest;
    if (whole > 0)
        launch_fused_w<GS, 4, 1>(qx, qs, kx, ks, vx, vs, heads, L, d, o, ldo, 0, whole, per_head, stream);
    if (rest == 0)
        return hipGetLastError();
    if (4 * rest <= round && L >= 8 * 64)
        launch_fused_w<GS, 2, 4>(qx, qs, kx, ks, vx, vs, heads, L, d, o, ldo, 2 * whole, 2 * rest, 2 * per_head,
                                 stream);
    else if (4 * rest > round && 2 * rest <= round)
        launch_fused_w<GS, 4, 2>(qx, qs, kx, ks, vx, vs, heads, L, d, o, ldo, whole, rest, per_head, stream);
    else
        launch_fused_w<GS, 2, 2>(qx, qs, kx, ks, vx, vs, heads, L, d, o, ldo, 2 * whole, 2 * rest, 2 * per_head,
                                 stream);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attention_operands(const uint16_t* q, const uint16_t* k, const uint16_t* v, int64_t heads,
                                     int64_t L, int64_t d, int lzs_group, uint8_t* qx, uint16_t* qs,
                                     uint8_t* kx, uint16_t* ks, uint8_t* vx, uint16_t* vs, hipStream_t stream)
{
    const AttnOperands a{q, k, v, qx, kx, vx, qs, ks, vs};
    const int64_t vblocks = heads * (L / 64) * (d / 64);
    const int64_t rblocks = (heads * L * (d / 8) + 256 * kRowItems - 1) / (256 * kRowItems);
    const dim3 grid((unsigned)(vblocks + 2 * rblocks)), block(256);
    switch (lzs_group) {
    case 8: quantize_operands_kernel<8><<<grid, block, 0, stream>>>(a, heads, L, d, (uint32_t)vblocks, (uint32_t)rblocks); break;
    case 16: quantize_operands_kernel<16><<<grid, block, 0, stream>>>(a, heads, L, d, (uint32_t)vblocks, (uint32_t)rblocks); break;
    case 32: quantize_operands_kernel<32><<<grid, block, 0, stream>>>(a, heads, L, d, (uint32_t)vblocks, (uint32_t)rblocks); break;
    default: quantize_operands_kernel<64><<<grid, block, 0, stream>>>(a, heads, L, d, (uint32_t)vblocks, (uint32_t)rblocks); break;
    }
    return hipGetLastError();
}

hipError_t launch_attention_fused(const uint8_t* qx, const uint16_t* qs, const uint8_t* kx,
                                  const uint16_t* ks, const uint8_t* vx, const uint16_t* vs,
                                  int64_t heads, int64_t L, int64_t d, int lzs_group, uint16_t* o,
                                  int64_t ldo, hipStream_t stream)
{
    switch (lzs_group) {
    case 8: return launch_fused_gs<8>(qx, qs, kx, ks, vx, vs, heads, L, d, o, ldo, stream);
    case 16: return launch_fused_gs<16>(qx, qs, kx, ks, vx, vs, heads, L, d, o, ldo, stream);
    case 32: return launch_fused_gs<32>(qx, qs, kx, ks, vx, vs, heads, L, d, o, ldo, stream);
    default: return launch_fused_gs<64>(qx, qs, kx, ks, vx, vs, heads, L, d, o, ldo, stream);
    }
}

}  // namespace quartz

// What the kernels on bf16 parts share (conv_packets.hip: forward and backward-data, conv_wgrad_packets.hip and
// conv_wgrad_staged.hip: weight gradient, conv_direct.hip and fc_direct.hip: small launches): the split of an fp32 number,
// the tile shapes, the multiplication of one step.
#pragma once
#include "common.h"

namespace purine {
namespace packets {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int PLANES = 3;

// An operand is split as 2^16 times its value, and the joined sums are scaled back: 2^16 x = p0 + p1 + p2 exactly for
// every fp32 x of less than 2^112, because the last bit of the smallest normal number (2^-149) is then bf16's smallest
// subnormal. (Unscaled, the third part is lost below 2^-110 and the second below 2^-118: 2e-5 of the operand at 2^-120,
// 1.5e-3 at 2^-126.) Scaling by powers of two leaves every rounding of ordinary numbers where it was. What does not
// fit above, operands of 2^112 or results of 2^96 and more, comes out infinite or NaN, as infinities and NaNs do, and is
// computed again from the fp32 operands.
constexpr float SPLIT_SCALE = 65536.0f, JOIN_SCALE = 1.0f / (65536.0f * 65536.0f);

// The parts of two numbers, or (SCALED) of two that have the factor already. Thirteen instructions, two of them the scaling.
template <bool SCALED = false>
__device__ __forceinline__ void split_pair(float x, float y, uint32_t (&part)[PLANES]) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    if (!SCALED) { x *= SPLIT_SCALE; y *= SPLIT_SCALE; }
#pragma unroll
    for (int pl = 0; pl < PLANES; ++pl) {
        const floatx2 f = {x, y};
        part[pl] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
        x -= __uint_as_float(part[pl] << 16);
        y -= __uint_as_float(part[pl] & 0xffff0000u);
    }
}

// (The empty asm keeps the compiler from moving an element's scaling into the branch around its load, where it would wait
// for that load before the next is issued: layout of 493 x 361 x 5x5 weights and their images, 71 us with, 67 without.)
__device__ __forceinline__ void store_split8(float (&v)[8], unsigned char* base, size_t plane_bytes) {
#pragma unroll
    for (int e = 0; e < 8; ++e) asm volatile("" : "+v"(v[e]));
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    u32x4 q[PLANES];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        uint32_t part[PLANES];
        split_pair(v[2 * e], v[2 * e + 1], part);
#pragma unroll
        for (int pl = 0; pl < PLANES; ++pl) q[pl][e] = part[pl];
    }
#pragma unroll
    for (int pl = 0; pl < PLANES; ++pl) *reinterpret_cast<u32x4*>(base + pl * plane_bytes) = q[pl];
}

template <int TM, int TN, int WM, int WN>
struct Tile {
    static constexpr int BM = TM * WM * 32, BN = TN * WN * 32, NW = WM * WN;
    static constexpr int A_BYTES = PLANES * 2 * BM * 16, B_BYTES = PLANES * 2 * BN * 16;
    static constexpr int STAGE = A_BYTES + B_BYTES;
    static constexpr int NS = STAGE * 3 + 2048 <= 80 * 1024 ? 3 : 2;      // ring of step buffers; two workgroups per CU
    static constexpr int LDS = NS * STAGE + 1024 + BM * 4;                // + spare KB + bias
    static constexpr int LA = A_BYTES / 1024;                             // direct-to-LDS loads of a wavefront: 64 packets each
    static constexpr int RA = (LA + NW - 1) / NW;
    static constexpr int LB = B_BYTES / 1024;
    static constexpr int RBL = (LB + NW - 1) / NW;
    static constexpr int PG = BN / 64, WPG = NW / PG;                     // pixel groups of 64; wavefronts per group
    static constexpr int RB = (2 * PLANES + WPG - 1) / WPG;
    static constexpr int LOADS = RA + RB;                                 // per wavefront and step, whatever happens
    static_assert(NW % PG == 0 && LOADS * (NS - 1) <= 60, "");
};

// cycles: MFMA time of a step on one SIMD (TM * TN * 6 * 32); eff / eff_w: the share of it that the tile
// reaches in the forward / backward-data and in the weight-gradient kernel (256 -> 384 channels 3x3 at
// 13x13, N = 128, whole operators less the layout pass: forward 168 us with 64x256, 187 with 128x128, 195
// with 64x128, 200 with 96x128, 215 with 32x256; weight gradient 180 with 128x128, 194 with 64x256, 193 with
// 96x128, 218 with 64x128: there the filter columns share no packets, so the squarer tile moves less).
struct PacketTile { int bm, bn, cycles; float eff, eff_w; };
#define PACKET_TILES(CALL)                                              \
    switch (bm * 1000 + bn) {                                           \
        case 128128: return CALL(2, 2, 2, 2);                           \
        case 96128:  return CALL(3, 1, 1, 4);                           \
        case 64256:  return CALL(2, 2, 1, 4);                           \
        case 64128:  return CALL(1, 2, 2, 2);                           \
        case 32256:  return CALL(1, 2, 1, 4);                           \
        default: return hipErrorInvalidValue;                           \
    }
constexpr PacketTile kTiles[] = {{128, 128, 768, 0.68f, 0.74f}, {64, 256, 768, 0.74f, 0.69f}, {96, 128, 576, 0.70f, 0.69f},
                                 {64, 128, 384, 0.64f, 0.63f}, {32, 256, 384, 0.58f, 0.60f}};

// The MFMAs of one reduction step, from the step's LDS buffer: the largest of the six products into
// `hi`, the five corrections into `lo`.
template <typename T, int TM, int TN>
__device__ __forceinline__ void multiply_step(const unsigned char* st, int a_off, int b_off, floatx16 (&hi)[TM][TN], floatx16 (&lo)[TM][TN]) {
    bf16x8 av[PLANES][TM], bv[PLANES][TN];
#pragma unroll
    for (int pl = 0; pl < PLANES; ++pl) {
#pragma unroll
        for (int a = 0; a < TM; ++a) av[pl][a] = *reinterpret_cast<const bf16x8*>(st + a_off + (pl * 2 * T::BM + a * 32) * 16);
#pragma unroll
        for (int b = 0; b < TN; ++b) bv[pl][b] = *reinterpret_cast<const bf16x8*>(st + b_off + (pl * 2 * T::BN + b * 32) * 16);
    }
    auto mul = [&](int i, int j, floatx16 (&acc)[TM][TN]) {
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[i][a], bv[j][b], acc[a][b], 0, 0, 0);
    };
    mul(0, 0, hi);
    mul(0, 1, lo);
    mul(1, 0, lo);
    mul(1, 1, lo);
    mul(0, 2, lo);
    mul(2, 0, lo);
}

// The kernels of small launches hold a step's operands in registers: a lane's eight elements of a row (a) and of a column (b), bf16 as four
// pairs (PL = 1, into hi) or fp32, split here.
template <int PL>
__device__ __forceinline__ void multiply_loaded(const unsigned* a, const unsigned* b, floatx16& hi, floatx16& lo) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    u32x4 ap[PL], bp[PL];
    if constexpr (PL == 1) {
        ap[0] = u32x4{a[0], a[1], a[2], a[3]};
        bp[0] = u32x4{b[0], b[1], b[2], b[3]};
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t pa[PLANES], pb[PLANES];
            split_pair(__uint_as_float(a[2 * e]), __uint_as_float(a[2 * e + 1]), pa);
            split_pair(__uint_as_float(b[2 * e]), __uint_as_float(b[2 * e + 1]), pb);
#pragma unroll
            for (int pl = 0; pl < PLANES; ++pl) { ap[pl][e] = pa[pl]; bp[pl][e] = pb[pl]; }
        }
    }
    auto mul = [&](int i, int j, floatx16& acc) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ap[i]), __builtin_bit_cast(bf16x8, bp[j]), acc, 0, 0, 0);
    };
    mul(0, 0, hi);
    if constexpr (PL == 3) {
        mul(0, 1, lo);
        mul(1, 0, lo);
        mul(1, 1, lo);
        mul(0, 2, lo);
        mul(2, 0, lo);
    }
}

// Their wavefronts' sums of one tile in LDS, and element (e, l) of all of them: one rounding at the end, however many wavefronts.
template <int PL>
__device__ __forceinline__ void put_sums(float (&to)[16][64], int lane, const floatx16& hi, const floatx16& lo) {
#pragma unroll
    for (int e = 0; e < 16; ++e) to[e][lane] = PL == 3 ? (hi[e] + lo[e]) * JOIN_SCALE : hi[e];
}
template <int WAVES>
__device__ __forceinline__ float all_sums(const float (*sums)[16][64], int e, int l) {
    double all = 0.0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) all += (double)sums[w][e][l];
    return (float)all;
}

// Every load of this wavefront but the `YOUNGER` youngest has written its LDS packets; then all
// wavefronts meet. A bare barrier: a fence would wait for the loads in flight as well. The empty asm
// statements keep the compiler from moving LDS accesses across.
template <int YOUNGER>
__device__ __forceinline__ void packets_landed() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0070 | (YOUNGER & 15) | ((YOUNGER >> 4) << 14));      // vmcnt(YOUNGER), lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Adds the two accumulator sets (into hi), scales them back and returns a bit per element that is infinite or NaN.
template <int TM, int TN>
__device__ __forceinline__ unsigned long long join_sets(floatx16 (&hi)[TM][TN], const floatx16 (&lo)[TM][TN]) {
    static_assert(TM * TN * 16 <= 64, "");
    unsigned long long bad = 0;
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float v = hi[a][b][e] + lo[a][b][e];
                if (!(__builtin_fabsf(v) <= 3.402823466e38f)) bad |= 1ull << ((a * TN + b) * 16 + e);
                hi[a][b][e] = v * JOIN_SCALE;
            }
    return bad;
}

template <int TM, int TN>
__device__ __forceinline__ void replace_element(floatx16 (&hi)[TM][TN], int idx, float v) {
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int k = 0; k < 16; ++k) hi[a][b][k] = (a * TN + b) * 16 + k == idx ? v : hi[a][b][k];
}

// Where the filter values of GEMM row i and tap (tr, tc) lie: channel ci's at w[fixed + ci * stride], for ci < lim.
// mode: 0 forward (row = output channel), 1 backward-data with unit stride (row = input channel), 2 phase-folded
// (row = (c, a, b), taps a + sh * r', b + sw * s'). Ci: reduction channels.
struct FilterRun { int fixed, stride, lim; };
__device__ __forceinline__ FilterRun filter_run(int mode, int i, int tr, int tc, int C, int R, int S, int sh, int sw, int Ci, const FastDiv& div_phases,
                                                const FastDiv& div_sw) {
    if (mode == 0) return {(i * C * R + tr) * S + tc, R * S, Ci};
    if (mode == 1) return {(i * R + tr) * S + tc, C * R * S, Ci};
    const int c = fastdiv(i, div_phases), ab = i - c * sh * sw;
    const int pa = fastdiv(ab, div_sw), pb = ab - pa * sw;
    const int r = pa + sh * tr, s = pb + sw * tc;
    return {(c * R + r) * S + s, C * R * S, r < R && s < S ? Ci : 0};
}

}  // namespace packets
}  // namespace purine

// bf16 MFMA implicit GEMM with the input patch staged in LDS, for rows of any width, any gather stride
// and tiles that cross images: of the layers that conv_patch_bf16.hip (rows of whole 16-byte packets, one
// image per tile) refuses or has too few tiles for its two roles, those where this one is expected to be
// faster than what they would run on else (plan_conv_pix). Conv / ConvBwdData of paper Figure 1(b).
//
// Bound: LDS reads beside the MFMAs where the chip is full (3x3, 96 -> 128 channels at 28x28, N = 128, 31 us, 711 TFLOP/s: 47 MB
// to and from HBM, 1.5 TB/s, the matrix pipes 42 % busy, a quarter of the LDS cycles lost to conflicts), one workgroup's
// serial chain (first patch, channel groups one after another, stores) where it is not (256 -> 256 at 13x13, N = 128, 85 tiles of
// 256 pixels on three row tiles, 40 us, 34 %). A workgroup of four wavefronts owns BM
// output rows and BN consecutive output pixels, counted over all images. Per group of 16 gathered
// channels the input rows its taps touch are loaded once from NCHW: a thread takes four pixels of eight
// channels as 8-byte loads at whatever alignment the row has (the last four pixels of a row are taken
// from its end, so that no load leaves the row), transposes them in registers and stores [position][8
// channels] packets. Positions outside the image are zeros that are written once, so the tap loop
// has no bounds test, and nothing is copied in HBM. The patch lies in planes (position parity, channel
// half), because a lane owns two adjacent pixels (4-byte stores) and reads every other position. The
// filter comes from a copy in the order of its LDS tiles, by loads that write LDS directly, a stage (a
// run of taps) ahead; the next group's patch is requested at the group's first stage and stored after
// its last. One barrier per stage.
#include "packets.h"
#include "pix_common.h"
#include <cmath>

namespace purine {
namespace pix {
namespace {

using packets::bf16x8;
using packets::filter_run;
using packets::FilterRun;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x2 __attribute__((aligned(2))) u32x2_any;      // four pixels, at any element

struct PatchAnyParams {
    const void* a;              // repacked filter
    unsigned a_bytes;
    int taps, cgs;
    int stage_taps, stages;     // taps per stage, stages per group
    int pw;                     // patch columns
    int h_base, w_base;         // input row / column of patch row / column 0 of output row / column 0
    int c0, ncol, quads;        // input columns [c0, c0 + ncol) inside the patch; loads of four per row
    int img_rows;               // patch rows of a whole image
    int plane_bytes;
    int pairs;                  // output written as 4-byte pixel pairs
    unsigned dx_bytes;          // stride-2 depth-to-space output of less than 2^31 bytes: its span, else 0
    FastDiv div_ho, div_quads, div_img;
};

// Filter copy, one thread per packet of eight channels: [row tile][group][tap][half][row][8], zero past the last
// row or channel.
struct FilterPackets {
    const uint16_t* w; u32x4* a;
    int mode, K, C, R, S, sh, sw, St, Co, Ci, bm, total;
    FastDiv div_bm, div_taps, div_cgs, div_st, div_phases, div_sw;
    int taps, cgs;
};
__global__ __launch_bounds__(256) void pack_filter_bf16_kernel(const FilterPackets q) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= q.total) return;
    int u = fastdiv(t, q.div_bm);
    const int row = t - u * q.bm, half = u & 1;
    int rest = u >> 1;
    u = fastdiv(rest, q.div_taps);
    const int tap = rest - u * q.taps;
    const int rt = fastdiv(u, q.div_cgs), cg = u - rt * q.cgs;
    const int tr = fastdiv(tap, q.div_st), tc = tap - tr * q.St;
    const int i = rt * q.bm + row, ci0 = cg * 16 + half * 8;
    FilterRun f{0, 0, 0};
    if (i < q.Co) f = filter_run(q.mode, i, tr, tc, q.C, q.R, q.S, q.sh, q.sw, q.Ci, q.div_phases, q.div_sw);
    uint32_t v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = ci0 + e < f.lim ? q.w[(size_t)f.fixed + (size_t)(ci0 + e) * f.stride] : 0u;
    q.a[t] = u32x4{v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16, v[6] | v[7] << 16};
}

// Output of an NCHW tensor below 2^31 bytes through raw buffer accesses on the whole tensor (a lane's pixels
// and its half's four rows are offset registers, a row's part a scalar). Tile column b of a lane is pixel
// px + b; with `pairs` (TN == 2, even planes) the two are one packet.
template <int TM, int TN, bool FWD>
__device__ __forceinline__ void store_any(const PixParams& p, floatx16 (&acc)[TM][TN], int i_base, int px, int lane, const float* bias_lds,
                                          int i_tile0, bool pairs) {
    const bool has_bias = FWD && p.bias != nullptr, relu = FWD && p.relu;
    const bool has_mask = !FWD && p.mask != nullptr, has_beta = !FWD && p.beta != 0.0f;
    const int khalf = lane >> 5;
    const int rows0 = __builtin_amdgcn_readfirstlane(i_base);
    const __amdgpu_buffer_rsrc_t r_out = __builtin_amdgcn_make_buffer_rsrc(p.out, (short)0, (int)p.out_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t r_mask = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(has_mask ? p.mask : p.out), (short)0,
                                                                            (int)p.out_bytes, 0x00020000);
    unsigned voff[TN];
#pragma unroll
    for (int b = 0; b < TN; ++b) {
        const bool live = px + b < p.M;
        const int n = fastdiv(live ? px + b : 0, p.div_howo);
        voff[b] = live ? (unsigned)(n * p.out_ns + (px + b - n * p.HoWo) + khalf * 4 * p.HoWo) * 2u : 0x80000000u;
    }
    const int last = p.Co - khalf * 4;           // rows of this lane's half that exist: row_lo < last
    auto rows = [&](auto relu_c, auto pairs_c) {
        constexpr bool RELU = decltype(relu_c)::value, PAIRS = TN == 2 && decltype(pairs_c)::value;
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {
                const int row0 = rows0 + a * 32 + qd * 8;
                if (row0 >= p.Co) continue;                       // uniform
                floatx4 bq = {0.0f, 0.0f, 0.0f, 0.0f};
                if (has_bias) bq = *reinterpret_cast<const floatx4*>(&bias_lds[row0 + khalf * 4 - i_tile0]);
                uint32_t m[4][TN], o[4][TN];
                auto fetch = [&](const __amdgpu_buffer_rsrc_t& r, uint32_t (&v)[4][TN]) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int soff = (row0 + e) * p.HoWo * 2;
                        const bool ok = row0 + e < last;
                        if constexpr (PAIRS) {
                            const uint32_t w = __builtin_amdgcn_raw_buffer_load_b32(r, ok ? voff[0] : 0x80000000u, soff, 0);
                            v[e][0] = w << 16; v[e][1] = w & 0xffff0000u;
                        } else {
#pragma unroll
                            for (int b = 0; b < TN; ++b)
                                v[e][b] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, ok ? voff[b] : 0x80000000u, soff, 0) << 16;
                        }
                    }
                };
                if (has_mask) fetch(r_mask, m);
                if (has_beta) fetch(r_out, o);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int soff = (row0 + e) * p.HoWo * 2;
                    const bool ok = row0 + e < last;
                    float x[TN];
#pragma unroll
                    for (int b = 0; b < TN; ++b) {
                        x[b] = acc[a][b][qd * 4 + e];
                        if (FWD) x[b] += bq[e];
                        if (RELU) x[b] = x[b] > 0.0f ? x[b] : 0.0f;
                        if (has_mask) x[b] = __uint_as_float(m[e][b]) > 0.0f ? x[b] : 0.0f;
                        if (has_beta) x[b] += __uint_as_float(o[e][b]);
                    }
                    if constexpr (PAIRS) {
                        __builtin_amdgcn_raw_buffer_store_b32(pack_bf16(x[0], x[1]), r_out, ok ? voff[0] : 0x80000000u, soff, 0);
                    } else {
#pragma unroll
                        for (int b = 0; b < TN; ++b)
                            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(pack_bf16(x[b], 0.0f) & 0xffffu), r_out, ok ? voff[b] : 0x80000000u, soff, 0);
                    }
                }
            }
    };
    auto by_pairs = [&](auto relu_c) {
        if (TN == 2 && pairs) rows(relu_c, std::true_type{}); else rows(relu_c, std::false_type{});
    };
    if (relu) by_pairs(std::true_type{}); else by_pairs(std::false_type{});
}

// Depth-to-space epilogue of stride 2 x 2 (row i = (c, a, b) of coarse pixel (hq, wq) is dx[n, c, 2 hq + a - ph, 2 wq + b - pw]) for
// a dx below 2^31 bytes: a and b follow from the accumulator element, so a lane needs four offsets per pixel.
template <int TM, int TN>
__device__ __forceinline__ void store_any_d2s2(const PixParams& p, floatx16 (&acc)[TM][TN], int i_base, int px, int lane, unsigned dx_bytes) {
    const bool has_mask = p.mask != nullptr, has_beta = p.beta != 0.0f;
    const int khalf = lane >> 5;
    const int rows0 = __builtin_amdgcn_readfirstlane(i_base);
    const int plane = p.H * p.W;
    const __amdgpu_buffer_rsrc_t r_out = __builtin_amdgcn_make_buffer_rsrc(p.out, (short)0, (int)dx_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t r_mask = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(has_mask ? p.mask : p.out), (short)0, (int)dx_bytes, 0x00020000);
    unsigned voff[TN][4];
#pragma unroll
    for (int b = 0; b < TN; ++b) {
        const bool live = px + b < p.M;
        const int n = fastdiv(live ? px + b : 0, p.div_howo), rem = (live ? px + b : 0) - n * p.HoWo;
        const int hq = fastdiv(rem, p.div_wo), wq = rem - hq * p.Wo;
        const int hb = (hq + p.hq_min) * 2 - p.ph, wb = (wq + p.wq_min) * 2 - p.pw;
#pragma unroll
        for (int ab = 0; ab < 4; ++ab) {
            const int h = hb + (ab >> 1), w = wb + (ab & 1);
            const bool ok = live & ((unsigned)h < (unsigned)p.H) & ((unsigned)w < (unsigned)p.W);
            voff[b][ab] = ok ? (unsigned)(n * p.out_ns + khalf * plane + h * p.W + w) * 2u : 0x80000000u;
        }
    }
    const int last = p.C - khalf;                // channels of this lane's half that exist: c_lo < last
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
            const int c_lo = (rows0 + a * 32 + qd * 8) >> 2;
            if (c_lo >= p.C) continue;           // uniform
            const int soff = c_lo * plane * 2;
            const bool row_ok = c_lo < last;
            uint32_t m[TN][4], o[TN][4];
            auto fetch = [&](const __amdgpu_buffer_rsrc_t& r, uint32_t (&v)[TN][4]) {
#pragma unroll
                for (int b = 0; b < TN; ++b)
#pragma unroll
                    for (int ab = 0; ab < 4; ++ab)
                        v[b][ab] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r, row_ok ? voff[b][ab] : 0x80000000u, soff, 0) << 16;
            };
            if (has_mask) fetch(r_mask, m);
            if (has_beta) fetch(r_out, o);
#pragma unroll
            for (int b = 0; b < TN; ++b)
#pragma unroll
                for (int ab = 0; ab < 4; ++ab) {
                    float v = acc[a][b][qd * 4 + ab];
                    if (has_mask) v = __uint_as_float(m[b][ab]) > 0.0f ? v : 0.0f;
                    if (has_beta) v += __uint_as_float(o[b][ab]);
                    __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(pack_bf16(v, 0.0f) & 0xffffu), r_out, row_ok ? voff[b][ab] : 0x80000000u, soff, 0);
                }
        }
}

constexpr int AHEAD = 3;
constexpr int row_ahead(int rt) { return rt > 3 ? 2 : 3; }
constexpr int ring_slots(int rt, bool rows) { return rt == 0 ? 2 : rows ? row_ahead(rt) + 1 : AHEAD + 1; }
template <int TM, int TN, int WM, int WN>
struct AnyTile {
    static constexpr int BM = TM * WM * 32, BN = TN * WN * 32;
    static constexpr int TAP_BYTES = BM * 32;
};

// ROUNDS: patch loads (four pixels of eight channels each) per thread and channel group.
// RT: 0, or the taps are RT x RT and the loops over them unrolled. Then
//   ROWS: a stage is a filter row, and filters are requested row_ahead(RT) stages ahead (the patch one group);
//   else a group's whole filter is one stage, and filter and patch are requested AHEAD groups ahead: launches of few
//   workgroups, where a group's loads would otherwise be waited for in every one of them.
template <bool MINUS, bool D2S, int TM, int TN, int WM, int WN, int ROUNDS, int RT, bool ROWS>
__global__ __launch_bounds__(256, 2) void igemm_patch_any_bf16_kernel(const PixParams p, const PatchAnyParams q) {
    typedef AnyTile<TM, TN, WM, WN> T;
    static_assert(WM * WN == 4, "four wavefronts");
    constexpr int BM = T::BM, BN = T::BN;
    constexpr int SLOTS = ring_slots(RT, ROWS), DIST = SLOTS - 1;      // ring of filter stages; distance of the requests
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int slot_bytes = q.stage_taps * T::TAP_BYTES;
    const int PB = q.plane_bytes, patch_bytes = 4 * PB + 128;         // + spare packets for threads without a load
    float* bias_s = reinterpret_cast<float*>(smem);
    unsigned char* ring = smem + BM * 4;
    unsigned char* patch = ring + SLOTS * slot_bytes;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int id = xcd_tile(blockIdx.x, gridDim.x);
    const int pt = id / p.tiles_i, rt = id - pt * p.tiles_i;
    const int i0 = rt * BM, p0 = pt * BN;

    // ---- filter: stage s (tap run s % stages of group s / stages) is contiguous in the copy
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(q.a), (short)0, (int)q.a_bytes, 0x00020000);
    const int group_bytes = q.taps * T::TAP_BYTES;
    auto load_a = [&](int g, int c, int slot) {
        const int t0 = c * q.stage_taps;
        const int units = min(q.stage_taps, q.taps - t0) * (T::TAP_BYTES / 1024);
        const int base = (rt * q.cgs + g) * group_bytes + t0 * T::TAP_BYTES;
        for (int u = wave; u < units; u += 4)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (__attribute__((address_space(3))) void*)(ring + slot * slot_bytes + u * 1024), 16,
                                                     lane * 16, base + u * 1024, 0, 0);
    };
    // ... RT: the same number of loads in every wavefront, always issued, so that waits can count them; those past the
    // stage's or the reduction's end fetch nothing
    constexpr int STAGE_TAPS = ROWS ? RT : RT * RT, UNITS = STAGE_TAPS * (T::TAP_BYTES / 1024), LOADS_A = (UNITS + 3) / 4;
    unsigned char* spare_kb = patch + 2 * patch_bytes;
    auto load_stage = [&](int s, int slot) {
        const bool exists = s < q.cgs * (ROWS ? RT : 1);
#pragma unroll
        for (int j = 0; j < LOADS_A; ++j) {
            const int u = j * 4 + wave;
            const bool live = exists && u < UNITS;
            unsigned v = live ? (unsigned)(lane * 16) : 0x80000000u;
            asm volatile("" : "+v"(v));          // one load, not one on either side of a branch
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (__attribute__((address_space(3))) void*)(u < UNITS ? ring + slot * slot_bytes + u * 1024 : spare_kb), 16,
                                                     v, live ? rt * q.cgs * group_bytes + (s * UNITS + u) * 1024 : 0, 0, 0);
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    float bias_v = 0.0f;
    if (!MINUS && p.bias != nullptr && tid < BM && i0 + tid < p.Co) bias_v = Elem<uint16_t>::load((const uint16_t*)p.bias, i0 + tid);
    if (!RT) load_a(0, 0, 0);

    // ---- the tile's output rows, counted over (image, row), and its patch
    const int rho0 = fastdiv(p0, p.div_wo);
    const int v0 = fastdiv(rho0, q.div_ho), ho0 = rho0 - v0 * p.Ho;
    const int p_last = min(p0 + BN, p.M) - 1;
    const int rho1 = fastdiv(p_last, p.div_wo);
    const int v1 = fastdiv(rho1, q.div_ho);
    const int gh = p.g_mul_h;
    const int first_rows = (p.Ho - 1 - ho0) * gh + p.Rt;               // patch rows of image v0, were it the last
    // patch row of output row (v, ho)
    auto prow_of = [&](int v, int ho) {
        return v == v0 ? (ho - ho0) * gh : first_rows + (v - v0 - 1) * q.img_rows + ho * gh;
    };
    const int nrows = prow_of(v1, rho1 - v1 * p.Ho) + p.Rt;
    auto patch_at = [&](int P, int h) { return ((P & 1) * 2 + h) * PB + (P >> 1) * 16; };

    unsigned src[ROUNDS];          // byte offset of the four pixels in channel 0
    int l_even[ROUNDS], l_odd[ROUNDS], l_step[ROUNDS];     // LDS offsets of pixels 0 / 1; pixels 2 / 3 lie l_step further
    unsigned half_off[ROUNDS];     // 0, or where the second half's first channel lies
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int t = tid + r * 256, per = nrows * q.quads;
        const int half = t >= per ? 1 : 0;
        const bool task = t < 2 * per;
        const int u = task ? t - half * per : 0;
        const int prow = fastdiv(u, q.div_quads);
        const int col = min((u - prow * q.quads) * 4, q.ncol - 4);
        int v = v0, h = ho0 * gh + q.h_base + prow;
        if (prow >= first_rows) {
            const int w = prow - first_rows, k = fastdiv(w, q.div_img);
            v = v0 + 1 + k;
            h = q.h_base + w - k * q.img_rows;
        }
        const bool live = task && (unsigned)h < (unsigned)p.Hi;
        half_off[r] = half ? (unsigned)(8 * p.HiWi) * 2u : 0u;
        src[r] = live ? (unsigned)(v * p.in_ns + h * p.Wi + q.c0 + col) * 2u : 0u;
        const int P = prow * q.pw + q.c0 + col - q.w_base;
        l_even[r] = live ? patch_at(P, half) : 4 * PB + (tid & 7) * 16;
        l_odd[r] = live ? patch_at(P + 1, half) : 4 * PB + (tid & 7) * 16;
        l_step[r] = live ? 16 : 0;
    }
    typedef u32x2 PatchRegs[ROUNDS][8];
    PatchRegs pre[RT && !ROWS ? AHEAD : 1];
    // (Channels past the last one of the last group: the last channel, or the first half's, is read again; store_patch drops it.)
    auto load_patch = [&](int g, PatchRegs& pre) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const char* base = (const char*)p.in + (size_t)min(g * 16 + e, p.Ci - 1) * p.HiWi * 2;
            const bool both = g * 16 + 8 + e < p.Ci;
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r) {
                unsigned off = src[r] + (both ? half_off[r] : 0u);
                asm volatile("" : "+v"(off));        // one load, its address a scalar base and this offset
                pre[r][e] = *reinterpret_cast<const u32x2_any*>(base + off);
            }
        }
    };
    auto store_patch = [&](int g, PatchRegs& pre) {
        unsigned char* dst = patch + (g & 1) * patch_bytes;
        if ((g + 1) * 16 > p.Ci) {
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const bool exists = g * 16 + (half_off[r] ? 8 : 0) + e < p.Ci;
                    pre[r][e] = u32x2{exists ? pre[r][e][0] : 0u, exists ? pre[r][e][1] : 0u};
                }
        }
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
            for (int px = 0; px < 4; ++px) {
                const unsigned sel = (px & 1) ? 0x07060302u : 0x05040100u;
                u32x4 o;
#pragma unroll
                for (int c2 = 0; c2 < 4; ++c2) o[c2] = __builtin_amdgcn_perm(pre[r][2 * c2 + 1][px >> 1], pre[r][2 * c2][px >> 1], sel);
                *reinterpret_cast<u32x4*>(dst + ((px & 1) ? l_odd[r] : l_even[r]) + (px >> 1) * l_step[r]) = o;
            }
    };
    if constexpr (RT != 0 && ROWS) {
        load_stage(0, 0);
        load_patch(0, pre[0]);
#pragma unroll
        for (int k = 1; k < DIST; ++k) load_stage(k, k);
    } else if constexpr (RT != 0) {
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) { load_stage(k, k); load_patch(k, pre[k]); }
    } else {
        load_patch(0, pre[0]);
    }

    // ---- this lane's pixels: position P + shift sits at half * PB + 8 * P + (P & 1) * (2 * PB - 8)
    int b_same[TN], b_flip[TN];
    const int px0 = p0 + wn * TN * 32 + TN * (lane & 31);
#pragma unroll
    for (int b = 0; b < TN; ++b) {
        const int px = min(px0 + b, p_last);         // pixels past the end read the last one and are not stored
        const int rho = fastdiv(px, p.div_wo), wo = px - rho * p.Wo;
        const int v = fastdiv(rho, q.div_ho);
        const int P = prow_of(v, rho - v * p.Ho) * q.pw + wo * p.g_mul_w;
        const int lin = (lane >> 5) * PB + P * 8;
        b_same[b] = lin + (P & 1) * (2 * PB - 8);
        b_flip[b] = lin + ((P & 1) ^ 1) * (2 * PB - 8);
    }
    const int a_row = ((lane >> 5) * BM + wm * TM * 32 + (lane & 31)) * 16;

    // ---- zeros around the image, in both buffers
    for (int i = tid; i < 2 * patch_bytes / 16; i += 256) *reinterpret_cast<u32x4*>(patch + i * 16) = u32x4{0u, 0u, 0u, 0u};
    if (!MINUS && tid < BM) bias_s[tid] = bias_v;
    // All but the `YOUNGER` youngest loads have landed (63: none is waited for), this wavefront's LDS traffic is done,
    // then all meet. (Bare: a fence would wait for every load.)
    auto meet = [&](auto younger) {
        constexpr int Y = decltype(younger)::value;
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0070 | (Y & 15) | ((Y >> 4) << 14));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    meet(std::integral_constant<int, 63>{});
    store_patch(0, pre[0]);

    floatx16 acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.0f;

    struct Frags { bf16x8 a[TM], b[TN]; };
    auto multiply = [&](const Frags& f) {
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[a], f.b[b], acc[a][b], 0, 0, 0);
    };
    const int reverse = MINUS ? (p.Rt - 1) * q.pw + p.St - 1 : 0;
    // fragments of tap (r, c) from the filter at `sa` and the patch at `sb`
    auto fetch_tap = [&](const unsigned char* sa, const unsigned char* sb, int r, int c, Frags& f) {
        const int shift = MINUS ? (RT - 1 - r) * q.pw + RT - 1 - c : r * q.pw + c;
        const bool odd = shift & 1;
#pragma unroll
        for (int a = 0; a < TM; ++a) f.a[a] = *reinterpret_cast<const bf16x8*>(sa + a * 32 * 16);
#pragma unroll
        for (int b = 0; b < TN; ++b) f.b[b] = *reinterpret_cast<const bf16x8*>(sb + shift * 8 + (odd ? b_flip[b] : b_same[b]));
    };
    if constexpr (RT != 0 && ROWS) {
        int slot = 0, stage = 0;
        for (int g = 0; g < q.cgs; ++g) {
            const unsigned char* sb = patch + (g & 1) * patch_bytes;
            auto row = [&](auto r_c) {
                constexpr int r = decltype(r_c)::value;
                // this stage's filter was requested DIST stages ago; younger are the other stages' and, where a group's first
                // stage lies among those DIST, the next patch's
                meet(std::integral_constant<int, (DIST - 1) * LOADS_A + ((r > 0 && r <= DIST) || r + RT <= DIST ? 8 * ROUNDS : 0)>{});
                load_stage(stage + DIST, slot == 0 ? SLOTS - 1 : slot - 1);
                if (r == 0) load_patch(g + 1, pre[0]);
                __builtin_amdgcn_sched_barrier(0);
                const unsigned char* sa = ring + slot * slot_bytes + a_row;
                Frags f[2];
                fetch_tap(sa, sb, r, 0, f[0]);
#pragma unroll
                for (int c = 0; c < RT; ++c) {
                    if (c + 1 < RT) fetch_tap(sa + (c + 1) * T::TAP_BYTES, sb, r, c + 1, f[(c + 1) & 1]);
                    multiply(f[c & 1]);
                }
                ++stage;
                slot = slot + 1 == SLOTS ? 0 : slot + 1;
            };
            static_assert(RT <= 5, "");
            row(std::integral_constant<int, 0>{});
            if constexpr (RT > 1) row(std::integral_constant<int, 1>{});
            if constexpr (RT > 2) row(std::integral_constant<int, 2>{});
            if constexpr (RT > 3) row(std::integral_constant<int, 3>{});
            if constexpr (RT > 4) row(std::integral_constant<int, 4>{});
            store_patch(g + 1, pre[0]);
        }
        meet(std::integral_constant<int, 0>{});        // no load may outlive the workgroup's LDS
    } else if constexpr (RT != 0) {
        // Group g's filter was requested before its patch, so the wait for the patch (at its stores) is the wait for both.
        int slot = 0;
        auto step = [&](int g, PatchRegs& mine, PatchRegs& next) {
            meet(std::integral_constant<int, 63>{});
            load_stage(g + AHEAD, slot == 0 ? AHEAD : slot - 1);         // group g - 1's slot
            load_patch(g + AHEAD, mine);
            __builtin_amdgcn_sched_barrier(0);
            const unsigned char* sa = ring + slot * slot_bytes + a_row;
            const unsigned char* sb = patch + (g & 1) * patch_bytes;
            constexpr int SETS = 4, TAPS = RT * RT;           // fragments three taps ahead
            Frags f[SETS];
#pragma unroll
            for (int t = 0; t < SETS - 1 && t < TAPS; ++t) fetch_tap(sa + t * T::TAP_BYTES, sb, t / RT, t % RT, f[t]);
#pragma unroll
            for (int t = 0; t < TAPS; ++t) {
                constexpr int L = SETS - 1;
                if (t + L < TAPS) fetch_tap(sa + (t + L) * T::TAP_BYTES, sb, (t + L) / RT, (t + L) % RT, f[(t + L) % SETS]);
                multiply(f[t % SETS]);
            }
            store_patch(g + 1, next);        // (past the last group too: unread, and the compiler can count the loads)
            slot = slot == AHEAD ? 0 : slot + 1;
        };
        static_assert(AHEAD == 3, "");
        for (int g = 0; g < q.cgs; g += AHEAD) {
            step(g, pre[0], pre[1]);
            if (g + 1 < q.cgs) step(g + 1, pre[1], pre[2]);
            if (g + 2 < q.cgs) step(g + 2, pre[2], pre[0]);
        }
        meet(std::integral_constant<int, 0>{});        // no load may outlive the workgroup's LDS
    } else {
        int slot = 0;
        for (int g = 0; g < q.cgs; ++g) {
            const bool more = g + 1 < q.cgs;
            int tr = 0, tc = 0;
            for (int c = 0; c < q.stages; ++c) {
                // behind the group's first stage the next patch's loads are in flight, issued after the filter of this stage
                if (c == 1 && more) meet(std::integral_constant<int, 8 * ROUNDS>{});
                else meet(std::integral_constant<int, 0>{});
                const bool wrap = c + 1 == q.stages;
                if (!wrap || more) load_a(wrap ? g + 1 : g, wrap ? 0 : c + 1, slot ^ 1);
                asm volatile("" ::: "memory");
                if (c == 0 && more) load_patch(g + 1, pre[0]);
                __builtin_amdgcn_sched_barrier(0);
                const int nt = min(q.stage_taps, q.taps - c * q.stage_taps);
                const unsigned char* sa = ring + slot * slot_bytes + a_row;
                const unsigned char* sb = patch + (g & 1) * patch_bytes;
                auto fetch = [&](Frags& f) {
                    const int fwd = tr * q.pw + tc;
                    const int shift = MINUS ? reverse - fwd : fwd;
                    const bool odd = shift & 1;
#pragma unroll
                    for (int a = 0; a < TM; ++a) f.a[a] = *reinterpret_cast<const bf16x8*>(sa + a * 32 * 16);
#pragma unroll
                    for (int b = 0; b < TN; ++b) f.b[b] = *reinterpret_cast<const bf16x8*>(sb + shift * 8 + (odd ? b_flip[b] : b_same[b]));
                    sa += T::TAP_BYTES;
                    if (++tc == p.St) { tc = 0; ++tr; }
                };
                // fragments one tap ahead, in two register sets
                Frags f0, f1;
                fetch(f0);
                for (int t = 0; t < nt; t += 2) {
                    if (t + 1 < nt) fetch(f1);
                    multiply(f0);
                    if (t + 1 >= nt) break;
                    if (t + 2 < nt) fetch(f0);
                    multiply(f1);
                }
                slot ^= 1;
            }
            if (more) store_patch(g + 1, pre[0]);
        }
    }

    if constexpr (D2S) {
        if (q.dx_bytes) store_any_d2s2<TM, TN>(p, acc, i0 + wm * TM * 32, px0, lane, q.dx_bytes);
        else store_tile_at<uint16_t, true, true, TM, TN, false>(p, (uint16_t*)p.out, acc, i0 + wm * TM * 32, [&](int b) { return px0 + b; }, lane >> 5,
                                                           bias_s, i0, 0x7fffffff);
    } else if (RT == 0 && p.out_bytes == 0) {          // views of 2^31 bytes and more: 64-bit addresses
        store_tile_at<uint16_t, false, true, TM, TN, !MINUS>(p, (uint16_t*)p.out, acc, i0 + wm * TM * 32, [&](int b) { return px0 + b; }, lane >> 5,
                                                             bias_s, i0, 0x7fffffff);
    } else {
        store_any<TM, TN, !MINUS>(p, acc, i0 + wm * TM * 32, px0, lane, bias_s, i0, q.pairs != 0);
    }
}

template <bool MINUS, bool D2S, int TM, int TN, int WM, int WN, int ROUNDS, int RT = 0, bool ROWS = false>
hipError_t launch_one(const PixParams& p, const PatchAnyParams& q, int lds, hipStream_t st) {
    const long long total = (long long)p.tiles_i * p.tiles_pix;
    if (total <= 0 || total > 0x7fffffffLL) return hipErrorInvalidValue;
    const auto kern = &igemm_patch_any_bf16_kernel<MINUS, D2S, TM, TN, WM, WN, ROUNDS, RT, ROWS>;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
    }
    ProbeScope probe(st);
    (void)hipGetLastError();   // drop stale status left by earlier, unrelated runtime calls
    hipLaunchKernelGGL((igemm_patch_any_bf16_kernel<MINUS, D2S, TM, TN, WM, WN, ROUNDS, RT, ROWS>), dim3((unsigned)total), dim3(256), (size_t)lds, st, p, q);
    return hipGetLastError();
}

template <bool MINUS, bool D2S, int RT, bool ROWS>
hipError_t by_tile(const PixParams& p, const PatchAnyParams& q, const PatchAnyPlan& k, hipStream_t st) {
#define ANY_CALL(TM, TN, WM, WN)                                                                   \
    (k.rounds == 1 ? launch_one<MINUS, D2S, TM, TN, WM, WN, 1, RT, ROWS>(p, q, k.lds, st)            \
                   : launch_one<MINUS, D2S, TM, TN, WM, WN, 2, RT, ROWS>(p, q, k.lds, st))
    if constexpr (RT != 0 && !ROWS) {
        if (k.rounds != 1) return hipErrorInvalidValue;
        return launch_one<MINUS, D2S, 1, 1, 1, 4, 1, RT, false>(p, q, k.lds, st);
    } else {
        // (depth-to-space: accumulators and addresses of the two largest tiles do not fit the registers)
        switch (k.bm * 1000 + k.bn) {
            case 128256: if constexpr (!D2S) return ANY_CALL(4, 2, 1, 4); else return hipErrorInvalidValue;
            case 96256:  if constexpr (!D2S) return ANY_CALL(3, 2, 1, 4); else return hipErrorInvalidValue;
            case 96128:  return ANY_CALL(3, 1, 1, 4);
            case 64256:  return ANY_CALL(2, 2, 1, 4);
            case 64128:  return ANY_CALL(1, 2, 2, 2);
            case 32256:  return ANY_CALL(1, 2, 1, 4);
            case 32128:  return ANY_CALL(1, 1, 1, 4);
            default: return hipErrorInvalidValue;
        }
    }
#undef ANY_CALL
}

template <bool MINUS, bool D2S>
hipError_t by_taps(const PixParams& p, const PatchAnyParams& q, const PatchAnyPlan& k, hipStream_t st) {
    constexpr int OTHER = D2S ? 2 : 5;
    // an output that spans 2^31 bytes or more: the kernel for any taps has the epilogue for it, and runs with the same tile
    // and stages (its ring has fewer slots than theirs), so that the plan does not depend on the tensors' strides
    if (!D2S && p.out_bytes == 0) return by_tile<MINUS, D2S, 0, false>(p, q, k, st);
    if (k.rt == 3) return k.ahead ? by_tile<MINUS, D2S, 3, false>(p, q, k, st) : by_tile<MINUS, D2S, 3, true>(p, q, k, st);
    if (k.rt == OTHER) return k.ahead ? by_tile<MINUS, D2S, OTHER, false>(p, q, k, st) : by_tile<MINUS, D2S, OTHER, true>(p, q, k, st);
    return by_tile<MINUS, D2S, 0, false>(p, q, k, st);
}

// The tiles and what they cost: a workgroup by itself lasts `fixed` microseconds and per group of 16 channels
// `group` + stages * `stage` + taps * max(its MFMA time, `tap`) cycles; with several on a CU its share of the CU is
// `wg` microseconds, the taps' MFMA time over `eff` and `fill` cycles per patch load. Fitted to 610 layers drawn
// over the sizes the library is used at (3x3 and 5x5, stride 1 and 2, 16 - 512 channels, 7 - 66 pixels a side, 1 - 256
// images): the tile picked is on average 1.6 % behind the best of the eight, 11 % at the 95th percentile; the
// layers together 1.59 times as fast as on the blocked copy (and the one-image patch kernel where rows were
// whole packets), the worst of them 5 % slower. (This picks the tile. Outside those sizes some layers are faster on the other
// kernels: which of them runs is decided by the times at the end of plan_patch_any.)
struct AnyTileCost { int bm, bn, resident; bool ahead; float tap, stage, group, fixed, eff, wg, fill; };
constexpr AnyTileCost kAnyTiles[] = {
    {128, 256, 2, false, 200.0f, 760.0f, 0.0f, 4.7f, 0.66f, 5.4f, 0.05f}, {96, 256, 2, false, 99.0f, 730.0f, 0.0f, 4.4f, 0.62f, 4.0f, 0.03f},
    {96, 128, 3, false, 72.0f, 580.0f, 350.0f, 4.1f, 0.73f, 2.8f, 4.3f},  {64, 256, 2, false, 208.0f, 0.0f, 1150.0f, 4.3f, 0.85f, 3.7f, 2.8f},
    {64, 128, 4, false, 158.0f, 0.0f, 1100.0f, 3.2f, 0.55f, 2.1f, 2.2f},  {32, 256, 4, false, 163.0f, 0.0f, 945.0f, 3.3f, 0.60f, 2.2f, 2.2f},
    {32, 128, 5, false, 22.0f, 440.0f, 370.0f, 2.7f, 0.57f, 1.3f, 3.4f},  {32, 128, 4, true, 14.0f, 790.0f, 520.0f, 3.5f, 0.27f, 2.2f, 0.0f}};

}  // namespace

// How the layer would run here and the expected time. Pure host arithmetic on the pass's extents: never on the strides of
// its tensors, which the scratch query does not know. (Loads have 32-bit byte offsets: every tensor spans less than 2^31 elements.)
PatchAnyPlan plan_patch_any(const PixParams& p, int mode, int force) {
    PatchAnyPlan best{};
    if (p.Rt * p.St < 2 || p.Ci < 8 || p.Wi < 4) return best;
    if (mode != 2 && (long long)p.M * p.Co * 2 >= 0x7fffffffLL) return best;   // dense: the epilogue addresses it as a raw buffer
    const int gh = p.g_mul_h, gw = p.g_mul_w;
    PatchAnyPlan k{};
    k.taps = p.Rt * p.St; k.cgs = (p.Ci + 15) / 16;
    k.pw = (p.Wo - 1) * gw + p.St;
    k.w_base = mode == 0 ? p.g_add_w : p.g_add_w - (p.St - 1);
    k.h_base = mode == 0 ? p.g_add_h : p.g_add_h - (p.Rt - 1);
    k.c0 = k.w_base > 0 ? k.w_base : 0;
    const int c1 = p.Wi < k.w_base + k.pw ? p.Wi : k.w_base + k.pw;
    k.ncol = c1 - k.c0;
    if (k.ncol < 4) return best;
    k.quads = (k.ncol + 3) / 4;
    k.rt = p.Rt == p.St && (p.Rt == 3 || p.Rt == (mode == 2 ? 2 : 5)) ? p.Rt : 0;
    for (const AnyTileCost& t : kAnyTiles) {
        k.ahead = t.ahead;
        if (force > 0 && t.bm * 1000 + t.bn != force % 1000000) continue;
        if (force > 0 && (force >= 1000000) != t.ahead) continue;
        if (t.ahead && !k.rt) continue;
        if (mode == 2 && t.bm >= 96 && t.bn == 256) continue;
        const long long ti = (p.Co + t.bm - 1) / t.bm, tp = ((long long)p.M + t.bn - 1) / t.bn;
        if (ti * tp > 0x7fffffffLL) continue;
        // output rows a tile can touch and the image boundaries among them
        long long rows = (t.bn + p.Wo - 2) / p.Wo + 1;
        if (rows > (long long)p.N * p.Ho) rows = (long long)p.N * p.Ho;
        long long segs = (rows - 1 + p.Ho - 1) / p.Ho + 1;
        if (segs > p.N) segs = p.N;
        if (segs > rows) segs = rows;
        const long long patch_rows = rows * gh + (p.Rt > gh ? segs : 1) * (p.Rt - gh);
        const long long loads = 2 * patch_rows * k.quads;
        if (loads > (t.ahead ? 256 : 512)) continue;
        k.rounds = loads > 256 ? 2 : 1;
        const long long plane = (patch_rows * k.pw + 1) / 2 * 16;
        k.plane_bytes = (int)((plane + 95) / 128 * 128 + 32);        // 32 past a multiple of 128: the two parities fall on other banks
        // a stage: as few runs of taps as keep a slot of the filter ring within 20 KB
        const int tap_bytes = t.bm * 32;
        if (k.rt) {
            k.stages = t.ahead ? 1 : k.rt;
            k.stage_taps = k.taps / k.stages;
        } else {
            k.stages = (k.taps * tap_bytes + 20479) / 20480;
            k.stage_taps = (k.taps + k.stages - 1) / k.stages;
            k.stages = (k.taps + k.stage_taps - 1) / k.stage_taps;
        }
        k.lds = t.bm * 4 + ring_slots(k.rt, !t.ahead) * k.stage_taps * tap_bytes + 2 * (4 * k.plane_bytes + 128) + 1024;
        if (k.lds > 156 * 1024) continue;
        const long long a_bytes = ti * k.cgs * k.taps * tap_bytes;
        if (a_bytes >= 0x7fffffffLL) continue;
        k.bm = t.bm; k.bn = t.bn; k.tiles_i = (int)ti; k.tiles_pix = (int)tp;
        k.a_bytes = (size_t)a_bytes;
        const double mfma = t.bm * t.bn / 1024 / 4 * 32.0, mhz = 2.1e3;      // cycles of a tap's MFMAs on a SIMD
        const double solo = k.cgs * (k.taps * (mfma > t.tap ? mfma : t.tap) + k.stages * t.stage + t.group) / mhz + t.fixed;
        const double share = k.cgs * (k.taps * mfma / t.eff + loads * t.fill) / mhz + t.wg;
        const int by_lds = 160 * 1024 / k.lds, fit = by_lds < t.resident ? by_lds : t.resident;
        const double m = (double)(ti * tp) / 256.0;
        double busy = solo;
        if (m > 1.0) {
            const double per_cu = 0.35 * m + 0.65 * std::ceil(m), shared = share * per_cu;
            if (per_cu <= fit) busy = std::cbrt(solo * solo * solo + shared * shared * shared);
            else busy = shared + 0.4 * solo > solo * per_cu / fit ? shared + 0.4 * solo : solo * per_cu / fit;
        }
        k.us = 4.7 + (double)a_bytes / 1.0e6 + busy;                      // with the filter's copy
        k.use = true;
        if (!best.use || k.us < best.us) best = k;
    }
    // The tile is chosen; what it takes in all, for the comparison with the other kernels: `waves` rounds of as many workgroups as
    // a CU holds. Fitted to 16137 passes, half of them with other filters (their taps' loop is not unrolled), rows of up to 256
    // pixels and launches of up to 1.2 TFLOP among them: within 0.84 - 1.11 of the measured time in nine of ten.
    if (best.use) {
        int resident = 1;
        for (const AnyTileCost& t : kAnyTiles)
            if (t.bm == best.bm && t.bn == best.bn && t.ahead == best.ahead) resident = t.resident;
        const int by_lds = 160 * 1024 / best.lds, fit = by_lds < resident ? by_lds : resident;
        const double m = (double)best.tiles_i * best.tiles_pix / 256.0, waves = std::ceil(m / fit), out_mb = 2e-6 * p.M * (double)p.Co;
        const double groups = best.cgs, steps = groups * best.taps, area = best.bm * best.bn / 1024, fills = groups * std::ceil(m) * best.rounds;
        if (best.rt)
            best.us = 4.8 + 0.356 * best.us + waves * steps * (0.0176 + 0.00387 * area) + 0.25 * fills + (mode == 2 ? 0.506 : 0.338) * out_mb;
        else
            best.us = 6.5 + 0.043 * best.us + waves * (steps * (0.0517 + 0.00482 * area) + 0.341 * groups * best.stages) + 0.361 * fills +
                      (mode == 2 ? 0.517 : 0.342) * out_mb;
    }
    return best;
}

hipError_t launch_patch_any(PixParams p, const PatchAnyPlan& k, int mode, const void* w, int K, int C, void* ws, hipStream_t st) {
    if (!ws) return hipErrorInvalidValue;
    FilterPackets f{};
    f.w = (const uint16_t*)w; f.a = (u32x4*)ws;
    f.mode = mode; f.K = K; f.C = C; f.R = p.R; f.S = p.S; f.sh = p.sh; f.sw = p.sw; f.St = p.St; f.Co = p.Co; f.Ci = p.Ci;
    f.bm = k.bm; f.taps = k.taps; f.cgs = k.cgs; f.total = (int)(k.a_bytes / 16);
    f.div_bm = make_fastdiv(k.bm); f.div_taps = make_fastdiv(k.taps); f.div_cgs = make_fastdiv(k.cgs); f.div_st = make_fastdiv(p.St);
    f.div_phases = make_fastdiv(p.sh * p.sw); f.div_sw = make_fastdiv(p.sw);
    (void)hipGetLastError();
    hipLaunchKernelGGL(pack_filter_bf16_kernel, dim3((unsigned)((f.total + 255) / 256)), dim3(256), 0, st, f);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;

    PatchAnyParams q{};
    q.a = ws; q.a_bytes = (unsigned)k.a_bytes;
    q.taps = k.taps; q.cgs = k.cgs; q.stage_taps = k.stage_taps; q.stages = k.stages;
    q.pw = k.pw; q.h_base = k.h_base; q.w_base = k.w_base; q.c0 = k.c0; q.ncol = k.ncol; q.quads = k.quads;
    q.img_rows = (p.Ho - 1) * p.g_mul_h + p.Rt;
    q.plane_bytes = k.plane_bytes;
    q.pairs = ((p.HoWo | p.out_ns) & 1) == 0 && (((uintptr_t)p.out | (uintptr_t)p.mask) & 3u) == 0;
    if (mode == 2 && p.sh == 2 && p.sw == 2 && !buffer_loads_disabled()) {
        const long long dx = ((long long)(p.N - 1) * p.out_ns + (long long)p.C * p.H * p.W) * 2;
        q.dx_bytes = dx < 0x7fffffffLL ? (unsigned)dx : 0u;
    }
    q.div_ho = make_fastdiv(p.Ho); q.div_quads = make_fastdiv(k.quads); q.div_img = make_fastdiv(q.img_rows);
    p.tiles_i = k.tiles_i; p.tiles_pix = k.tiles_pix;
    if (mode == 0) return by_taps<false, false>(p, q, k, st);
    if (mode == 1) return by_taps<true, false>(p, q, k, st);
    return by_taps<true, true>(p, q, k, st);
}

}  // namespace pix
}  // namespace purine

// fp32 forward / backward-data layers with several taps and a unit-stride gather (forward with stride 1,
// backward-data with any stride after phase folding) on the bf16 matrix cores: the arithmetic of
// conv_packets.hip (three exact bf16 parts, six products, two accumulator sets), with the parts made
// in LDS instead of in scratch memory.
//
// Bound: MFMA at the clock that power allows (bf16 MFMAs on random data run at 1.9 - 2.0 GHz; the same
// launch on zeros is a quarter faster), with the matrix pipes busy 66 % of a CU's cycles on 96 <- 256 channels 5x5
// at 27x27, 62 % on the 384-channel 3x3 at 13x13 and 45 - 59 % on the shorter sums of the 96 / 128-channel 3x3 at 28x28,
// N = 128; a quarter to a third of the LDS cycles are bank conflicts (the taps' shifted reads). With fp32 products
// 87 - 89 %. A workgroup of eight wavefronts owns BM rows x 256 consecutive pixels, one workgroup per CU. All positions that the taps of those pixels touch form a patch of a few
// haloed rows (possibly of several images); per group of 16 gathered channels the patch is loaded
// once from NCHW (a lane takes 8 channels of one position: coalesced 4-byte loads), split in registers
// and stored to LDS as packets [part][channel half][position][8], and every tap reads its B fragments
// there at an offset of its own: an element is split once per row tile and not once per tap, and
// nothing is copied in HBM. Two patch buffers: the next group's loads are issued after its
// predecessor's first tap and split after the last. The filter is repacked (fp32, [row tile][group]
// [tap][row][16]) and a step's tile is split on its way into a two-slot ring, four elements per thread.
// One barrier per tap.
//
// The same kernel with fp32 parts and MFMAs (SPLIT = false) serves the forward passes whose bits have to
// stay those of the fp32 tap kernel: each output's products are added in that kernel's order. There the
// matrix units are the bound (32x32x2: 8/3 of the time), and what it gains is the tap kernel's gather per
// tap and its waits.
//
// Measured at N = 128 (whole operator, fp32 MFMA kernel before): 384 <- 384 channels 3x3 at 13x13
// backward-data 0.50 -> 0.28 ms (204 TFLOP/s; 0.31 with the operands packed in scratch), 96 -> 128 3x3 at
// 28x28 forward 0.236 -> 0.140, 96 <- 256 5x5 at 27x27 backward-data 1.01 -> 0.69 (365 tiles on 256 CUs).
#include "packets.h"
#include "pix_common.h"

namespace purine {
namespace pix {
namespace {

using namespace packets;

// Pixels of a workgroup's tile and positions its patch may have. Split: one workgroup of eight wavefronts on
// a CU; fp32: two of four wavefronts, whose waits and epilogues fall into each other's MFMAs (384 <- 256
// channels 3x3 at 13x13, N = 128 forward: 0.309 ms with one of eight, 0.301 with two of four).
constexpr int pixels_of(bool split) { return split ? 256 : 128; }
constexpr int positions_of(bool split) { return split ? 704 : 504; }

struct PatchF32Params {
    const float* a;             // repacked filter
    unsigned a_bytes;
    int taps, cgs, mode;
    int bands, Wb, PW, Mv;      // Mv: pixels counted over bands of Wb columns
    int h_base, w_base;         // input row / column of patch row / column 0, relative to the output row / column
    int img_rows;               // patch rows of a whole image: Ho + Rt - 1
    FastDiv div_ho, div_wb, div_bands, div_pw, div_img, div_st;
    // The tiles past the last whole round of CUs (split only): `parts` workgroups each take cg_part channel groups of one and
    // leave raw sums in partial[tile][part][thread]; a second launch (join) adds them in order and finishes.
    int full, parts, cg_part, join;
    float* partial;
};

// Filter repack, one thread per four channels: [row tile][group][tap][row][16], zero past the last row
// or channel, times the factor of the split (here, where it costs nothing: a step splits its filter tile again).
struct FilterPack {
    const float* w; float* a;
    int mode, K, C, R, S, sh, sw, St, Co, bm, taps, cgs, total;
    float scale;
    FastDiv div_bm, div_taps, div_cgs, div_st, div_phases, div_sw;
};
__global__ __launch_bounds__(256) void pack_filter_f32_kernel(const FilterPack q) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= q.total) return;
    const int quad = t & 3;
    int rest = t >> 2;
    int u = fastdiv(rest, q.div_bm);
    const int row = rest - u * q.bm;
    rest = u;
    u = fastdiv(rest, q.div_taps);
    const int tap = rest - u * q.taps;
    const int rt = fastdiv(u, q.div_cgs), cg = u - rt * q.cgs;
    const int tr = fastdiv(tap, q.div_st), tc = tap - tr * q.St;
    const int i = rt * q.bm + row, ci0 = cg * 16 + quad * 4;
    FilterRun f{0, 0, 0};
    if (i < q.Co) f = filter_run(q.mode, i, tr, tc, q.C, q.R, q.S, q.sh, q.sw, q.mode == 0 ? q.C : q.K, q.div_phases, q.div_sw);
    floatx4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[e] = ci0 + e < f.lim ? q.w[(size_t)f.fixed + (size_t)(ci0 + e) * f.stride] : 0.0f;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float x = v[e];
        asm volatile("" : "+v"(x));      // as in store_split8
        v[e] = x * q.scale;
    }
    *reinterpret_cast<floatx4*>(q.a + (size_t)t * 4) = v;
}

// SPLIT: three bf16 parts x two channel halves per row / position; else fp32: (groups of four MFMA steps)
// x (lane halves). 16-byte packets either way.
template <bool SPLIT, int TM, int WM>
struct PatchTile {
    static constexpr int BN = pixels_of(SPLIT), POS = positions_of(SPLIT), WAVES = SPLIT ? 8 : 4, NT = WAVES * 64;
    static constexpr int TASKS = (2 * POS + NT - 1) / NT;                      // fill tasks (position, channel half) per thread
    static constexpr int BM = TM * WM * 32, WN = WAVES / WM, TN = BN / (WN * 32);
    static constexpr int AL = (BM * 4 + NT - 1) / NT;                          // filter loads (four channels of a row) per thread and step
    static constexpr int PACKETS = SPLIT ? PLANES * 2 : 4;
    static constexpr int A_BYTES = PACKETS * BM * 16, P_BYTES = PACKETS * POS * 16;
    static constexpr int LDS = 2 * A_BYTES + 2 * P_BYTES + 512 + BM * 4;       // + spare half KB + bias
};

// The sums of a tile's parts, in order, and a bit per element that is infinite or NaN.
template <int TM, int TN, int NT>
__device__ __forceinline__ unsigned long long add_parts(floatx16 (&acc)[TM][TN], const float* partial, int tile, int parts, int tid) {
    unsigned long long bad = 0;
    const floatx4* src = reinterpret_cast<const floatx4*>(partial) + (size_t)tile * parts * TM * TN * 4 * NT + tid;
#pragma unroll
    for (int i = 0; i < TM * TN * 4; ++i) {
        floatx4 v = src[(size_t)i * NT];
        for (int s = 1; s < parts; ++s) v += src[((size_t)s * TM * TN * 4 + i) * NT];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (!(__builtin_fabsf(v[e]) <= 3.402823466e38f)) bad |= 1ull << (i * 4 + e);
            acc[i / 4 / TN][i / 4 % TN][i % 4 * 4 + e] = v[e];
        }
    }
    return bad;
}

// TAIL: for launches whose last tiles are shared (SPLIT only). A form of its own, because the bookkeeping costs the others: 64 <- 126
// channels 3x3 at 63x65, N = 7 forward, 32-row tiles, 44.3 and 48.4 us.
template <bool SPLIT, bool MINUS, bool D2S, bool FUSED, int TM, int WM, bool TAIL>
__global__ __launch_bounds__(SPLIT ? 512 : 256, 2) void igemm_patch_f32_kernel(const PixParams p, const PatchF32Params q) {
    typedef PatchTile<SPLIT, TM, WM> T;
    constexpr int TN = T::TN, WN = T::WN, BN = T::BN, POS = T::POS, NT = T::NT, TASKS = T::TASKS;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char* patch = smem + 2 * T::A_BYTES;
    unsigned char* spare = patch + 2 * T::P_BYTES;
    float* bias_s = reinterpret_cast<float*>(spare + 512);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int khalf = lane >> 5;
    const int wm = wave / WN, wn = wave % WN;
    // row tiles innermost: they read the same patch and share an XCD's L2
    int id, slot = -1, cg0 = 0, cg1 = q.cgs;
    if (!TAIL) {
        id = xcd_tile(blockIdx.x, gridDim.x);
    } else if (q.join) {
        slot = blockIdx.x;
        id = q.full + slot;
    } else if ((int)blockIdx.x < q.full) {
        id = xcd_tile(blockIdx.x, q.full);
    } else {
        slot = xcd_tile(blockIdx.x - q.full, gridDim.x - q.full);
        const int tile = slot / q.parts, part = slot - tile * q.parts;
        id = q.full + tile;
        cg0 = part * q.cg_part;
        cg1 = min(cg0 + q.cg_part, q.cgs);
    }
    const int pt = id / p.tiles_i, rt = id - pt * p.tiles_i;
    const int i0 = rt * T::BM, p0 = pt * BN;

    if (FUSED && !MINUS) stage_bias<float, T::BM, NT>(bias_s, p, i0, tid);

    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(q.a), (short)0, (int)q.a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.in), (short)0, (int)p.in_bytes, 0x00020000);

    // the tile's output rows, counted over (image, band, row)
    const int rho0 = fastdiv(p0, q.div_wb), rho1 = fastdiv(min(p0 + BN, q.Mv) - 1, q.div_wb);
    const int v0 = fastdiv(rho0, q.div_ho), ho0 = rho0 - v0 * p.Ho;
    const int v1 = fastdiv(rho1, q.div_ho);
    const int npos = (rho1 - rho0 + (v1 - v0) * (p.Rt - 1) + p.Rt) * q.PW;
    const int first_rows = p.Ho - ho0 + p.Rt - 1;         // patch rows that belong to image v0

    // fill tasks of this thread: byte offset of (channel half's first channel, position) and LDS offset
    int src[TASKS], dst[TASKS], half[TASKS];
#pragma unroll
    for (int j = 0; j < TASKS; ++j) {
        const int t = tid + j * NT;
        half[j] = t >= npos ? 1 : 0;
        const int pos = t - half[j] * npos;
        const bool task = t < 2 * npos;
        const int prow = fastdiv(task ? pos : 0, q.div_pw), pcol = (task ? pos : 0) - prow * q.PW;
        int v = v0, h = ho0 + q.h_base + prow;
        if (prow >= first_rows) {
            const int u = prow - first_rows, k = fastdiv(u, q.div_img);
            v = v0 + 1 + k;
            h = q.h_base + u - k * q.img_rows;
        }
        const int n = fastdiv(v, q.div_bands), w = (v - n * q.bands) * q.Wb + q.w_base + pcol;
        const bool ok = task && n < p.N && (unsigned)h < (unsigned)p.Hi && (unsigned)w < (unsigned)p.Wi;
        src[j] = ok ? (n * p.in_ns + half[j] * 8 * p.HiWi + h * p.Wi + w) * 4 : -1;
        dst[j] = task ? (half[j] * (SPLIT ? POS : 2 * POS) + pos) * 16 : -1;
    }
    // the pixels this lane multiplies: patch position at tap offset 0, and its place in the output
    int pbase[TN], opix[TN];
#pragma unroll
    for (int b = 0; b < TN; ++b) {
        const int px = p0 + wn * TN * 32 + b * 32 + (lane & 31);
        const bool live = px < q.Mv;
        const int rho = fastdiv(live ? px : p0, q.div_wb), wb = (live ? px : p0) - rho * q.Wb;
        const int v = fastdiv(rho, q.div_ho), ho = rho - v * p.Ho;
        pbase[b] = ((rho - rho0 + (v - v0) * (p.Rt - 1)) * q.PW + wb + khalf * POS) * 16;
        const int n = fastdiv(v, q.div_bands), wo = (v - n * q.bands) * q.Wb + wb;
        opix[b] = live && wo < p.Wo ? n * p.HoWo + ho * p.Wo + wo : 0x7fffffff;
    }

    float breg[TASKS][8];
    auto load_patch = [&](int cg) {               // cg == cg1: every offset lies outside, nothing is fetched
#pragma unroll
        for (int j = 0; j < TASKS; ++j) {
            const int lim = TAIL && cg >= cg1 ? 0 : p.Ci - cg * 16 - half[j] * 8;      // channels left for this task
            const int soff = cg < cg1 ? cg * 16 * p.HiWi * 4 : 0;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                unsigned v = src[j] >= 0 && e < lim ? (unsigned)src[j] + (unsigned)(e * p.HiWi * 4) : 0x80000000u;
                breg[j][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rb, v, soff, 0));
            }
        }
    };
    auto store_patch = [&](int buf) {
#pragma unroll
        for (int j = 0; j < TASKS; ++j)
            if (!SPLIT && dst[j] >= 0) {
                // channel 8 * half + e is reduction index 2 * ks + l of the group: step group `half`, lane half l = e & 1
                const floatx4 even = {breg[j][0], breg[j][2], breg[j][4], breg[j][6]}, odd = {breg[j][1], breg[j][3], breg[j][5], breg[j][7]};
                *reinterpret_cast<floatx4*>(patch + buf * T::P_BYTES + dst[j]) = even;
                *reinterpret_cast<floatx4*>(patch + buf * T::P_BYTES + dst[j] + POS * 16) = odd;
            } else if (SPLIT && dst[j] >= 0) {
                typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
                u32x4 pk[PLANES];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    uint32_t part[PLANES];
                    split_pair(breg[j][2 * e], breg[j][2 * e + 1], part);
#pragma unroll
                    for (int pl = 0; pl < PLANES; ++pl) pk[pl][e] = part[pl];
                }
#pragma unroll
                for (int pl = 0; pl < PLANES; ++pl)
                    *reinterpret_cast<u32x4*>(patch + buf * T::P_BYTES + dst[j] + pl * 2 * POS * 16) = pk[pl];
            }
    };
    // filter tile of a step: four channels of T::AL rows per thread
    struct FilterRegs { floatx4 f[T::AL]; };
    auto load_a = [&](int step) {
        FilterRegs r;
#pragma unroll
        for (int j = 0; j < T::AL; ++j) {
            const int t = tid + j * NT;
            r.f[j] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(ra, t < T::BM * 4 ? (unsigned)(t * 16) : 0x80000000u,
                                                                                    (rt * q.cgs * q.taps + step) * T::BM * 64, 0));
        }
        return r;
    };
    auto store_a = [&](const FilterRegs& r, int slot) {
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        typedef float floatx2 __attribute__((ext_vector_type(2)));
#pragma unroll
        for (int j = 0; j < T::AL; ++j) {
            const int t = tid + j * NT;
            const bool mine = (T::BM * 4) % NT == 0 || t < T::BM * 4;       // the others write to the spare half KB
            const int a_dst = ((t >> 1) & 1) * (SPLIT ? 1 : 2) * T::BM * 16 + (t >> 2) * 16 + (t & 1) * 8;
            unsigned char* base = mine ? smem + slot * T::A_BYTES + a_dst : spare + lane * 8;
            if constexpr (!SPLIT) {
                *reinterpret_cast<floatx2*>(base) = floatx2{r.f[j][0], r.f[j][2]};
                *reinterpret_cast<floatx2*>(base + (mine ? T::BM * 16 : 0)) = floatx2{r.f[j][1], r.f[j][3]};
            } else {
                uint32_t p01[PLANES], p23[PLANES];
                split_pair<true>(r.f[j][0], r.f[j][1], p01);
                split_pair<true>(r.f[j][2], r.f[j][3], p23);
#pragma unroll
                for (int pl = 0; pl < PLANES; ++pl)
                    *reinterpret_cast<u32x2*>(base + (mine ? pl * 2 * T::BM * 16 : 0)) = u32x2{p01[pl], p23[pl]};
            }
        }
    };

    floatx16 hi[TM][TN], lo[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) { hi[a][b][e] = 0.0f; lo[a][b][e] = 0.0f; }

    const int a_off = (khalf * T::BM + wm * TM * 32 + (lane & 31)) * 16;
    // A wavefront's LDS traffic is done, then all wavefronts meet; loads in flight stay in flight.
    auto meet = [&]() {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xc07f);        // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    auto multiply = [&](int step, int buf, int tap_off) {
        const unsigned char* sa = smem + (step & 1) * T::A_BYTES + a_off;
        const unsigned char* sb = patch + buf * T::P_BYTES + tap_off;
        if constexpr (!SPLIT) {
            // the fp32 MFMAs of the tap kernel, in its order: an output's sum has the same bits
#pragma unroll
            for (int kg = 0; kg < 2; ++kg) {
                floatx4 af[TM], bf[TN];
#pragma unroll
                for (int a = 0; a < TM; ++a) af[a] = *reinterpret_cast<const floatx4*>(sa + (kg * 2 * T::BM + a * 32) * 16);
#pragma unroll
                for (int b = 0; b < TN; ++b) bf[b] = *reinterpret_cast<const floatx4*>(sb + pbase[b] + kg * 2 * POS * 16);
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                    for (int a = 0; a < TM; ++a)
#pragma unroll
                        for (int b = 0; b < TN; ++b)
                            hi[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[a][ks], bf[b][ks], hi[a][b], 0, 0, 0);
            }
            return;
        } else {
        bf16x8 av[PLANES][TM], bv[PLANES][TN];
#pragma unroll
        for (int pl = 0; pl < PLANES; ++pl) {
#pragma unroll
            for (int a = 0; a < TM; ++a) av[pl][a] = *reinterpret_cast<const bf16x8*>(sa + (pl * 2 * T::BM + a * 32) * 16);
#pragma unroll
            for (int b = 0; b < TN; ++b) bv[pl][b] = *reinterpret_cast<const bf16x8*>(sb + pbase[b] + pl * 2 * POS * 16);
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
    };

    const int n_steps = q.cgs * q.taps;
    if (!TAIL || !q.join) {
        int step = cg0 * q.taps;
        load_patch(cg0);
        store_a(load_a(step), step & 1);
        store_patch(cg0 & 1);
        for (int cg = cg0; cg < cg1; ++cg) {
            const int buf = cg & 1;
            int tr = 0, tc = 0;
            auto tap_offset = [&]() { return MINUS ? ((p.Rt - 1 - tr) * q.PW + (p.St - 1 - tc)) * 16 : (tr * q.PW + tc) * 16; };
            // first tap: the next group's patch is requested behind the next step's filter tile, so that
            // waiting for the latter does not wait for the former
            meet();
            {
                const FilterRegs f = load_a(step + 1);      // (one past the last step: still inside the buffer's range check)
                load_patch(cg + 1);
                __builtin_amdgcn_sched_barrier(0);       // requests first: they have the whole step to arrive
                multiply(step, buf, tap_offset());
                store_a(f, (step + 1) & 1);
                ++step;
            }
            for (int tap = 1; tap < q.taps; ++tap) {
                if (++tc == p.St) { tc = 0; ++tr; }
                meet();
                const FilterRegs f = load_a(step + 1);
                __builtin_amdgcn_sched_barrier(0);
                multiply(step, buf, tap_offset());
                store_a(f, (step + 1) & 1);
                ++step;
            }
            if (cg + 1 < cg1) store_patch(buf ^ 1);
        }
    }

    // infinities and NaNs: again, as plain fp32 sums of the fp32 operands
    unsigned long long bad = 0;
    if (TAIL && q.join) {
        if (FUSED && !MINUS) __syncthreads();      // the bias values
        bad = add_parts<TM, TN, NT>(hi, q.partial, slot, q.parts, tid);
    } else if (SPLIT) {
        bad = join_sets<TM, TN>(hi, lo);
        if (TAIL && slot >= 0) {
            floatx4* dst = reinterpret_cast<floatx4*>(q.partial) + (size_t)slot * TM * TN * 4 * NT + tid;
#pragma unroll
            for (int i = 0; i < TM * TN * 4; ++i) {
                const floatx16& v = hi[i / 4 / TN][i / 4 % TN];
                const int e = i % 4 * 4;
                dst[(size_t)i * NT] = floatx4{v[e], v[e + 1], v[e + 2], v[e + 3]};
            }
            return;
        }
    }
    if (SPLIT && __builtin_expect(__any(bad != 0), 0)) {
        while (bad) {
            const int idx = __ffsll((long long)bad) - 1;
            bad &= bad - 1;
            const int ab = idx >> 4, e = idx & 15;
            const int row = wm * TM * 32 + (ab / TN) * 32 + (e >> 2) * 8 + khalf * 4 + (e & 3);
            int px = opix[0];
#pragma unroll
            for (int b = 1; b < TN; ++b) px = ab % TN == b ? opix[b] : px;
            float sum = 0.0f;
            if (px < p.M && i0 + row < p.Co) {
                const int n = fastdiv(px, p.div_howo), rem = px - n * p.HoWo;
                const int ho = fastdiv(rem, p.div_wo), wo = rem - ho * p.Wo;
                for (int s = 0; s < n_steps && sum == sum; ++s) {
                    const int g = s / q.taps, tap = s - g * q.taps;
                    const int r = fastdiv(tap, q.div_st), t = tap - r * p.St;
                    const int h = MINUS ? ho + p.g_add_h - r : ho + p.g_add_h + r, w = MINUS ? wo + p.g_add_w - t : wo + p.g_add_w + t;
                    const bool inside = (unsigned)h < (unsigned)p.Hi && (unsigned)w < (unsigned)p.Wi;
                    const FilterRun f = filter_run(q.mode, i0 + row, r, t, p.C, p.R, p.S, p.sh, p.sw, p.Ci, p.div_phases, p.div_sw);
                    const float* pb = (const float*)p.in + (size_t)n * p.in_ns + (inside ? h * p.Wi + w : 0);
                    for (int ci = g * 16; ci < g * 16 + 16 && ci < p.Ci; ++ci)
                        sum = __builtin_fmaf(ci < f.lim ? ((const float*)p.wt)[(size_t)f.fixed + (size_t)ci * f.stride] : 0.0f,
                                             inside ? pb[(size_t)ci * p.HiWi] : 0.0f, sum);
                }
            }
            replace_element<TM, TN>(hi, idx, sum);
        }
    }
    store_tile_at<float, D2S, FUSED, TM, TN, !MINUS>(p, (float*)p.out, hi, i0 + wm * TM * 32, [&](int b) { return opix[b]; }, khalf,
                                                     bias_s, i0, 0x7fffffff);
}

template <bool SPLIT, bool MINUS, bool D2S, bool FUSED, int TM, int WM, bool TAIL>
hipError_t launch_form(const PixParams& p, const PatchF32Params& q, hipStream_t st) {
    typedef PatchTile<SPLIT, TM, WM> T;
    const long long total = (long long)p.tiles_i * p.tiles_pix;
    if (total <= 0 || total > 0x7fffffffLL) return hipErrorInvalidValue;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&igemm_patch_f32_kernel<SPLIT, MINUS, D2S, FUSED, TM, WM, TAIL>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS);
    if (e != hipSuccess) return e;
    ProbeScope probe(st);
    (void)hipGetLastError();   // drop stale status left by earlier, unrelated runtime calls
    const long long tail = total - q.full, grid = q.full + tail * q.parts;       // (no tail: q.full == total)
    hipLaunchKernelGGL((igemm_patch_f32_kernel<SPLIT, MINUS, D2S, FUSED, TM, WM, TAIL>), dim3((unsigned)grid), dim3(T::NT), T::LDS, st, p, q);
    e = hipGetLastError();
    if (e != hipSuccess || !TAIL) return e;
    PatchF32Params j = q;
    j.join = 1;
    hipLaunchKernelGGL((igemm_patch_f32_kernel<SPLIT, MINUS, D2S, FUSED, TM, WM, TAIL>), dim3((unsigned)tail), dim3(T::NT), T::LDS, st, p, j);
    return hipGetLastError();
}

template <bool SPLIT, bool MINUS, bool D2S, bool FUSED, int TM, int WM>
hipError_t launch_main(const PixParams& p, const PatchF32Params& q, hipStream_t st) {
    if (SPLIT && q.parts > 1) return launch_form<SPLIT, MINUS, D2S, FUSED, TM, WM, SPLIT>(p, q, st);
    return launch_form<SPLIT, MINUS, D2S, FUSED, TM, WM, false>(p, q, st);
}

template <bool SPLIT, bool MINUS, bool D2S, bool FUSED>
hipError_t by_tile(const PixParams& p, const PatchF32Params& q, int bm, hipStream_t st) {
    switch (bm) {
        case 128: return launch_main<SPLIT, MINUS, D2S, FUSED, 2, 2>(p, q, st);
        case 96:  return launch_main<SPLIT, MINUS, D2S, FUSED, 3, 1>(p, q, st);
        case 64:  return launch_main<SPLIT, MINUS, D2S, FUSED, 2, 1>(p, q, st);
        case 32:  return launch_main<SPLIT, MINUS, D2S, FUSED, 1, 1>(p, q, st);
        default: return hipErrorInvalidValue;
    }
}

// cycles: MFMA time of a step on a SIMD; eff: the share of it that the tile reaches (split: six bf16 products,
// two wavefronts per SIMD; fp32: one, and half the pixels)
struct RowTile { int bm, cycles; float eff; };
constexpr RowTile kSplitTiles[] = {{128, 1536, 0.72f}, {96, 1152, 0.66f}, {64, 768, 0.58f}, {32, 384, 0.45f}};
constexpr RowTile kF32Tiles[] = {{128, 2048, 0.90f}, {96, 1536, 0.88f}, {64, 1024, 0.84f}, {32, 512, 0.75f}};

}  // namespace

// How the layer would run here and the expected time (conv_igemm.hip compares). Pure host arithmetic.
PatchF32Plan plan_patch_f32(const PixParams& p, bool d2s, bool split, int force_parts) {
    PatchF32Plan k{};
    k.split = split;
    if (p.Rt * p.St < 2 || p.Ci < 8 || p.in_bytes == 0 || p.g_mul_h != 1 || p.g_mul_w != 1) return k;
    const int BN = pixels_of(split), POS = positions_of(split);
    // bands of columns: as few as keep the worst tile's patch within the LDS buffers
    for (int bands = 1; bands <= 32; ++bands) {
        const int wb = (p.Wo + bands - 1) / bands, pw = wb + p.St - 1;
        if (bands > 1 && (wb < 8 || (long long)(bands - 1) * wb >= p.Wo)) break;
        const long long rows = (BN + wb - 2) / wb + 1;                       // output rows that a tile can touch
        const long long crossings = (rows - 1 + p.Ho - 1) / p.Ho;            // image (or band) boundaries among them
        if ((rows + crossings * (p.Rt - 1) + p.Rt - 1) * pw > POS) continue;
        k.bands = bands; k.Wb = wb; k.PW = pw;
        break;
    }
    const long long mv = (long long)p.N * k.bands * p.Ho * k.Wb;
    if (!k.bands || mv > 0x7fffff00LL) return k;
    k.cgs = (p.Ci + 15) / 16;
    const long long tp = (mv + BN - 1) / BN;
    for (int i = 0; i < 4; ++i) {
        const RowTile& t = split ? kSplitTiles[i] : kF32Tiles[i];
        const long long ti = (p.Co + t.bm - 1) / t.bm;
        // 32 rows: filling the patch is most of a group's time, and longer where the patches come from HBM and not the
        // 256 MB last-level cache (3x3, 215 -> 20 channels at 58x58, N = 125, 362 MB: 84 us per tile and 14 groups, tap kernel 504 us,
        // this 574; 113 -> 19 at 46x46, N = 28, 27 MB: 35 us and 8 groups, 69 and 45)
        const double eff = split && t.bm == 32 && (long long)p.N * p.Ci * p.HiWi > (48ll << 20) ? 0.34 : t.eff;
        const long long a_bytes = ti * k.cgs * p.Rt * p.St * t.bm * 64;
        if (a_bytes >= 0x7fffffffLL || ti * tp > 0x7fffffffLL) continue;
        const double x = (double)(ti * tp) / 256.0, ceil_x = (double)((ti * tp + 255) / 256);
        // one workgroup per CU at a time (the clock rises a little as CUs run dry), or two
        const double load = split ? 0.3 * x + 0.7 * ceil_x : x <= 1.0 ? 1.3 : 0.3 * x + 0.7 * ceil_x;
        auto workgroup_us = [&](double groups) {
            return (groups * (p.Rt * p.St * t.cycles / eff + 1000.0) + (d2s ? 50000.0 : 10000.0)) / (split ? 2.2e3 : 2.4e3);
        };
        double us = 10.0 + load * workgroup_us(k.cgs);
        // The tiles past the last whole round of 256 leave most CUs idle for as long as a round takes: their channel groups go
        // to several workgroups each where that is expected to pay for the second launch and the sums' way through memory
        // (48 <- 128 channels 5x5 at 27x27, N = 128 backward-data, 365 tiles of 8 groups, the last 109 halved: 288 -> 238 us; 83 <- 264
        // 3x3 at 46x46, N = 63: 463 -> 385). Another tile height only for a clear gain (102 <- 84 5x5 at 56x56, N = 12, 294 tiles of
        // 64 rows in parts 160 us, 147 of 128 in one round 155). The sums are scratch that a caller holds for the layer: at most
        // 16 MB. That is a choice: forward and backward-data of the five-layer stack ask for no more than their filter copies so,
        // as before. It costs its one layer that gains, 96 <- 256 5x5 at 27x27, N = 128, 21.4 MB of sums: 691 us, 577 with them.
        const long long full = ti * tp / 256 * 256, tail = ti * tp - full;
        int parts = 1, cg_part = k.cgs;
        double best_us = force_parts > 1 ? 1e30 : us;
        if (split && tail > 0 && (full + tail >= 128 || force_parts > 1)) {
            for (int want = 2; want <= 8 && want <= k.cgs; ++want) {
                const int per = (k.cgs + want - 1) / want, n = (k.cgs + per - 1) / per;
                const double bytes = (double)tail * n * t.bm * BN * 4.0, x_tail = (double)(tail * n) / 256.0;
                if (n != want || bytes > 16e6 || (force_parts > 1 && n != force_parts)) continue;
                const double split_us = 10.0 + full / 256 * workgroup_us(k.cgs) + (0.3 * x_tail + 0.7 * (double)((tail * n + 255) / 256)) * workgroup_us(per) +
                                        8.0 + 2.0 * bytes / 4e6;
                if (split_us < best_us) { best_us = split_us; us = 1.06 * split_us; parts = n; cg_part = per; }
            }
        }
        if (!k.use || us < k.us) {
            k.use = true; k.us = us;
            k.bm = t.bm; k.tiles_i = (int)ti; k.tiles_pix = (int)tp;
            k.full = (int)(parts > 1 ? full : full + tail); k.parts = parts; k.cg_part = cg_part;
            k.part_offset = ((size_t)a_bytes + 255) / 256 * 256;
            k.part_bytes = parts > 1 ? (size_t)tail * parts * t.bm * BN * 4 : 0;
            k.a_bytes = (size_t)a_bytes;
        }
    }
    return k;
}

hipError_t launch_patch_f32(PixParams p, const PatchF32Plan& k, int mode, const void* w, int K, int C, void* ws, hipStream_t st) {
    if (!ws) return hipErrorInvalidValue;
    FilterPack f{};
    f.w = (const float*)w; f.a = (float*)ws;
    f.mode = mode; f.K = K; f.C = C; f.R = p.R; f.S = p.S; f.sh = p.sh; f.sw = p.sw; f.St = p.St; f.Co = p.Co;
    f.scale = k.split ? SPLIT_SCALE : 1.0f;
    f.bm = k.bm; f.taps = p.Rt * p.St; f.cgs = k.cgs;
    f.total = (int)(k.a_bytes / 16);
    f.div_bm = make_fastdiv(k.bm); f.div_taps = make_fastdiv(f.taps); f.div_cgs = make_fastdiv(k.cgs); f.div_st = make_fastdiv(p.St);
    f.div_phases = make_fastdiv(p.sh * p.sw); f.div_sw = make_fastdiv(p.sw);
    (void)hipGetLastError();
    hipLaunchKernelGGL(pack_filter_f32_kernel, dim3((unsigned)((f.total + 255) / 256)), dim3(256), 0, st, f);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;

    PatchF32Params q{};
    q.a = (const float*)ws; q.a_bytes = (unsigned)k.a_bytes; q.mode = mode;
    p.wt = w; p.C = C;
    q.taps = f.taps; q.cgs = k.cgs;
    q.bands = k.bands; q.Wb = k.Wb; q.PW = k.PW; q.Mv = p.N * k.bands * p.Ho * k.Wb;
    q.h_base = mode == 0 ? p.g_add_h : p.g_add_h - (p.Rt - 1);
    q.w_base = mode == 0 ? p.g_add_w : p.g_add_w - (p.St - 1);
    q.img_rows = p.Ho + p.Rt - 1;
    q.full = k.full; q.parts = k.parts; q.cg_part = k.cg_part;
    q.partial = (float*)((char*)ws + k.part_offset);
    q.div_ho = make_fastdiv(p.Ho); q.div_wb = make_fastdiv(k.Wb); q.div_bands = make_fastdiv(k.bands); q.div_pw = make_fastdiv(k.PW);
    q.div_img = make_fastdiv(q.img_rows); q.div_st = make_fastdiv(p.St);
    p.tiles_i = k.tiles_i; p.tiles_pix = k.tiles_pix;
    const bool fused = p.bias || p.relu || p.mask;
    if (!k.split) {
        if (mode != 0) return hipErrorInvalidValue;
        return fused ? by_tile<false, false, false, true>(p, q, k.bm, st) : by_tile<false, false, false, false>(p, q, k.bm, st);
    }
    if (mode == 0) return fused ? by_tile<true, false, false, true>(p, q, k.bm, st) : by_tile<true, false, false, false>(p, q, k.bm, st);
    if (mode == 1) return fused ? by_tile<true, true, false, true>(p, q, k.bm, st) : by_tile<true, true, false, false>(p, q, k.bm, st);
    return fused ? by_tile<true, true, true, true>(p, q, k.bm, st) : by_tile<true, true, true, false>(p, q, k.bm, st);
}

}  // namespace pix
}  // namespace purine

// fp32 1x1 convolution without padding (forward with any stride, backward-data with stride 1) on the bf16 matrix
// cores: the arithmetic of packets.h (three exact bf16 parts, six products, two accumulator sets).
//
//     out[n][i][pix] = sum_j A[i][j] * in[n][j][pix]        A = W (forward) or W^T (backward-data)
//
// Bound: no roof alone (256 -> 256 channels at 27x27, N = 64 from HBM: 108 MB at 2.0 TB/s, matrix pipes 34 % busy): a wavefront's
// chain of loads, splitting and MFMAs, eight to sixteen of them on a CU. The filter of a row
// tile, all of its channels, is split once per workgroup into LDS; from then on no wavefront waits for another. The
// activations never pass through LDS: the MFMA's B operand is eight channels of one column per lane, which a lane
// loads straight from NCHW (32 adjacent pixels of two groups of eight channels per instruction), AHEAD steps of 16
// channels before their use, across the ends of its pixel strips, and splits in registers: each element once per row tile. The workgroups
// are persistent: one or two per CU walk strips of 32 pixels a wavefront, so that a filter is split 256 times
// and not once per tile, and one wavefront's stores fall into another's MFMAs. Row tiles of the same pixels run on the
// same XCD.
//
// (gemm1x1_kernel's fp32 MFMAs take 8/3 of the matrix time, and its workgroups load, compute and store in step.) Measured
// alone, before -> after, us forward and backward-data through the mask: 256 -> 256 channels at 27x27, N = 64: 77 -> 55 and
// 101 -> 64 (96 MB each: 1.7 TB/s, 113 TFLOP/s); 357 -> 467 at 21x21, N = 62: 111 -> 82 and 133 -> 132; 128 -> 128 at 28x28, N = 8: 14 -> 10 and 16 -> 11;
// at 14x14, N = 2: 13.4 -> 8.3 and 15.6 -> 8.5. Error against 64 bits a third to a half of the fp32 MFMAs'.
#include "packets.h"
#include "pix_common.h"

namespace purine {
namespace pix {
namespace {

using namespace packets;

constexpr int WAVES = 8, AHEAD = 2;   // (three or four steps ahead: the same, or a few per cent slower)

// bytes of eight channels' part of a row tile: a packet more than its rows, so that a wavefront filling it along the
// channels spreads over the banks
constexpr int filter_half(int tm) { return tm * 32 * 16 + 16; }
constexpr int filter_step(int tm) { return PLANES * 2 * filter_half(tm); }

struct Split1x1Params {
    int cgs;                    // groups of 16 gathered channels
    int strips, groups, waves;  // strips of 32 pixels; workgroups per row tile; wavefronts of each that take strips
    FastDiv div_kk;             // by 2 * cgs
};

template <bool TRANS, bool FUSED, int TM>
__global__ __launch_bounds__(WAVES * 64, TM == 1 ? 4 : 2) void gemm1x1_split_kernel(const PixParams p, const Split1x1Params q) {
    constexpr int BM = TM * 32, HALF = filter_half(TM), PLANE = 2 * HALF, STEP = PLANES * PLANE;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    float* bias_s = reinterpret_cast<float*>(smem + q.cgs * STEP);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int khalf = lane >> 5;
    // workgroups are dealt round-robin to the 8 XCDs: the row tiles of a group are 8 apart (neighbouring groups on one XCD,
    // for the cache lines that their strips share, measured the same to 10 % slower)
    const int xcd = blockIdx.x & 7, loc = blockIdx.x >> 3;
    const int grp = loc / p.tiles_i * 8 + xcd, rt = loc - loc / p.tiles_i * p.tiles_i;
    const int i0 = rt * BM;
    if (grp * q.waves >= q.strips) return;

    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.in), (short)0, (int)p.in_bytes, 0x00020000);
    const int stride = q.groups * q.waves;
    const int first = wave < q.waves ? grp * q.waves + wave : q.strips;     // the others only help with the filter
    auto origin = [&](int px) {                                            // gathered element of channel 0
        const int n = fastdiv(px, p.div_howo), rem = px - n * p.HoWo;
        const int ho = fastdiv(rem, p.div_wo), wo = rem - ho * p.Wo;
        return n * p.in_ns + ho * p.g_mul_h * p.Wi + wo * p.g_mul_w;
    };
    auto offset = [&](int strip) {
        const int px = strip * 32 + (lane & 31);
        return strip < q.strips && px < p.M ? (unsigned)(origin(px) + khalf * 8 * p.HiWi) * 4u : 0x80000000u;
    };

    float ring[AHEAD][8];
    int at_strip = first, at_step = 0;         // of the next request
    unsigned voff = offset(first);
    auto request = [&](float (&dst)[8]) {
        const int lim = p.Ci - at_step * 16 - khalf * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const unsigned at = e < lim ? voff : 0x80000000u;
            const int soff = (at_step * 16 + e) * p.HiWi * 4;
            dst[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rb, at, soff, 0));
        }
        if (++at_step == q.cgs) { at_step = 0; at_strip += stride; voff = offset(at_strip); }
    };
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) request(ring[k]);

    // the row tile's filter: a task is eight channels of a row, consecutive threads walk W's contiguous direction, a batch
    // of tasks costs one memory latency; rows and channels past the last are zero
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.wt), (short)0, p.Co * p.Ci * 4, 0x00020000);
    constexpr int BATCH = TRANS ? 1 : 2;
    const int tasks = q.cgs * 2 * BM;
    for (int t0 = tid; t0 < tasks; t0 += BATCH * WAVES * 64) {
        float v[BATCH][8];
        int dst[BATCH];
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
            const int t = t0 + j * WAVES * 64;
            const int kk = TRANS ? t / BM : t - (int)fastdiv(t, q.div_kk) * 2 * q.cgs, row = TRANS ? t % BM : fastdiv(t, q.div_kk);
            const int i = i0 + row, c0 = kk * 8;
            const bool ok = t < tasks && i < p.Co;
            dst[j] = t < tasks ? (kk >> 1) * STEP + (kk & 1) * HALF + row * 16 : -1;
            const bool whole = !TRANS && ok && c0 + 8 <= p.Ci;
            if (!TRANS) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const floatx4 f = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rw, whole ? (unsigned)(i * p.Ci + c0) * 4u : 0x80000000u, h * 16, 0));
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[j][h * 4 + e] = f[e];
                }
            }
            if (TRANS || (p.Ci & 7)) {          // single elements: of W^T, of a row's last channels
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const unsigned at = TRANS ? (unsigned)((c0 + e) * p.Co + i) * 4u : (unsigned)(i * p.Ci + c0 + e) * 4u;
                    const float f = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rw, ok && !whole && c0 + e < p.Ci ? at : 0x80000000u, 0, 0));
                    v[j][e] = whole ? v[j][e] : f;
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < BATCH; ++j)
            if (dst[j] >= 0) store_split8(v[j], smem + dst[j], PLANE);
    }
    if (FUSED && !TRANS) stage_bias<float, BM, WAVES * 64>(bias_s, p, i0, tid);
    __syncthreads();
    if (first >= q.strips) return;

    floatx16 hi[TM][1], lo[TM][1];
    auto clear = [&]() {
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int e = 0; e < 16; ++e) { hi[a][0][e] = 0.0f; lo[a][0][e] = 0.0f; }
    };
    clear();
    const unsigned char* a_ptr = smem + khalf * HALF + (lane & 31) * 16;
    int strip = first, step = 0;               // being multiplied
    const __amdgpu_buffer_rsrc_t r_out = __builtin_amdgcn_make_buffer_rsrc(p.out, (short)0, (int)p.out_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t r_mask = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.mask), (short)0, (int)p.out_bytes, 0x00020000);

    // a strip's sums are complete: infinities and NaNs again, as plain fp32 sums; epilogue
    auto finish = [&]() {
        const int pix = strip * 32 + (lane & 31);
        const bool live = pix < p.M;
        const int n = fastdiv(live ? pix : 0, p.div_howo);
        const unsigned vout = live ? (unsigned)(n * p.out_ns + (pix - n * p.HoWo) + khalf * 4 * p.HoWo) * 4u : 0x80000000u;
        const bool has_mask = FUSED && TRANS, has_beta = TRANS && p.beta != 0.0f;
        // accumulator register e of row tile a holds row a * 32 + (e / 4) * 8 + khalf * 4 + e % 4; a row past the last
        // lies outside the resource
        auto row_of = [&](int a, int e) { return i0 + a * 32 + (e >> 2) * 8 + (e & 3); };
        float mk[FUSED && TRANS ? 16 : 1];
        auto get_mask = [&](int a) {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int row = row_of(a, e);
                mk[FUSED && TRANS ? e : 0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r_mask, row + khalf * 4 < p.Co ? vout : 0x80000000u, row * p.HoWo * 4, 0));
            }
        };
        if (has_mask) get_mask(0);
        unsigned long long bad = join_sets<TM, 1>(hi, lo);
        if (__builtin_expect(__any(bad != 0), 0)) {
            while (bad) {
                const int idx = __ffsll((long long)bad) - 1;
                bad &= bad - 1;
                const int e = idx & 15, i = i0 + (idx >> 4) * 32 + (e >> 2) * 8 + khalf * 4 + (e & 3);
                float sum = 0.0f;
                if (live && i < p.Co) {
                    const float* b = (const float*)p.in + origin(pix);
                    const float* w = (const float*)p.wt + (TRANS ? (size_t)i : (size_t)i * p.Ci);
                    for (int c = 0; c < p.Ci && sum == sum; ++c)
                        sum = __builtin_fmaf(w[TRANS ? (size_t)c * p.Co : (size_t)c], b[(size_t)c * p.HiWi], sum);
                }
                replace_element<TM, 1>(hi, idx, sum);
            }
        }
#pragma unroll
        for (int a = 0; a < TM; ++a) {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int row = row_of(a, e);
                if (row >= p.Co) continue;                                   // uniform
                const unsigned at = row + khalf * 4 < p.Co ? vout : 0x80000000u;
                float v = hi[a][0][e];
                if (FUSED && !TRANS && p.bias) v += bias_s[row + khalf * 4 - i0];
                if (FUSED && !TRANS && p.relu) v = v > 0.0f ? v : 0.0f;
                if (has_mask) v = mk[FUSED && TRANS ? e : 0] > 0.0f ? v : 0.0f;
                if (has_beta) v += __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r_out, at, row * p.HoWo * 4, 0));
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r_out, at, row * p.HoWo * 4, 0);
            }
            if (has_mask && a + 1 < TM) get_mask(a + 1);
        }
    };
    // one step of 16 channels; true: that was the wavefront's last
    auto advance = [&](float (&src)[8]) {
        bf16x8 bv[PLANES];
        {
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            u32x4 pk[PLANES];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint32_t part[PLANES];
                split_pair(src[2 * e], src[2 * e + 1], part);
#pragma unroll
                for (int pl = 0; pl < PLANES; ++pl) pk[pl][e] = part[pl];
            }
#pragma unroll
            for (int pl = 0; pl < PLANES; ++pl) bv[pl] = __builtin_bit_cast(bf16x8, pk[pl]);
        }
        request(src);
        __builtin_amdgcn_sched_barrier(0);
        const unsigned char* sa = a_ptr + step * STEP;
        bf16x8 av[PLANES][TM];
#pragma unroll
        for (int pl = 0; pl < PLANES; ++pl)
#pragma unroll
            for (int a = 0; a < TM; ++a) av[pl][a] = *reinterpret_cast<const bf16x8*>(sa + pl * PLANE + a * 32 * 16);
        auto mul = [&](int i, int j, floatx16 (&acc)[TM][1]) {
#pragma unroll
            for (int a = 0; a < TM; ++a) acc[a][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[i][a], bv[j], acc[a][0], 0, 0, 0);
        };
        mul(0, 0, hi);
        mul(0, 1, lo);
        mul(0, 2, lo);
        mul(1, 0, lo);
        mul(1, 1, lo);
        mul(2, 0, lo);
        if (++step < q.cgs) return false;
        finish();
        clear();
        step = 0;
        strip += stride;
        return strip >= q.strips;
    };
    for (;;) {
        if (advance(ring[0])) return;
        if (advance(ring[1])) return;
    }
}

template <bool TRANS, bool FUSED, int TM>
hipError_t launch_one(const PixParams& p, const Split1x1Params& q, hipStream_t st) {
    const int lds = q.cgs * filter_step(TM) + TM * 32 * 4;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm1x1_split_kernel<TRANS, FUSED, TM>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    ProbeScope probe(st);
    (void)hipGetLastError();   // drop stale status left by earlier, unrelated runtime calls
    hipLaunchKernelGGL((gemm1x1_split_kernel<TRANS, FUSED, TM>), dim3((unsigned)(p.tiles_i * q.groups)), dim3(WAVES * 64), lds, st, p, q);
    return hipGetLastError();
}

template <bool TRANS, bool FUSED>
hipError_t by_tile(const PixParams& p, const Split1x1Params& q, int tm, hipStream_t st) {
    return tm == 1 ? launch_one<TRANS, FUSED, 1>(p, q, st) : launch_one<TRANS, FUSED, 2>(p, q, st);
}

}  // namespace

// Whether and how the layer runs here. Pure host arithmetic. force: test hook, row tiles (1, 2), or 0.
Split1x1Plan plan_gemm1x1_split(const PixParams& p, bool fwd, bool forced, int force) {
    Split1x1Plan k{};
    if (p.Rt * p.St != 1 || p.in_bytes == 0 || p.out_bytes == 0 || p.g_add_h != 0 || p.g_add_w != 0 || p.M > 0x7fffff00 || (long long)p.Co * p.Ci > 0x1fffffffLL) return k;
    k.cgs = (p.Ci + 15) / 16;
    k.strips = (p.M + 31) / 32;
    const double in_mb = 4e-6 * p.N * (double)p.HiWi * p.Ci, out_mb = 4e-6 * p.M * (double)p.Co;
    // 32 rows: half the registers, twice the wavefronts. 64: half the passes over the activations, which counts where they
    // leave the caches (198 -> 100 channels at 38x39, N = 216: 168 us with 32 rows, 133 with 64; 256 -> 256 at 27x27,
    // N = 64: 63 and 55; 384 -> 384 at 13x13, N = 64: 43 and 44, backward 45 and 51).
    k.tm = force ? force : p.Co > 32 && in_mb + out_mb > 64.0 ? 2 : 1;
    const int lds = k.cgs * filter_step(k.tm) + k.tm * 32 * 4;
    if (lds > 160 * 1024) return k;                                          // the whole filter has to fit
    k.tiles_i = (p.Co + k.tm * 32 - 1) / (k.tm * 32);
    const int per_cu = k.tm == 1 && lds <= 80 * 1024 ? 2 : 1;
    k.groups = 256 * per_cu / k.tiles_i / 8 * 8;                             // per row tile, as many on each XCD
    if (k.groups < 8) k.groups = 8;
    k.waves = WAVES;
    if ((long long)k.strips < (long long)k.groups * WAVES) {
        k.waves = (k.strips + k.groups - 1) / k.groups;
        k.groups = ((k.strips + k.waves - 1) / k.waves + 7) / 8 * 8;
    }
    if ((long long)k.tiles_i * k.groups > 0x7fffffffLL) return k;
    // Small launches (96 -> 96 channels at 54x54, N = 8, three passes 60 -> 51 us), and long sums, which keep the matrix units of gemm1x1_kernel busy
    // for longer than the memory (256 -> 256 at 27x27, N = 64, forward + masked backward-data, tensors from HBM: 170 us there, 116 here).
    // Not large launches of short sums: 96 -> 96 at 54x54, N = 64, with the weight gradient 164 us there, 168 here; 192 -> 176
    // at 28x28, N = 128 gains alone (182 and 142 us), but beside other streams' kernels the persistent workgroups wait for the
    // CUs that those hold (inception module of 128 images 1017 and 1046 us, of 50, 57 MB, 534 and 547). And not outputs that dwarf the input: a row's 128 bytes per
    // strip, at any alignment, leave two partial lines each, where gemm1x1_kernel writes 512 in one go (16 -> 300
    // at 62x62, N = 256: 332 us there, 554 here).
    // Within that, not where the workgroups of a dozen or more row tiles leave a wavefront strips of over 60 steps in all, one
    // workgroup per CU (555 -> 575 at 27x27, N = 18 forward 94 us there, 130 here; 75 such passes: 0.93 of the speed together), not
    // forward passes of up to 32 channels (32 -> 97 at 46x46, N = 13: 8.2 and 9.7; 463 passes: 1.02), and not large strided gathers
    // (453 -> 362, stride 2 at 60x62, N = 5: 31 and 44). The 5600 other passes that were timed: 1.2 times as fast.
    const long long chain = (long long)(k.strips + k.groups * k.waves - 1) / (k.groups * k.waves) * k.cgs;
    const bool strided = p.g_mul_h > 1 || p.g_mul_w > 1;
    const bool slower = (k.groups <= 16 && chain > 60) || (fwd && k.cgs <= 2);
    k.use = forced || (!slower && (in_mb + out_mb < 32.0 || (!strided && p.Ci >= 224 && out_mb < 3.0 * in_mb)));
    return k;
}

hipError_t launch_gemm1x1_split(PixParams p, const Split1x1Plan& k, bool trans, const void* w, hipStream_t st) {
    p.wt = w;
    p.tiles_i = k.tiles_i;
    const Split1x1Params q{k.cgs, k.strips, k.groups, k.waves, make_fastdiv(2 * k.cgs)};
    const bool fused = p.bias || p.relu || p.mask;
    if (!trans) return fused ? by_tile<false, true>(p, q, k.tm, st) : by_tile<false, false>(p, q, k.tm, st);
    return fused ? by_tile<true, true>(p, q, k.tm, st) : by_tile<true, false>(p, q, k.tm, st);
}

}  // namespace pix
}  // namespace purine

// fp32 forward / backward-data convolutions on the bf16 matrix cores, without losing precision.
//
// Bound: MFMA. The fp32 MFMA rate of the chip is 157 TFLOP/s, the bf16 rate sixteen times that, and
// an fp32 number is the exact sum of three bf16 numbers (8 + 8 + 8 significant bits). A product of two
// fp32 numbers is then nine bf16 products, of which the three smallest are below 2^-24 of it: six MFMAs
// of 32x32x16 take the place of eight of 32x32x2 and finish in 3/8 of their time. The largest of the
// six products accumulates in one register set, the five corrections in a second one, and the two
// are added once at the end: a correction never loses its low bits against a large running sum, and
// the main sum is rounded once per 16-deep MFMA group instead of once per two products. Measured
// against fp64 (one 32x32 tile, reduction length 64 .. 16384, uniform / normal / wide-range inputs)
// the error is 0.35 - 0.55 of the fp32 MFMA's; with one register set for all six products it is
// 0.65 - 1.25 of it, which is why there are two.
//
// Operands are laid out before the main kernel runs, in 16-byte packets of 8 consecutive reduction
// elements (8 channels of one position) per plane (the three bf16 parts):
//     activations [plane][n][channel group of 8][position][8]
//     filter      [row tile][step][plane][half][row of the tile][8],  step = (group of 16 channels, tap)
// so that a step's operand tiles are copied to LDS by loads that write LDS directly (16 bytes per lane,
// no registers, no VALU work but one offset per step and lane; a tap that falls into the padding is
// an offset outside the buffer, which loads zeros) and every MFMA fragment is one conflict-free 16-byte
// LDS read. The extra pass over the activations (4 bytes read, 6 written per element) is paid
// back where the gathered elements are used by several taps and row tiles.
#include "packets.h"
#include "pix_common.h"

namespace purine {
namespace pix {
namespace {

using namespace packets;

// One launch lays out both operands: workgroups below `x_blocks` take the activations (a thread per
// packet, lanes along positions: 8 coalesced 4-byte loads, three coalesced 16-byte stores), the others
// the filter (a thread per packet, lanes along rows; modes as in the filter repack of the tap kernels).
// Bound: HBM, 10 bytes per activation element.
struct PackParams {
    const float* x; unsigned char* xp;
    int Ci, HW, Cb, in_ns, x_blocks, x_total;       // x_total = N * Cb * HW packets
    FastDiv div_hw, div_cb;
    size_t plane_bytes;
    const float* w; unsigned char* wp;
    int mode, K, C, R, S, sh, sw, St, Co, bm, steps, taps, w_total;   // w_total = row tiles * steps * 2 * bm packets
    FastDiv div_bm, div_steps, div_taps, div_st, div_phases, div_sw;
};

__global__ __launch_bounds__(256) void pack_operands_kernel(const PackParams q) {
    float v[8];
    if ((int)blockIdx.x < q.x_blocks) {
        const int t = blockIdx.x * 256 + threadIdx.x;
        if (t >= q.x_total) return;
        const int ncb = fastdiv(t, q.div_hw), pos = t - ncb * q.HW;
        const int n = fastdiv(ncb, q.div_cb), cb = ncb - n * q.Cb;
        const float* src = q.x + (size_t)n * q.in_ns + (size_t)cb * 8 * q.HW + pos;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = cb * 8 + e < q.Ci ? src[(size_t)e * q.HW] : 0.0f;
        store_split8(v, q.xp + (size_t)t * 16, q.plane_bytes);
        return;
    }
    const int t = (blockIdx.x - q.x_blocks) * 256 + threadIdx.x;
    if (t >= q.w_total) return;
    const int rest = fastdiv(t, q.div_bm), row = t - rest * q.bm;       // rest = (row tile, step, half)
    const int half = rest & 1, ts = rest >> 1;
    const int rt = fastdiv(ts, q.div_steps), step = ts - rt * q.steps;
    const int cg = fastdiv(step, q.div_taps), tap = step - cg * q.taps;
    const int tr = fastdiv(tap, q.div_st), tc = tap - tr * q.St;
    const int i = rt * q.bm + row, ci0 = cg * 16 + half * 8;
    FilterRun f{0, 0, 0};
    if (i < q.Co) f = filter_run(q.mode, i, tr, tc, q.C, q.R, q.S, q.sh, q.sw, q.mode == 0 ? q.C : q.K, q.div_phases, q.div_sw);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = ci0 + e < f.lim ? q.w[(size_t)f.fixed + (size_t)(ci0 + e) * f.stride] : 0.0f;
    // [row tile][step][plane][half][row]
    store_split8(v, q.wp + ((size_t)ts * PLANES * 2 + half) * q.bm * 16 + (size_t)row * 16, (size_t)2 * q.bm * 16);
}

struct PacketParams {
    const void* a; const void* b;       // packed filter, packed activations
    unsigned a_bytes, b_bytes;
    int plane_bytes;                    // of the activations
    int Cb, taps, steps, splits, steps_per_split;
    int mode;                           // of the filter (filter_run), for outputs that are computed again
    FastDiv div_taps, div_st;
    size_t split_stride;                // elements between the splits' partial outputs
};

// D2S / FUSED / FWD: as in the other implicit-GEMM kernels (epilogue); MINUS: taps walk backwards.
template <bool MINUS, bool D2S, bool FUSED, int TM, int TN, int WM, int WN>
__global__ __launch_bounds__(WM * WN * 64, 2) void igemm_packets_kernel(const PixParams p, const PacketParams q) {
    typedef Tile<TM, TN, WM, WN> T;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char* spare = smem + T::NS * T::STAGE;
    float* bias_s = reinterpret_cast<float*>(spare + 1024);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int khalf = lane >> 5;
    const int wm = wave / WN, wn = wave % WN;

    // row tiles innermost: the row tiles of one pixel tile read the same activations and share an XCD's L2
    const int id = xcd_tile(blockIdx.x, gridDim.x);
    const int per_split = p.tiles_i * p.tiles_pix;
    const int split = id / per_split, tile = id - split * per_split;
    const int pt = tile / p.tiles_i, rt = tile - pt * p.tiles_i;
    const int i0 = rt * T::BM, j0 = pt * T::BN;
    const int s0 = split * q.steps_per_split;
    const int s1 = min(s0 + q.steps_per_split, q.steps);

    if (FUSED && !MINUS) stage_bias<float, T::BM, WM * WN * 64>(bias_s, p, i0, tid);

    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(q.a), (short)0, (int)q.a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(q.b), (short)0, (int)q.b_bytes, 0x00020000);

    // this lane's gathered pixel: its offset at tap (0, 0) (possibly outside the image) and coordinates
    const int pgrp = wave % T::PG, combo0 = wave / T::PG;
    int h0, w0, pix_off;
    {
        const int pix = j0 + pgrp * 64 + lane;
        const bool live = pix < p.M;
        const int n = fastdiv(live ? pix : 0, p.div_howo), rem = (live ? pix : 0) - n * p.HoWo;
        const int ho = fastdiv(rem, p.div_wo), wo = rem - ho * p.Wo;
        h0 = live ? ho * p.g_mul_h + p.g_add_h : -0x40000000;
        w0 = wo * p.g_mul_w + p.g_add_w;
        pix_off = (n * q.Cb * p.HiWi + (live ? h0 * p.Wi : 0) + w0) * 16;
    }

    // request step s (filter tile, gathered tile) into ring slot `slot`; past the end of the split's
    // range the loads fetch nothing, but are issued all the same, so that waits can count them
    int cg = 0, tr = 0, tc = 0;           // channel group and tap of the next step to be requested
    {
        cg = fastdiv(s0, q.div_taps);
        const int tap = s0 - cg * q.taps;
        tr = fastdiv(tap, q.div_st); tc = tap - tr * p.St;
    }
    auto request = [&](int s, int slot) {
        const bool exists = s < s1;
        unsigned char* sa = smem + slot * T::STAGE;
        unsigned char* sb = sa + T::A_BYTES;
        const int a_base = (rt * q.steps + s) * T::A_BYTES;
#pragma unroll
        for (int j = 0; j < T::RA; ++j) {
            const int t = j * T::NW + wave;
            const bool live = exists && (T::LA % T::NW == 0 || t < T::LA);
            const unsigned v = live ? (unsigned)(lane * 16) : 0x80000000u;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (__attribute__((address_space(3))) void*)(T::LA % T::NW == 0 || t < T::LA ? sa + t * 1024 : spare),
                                                     16, v, live ? a_base + t * 1024 : 0, 0, 0);
        }
        const int h = MINUS ? h0 - tr : h0 + tr, w = MINUS ? w0 - tc : w0 + tc;
        const int tap_off = (MINUS ? -(tr * p.Wi + tc) : tr * p.Wi + tc) * 16;
        const bool ok = exists && (unsigned)h < (unsigned)p.Hi && (unsigned)w < (unsigned)p.Wi;
        unsigned v = ok ? (unsigned)(pix_off + tap_off) : 0x80000000u;
        asm volatile("" : "+v"(v));       // one select, not a load on either side of a branch
#pragma unroll
        for (int j = 0; j < T::RB; ++j) {
            const int combo = j * T::WPG + combo0;                 // (plane, channel half)
            const bool live = (2 * PLANES) % T::WPG == 0 || combo < 2 * PLANES;
            const int soff = exists && live ? (combo >> 1) * q.plane_bytes + (cg * 2 + (combo & 1)) * p.HiWi * 16 : 0;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (__attribute__((address_space(3))) void*)(live ? sb + combo * T::BN * 16 + pgrp * 1024 : spare),
                                                     16, live ? v : 0x80000000u, soff, 0, 0);
        }
        tc += 1;
        if (tc == p.St) { tc = 0; tr += 1; }
        if (tr == p.Rt) { tr = 0; cg += 1; }
    };

    floatx16 hi[TM][TN], lo[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) { hi[a][b][e] = 0.0f; lo[a][b][e] = 0.0f; }

    __syncthreads();                      // bias in place; nothing is in flight yet
#pragma unroll
    for (int k = 0; k < T::NS - 1; ++k) request(s0 + k, k);

    const int a_off = (khalf * T::BM + wm * TM * 32 + (lane & 31)) * 16;
    const int b_off = T::A_BYTES + (khalf * T::BN + wn * TN * 32 + (lane & 31)) * 16;
    int slot = 0;
    for (int s = s0; s < s1; ++s) {
        // step s is in LDS, and every wavefront is done with the step before it, whose slot the next
        // request overwrites
        packets_landed<T::LOADS * (T::NS - 2)>();
        request(s + T::NS - 1, slot == 0 ? T::NS - 1 : slot - 1);
        multiply_step<T, TM, TN>(smem + slot * T::STAGE, a_off, b_off, hi, lo);
        slot = slot + 1 == T::NS ? 0 : slot + 1;
    }
    // the last requests must not outlive the workgroup's LDS
    __builtin_amdgcn_s_waitcnt(0x0070);

    // The sum of the two sets; what comes out infinite or NaN (such operands, or ones too large for the split) is
    // computed again from the fp32 operands as the fp32 kernel would.
    unsigned long long bad = join_sets<TM, TN>(hi, lo);
    if (__builtin_expect(__any(bad != 0), 0)) {
        while (bad) {
            const int idx = __ffsll((long long)bad) - 1;
            bad &= bad - 1;
            const int ab = idx >> 4, e = idx & 15;
            const int row = i0 + wm * TM * 32 + (ab / TN) * 32 + (e >> 2) * 8 + khalf * 4 + (e & 3);
            const int pix = j0 + wn * TN * 32 + (ab % TN) * 32 + (lane & 31);
            float sum = 0.0f;
            if (pix < p.M && row < p.Co) {
                const int n = fastdiv(pix, p.div_howo), rem = pix - n * p.HoWo;
                const int ho = fastdiv(rem, p.div_wo), wo = rem - ho * p.Wo;
                const int hb = ho * p.g_mul_h + p.g_add_h, wb = wo * p.g_mul_w + p.g_add_w;
                for (int s = s0; s < s1 && sum == sum; ++s) {
                    const int g = fastdiv(s, q.div_taps), tap = s - g * q.taps;
                    const int r = fastdiv(tap, q.div_st), t = tap - r * p.St;
                    const int h = MINUS ? hb - r : hb + r, w = MINUS ? wb - t : wb + t;
                    // a tap outside the image, or past the filter in a folded phase, is a zero that takes part: an
                    // infinite factor times it is NaN
                    const bool inside = (unsigned)h < (unsigned)p.Hi && (unsigned)w < (unsigned)p.Wi;
                    const FilterRun f = filter_run(q.mode, row, r, t, p.C, p.R, p.S, p.sh, p.sw, p.Ci, p.div_phases, p.div_sw);
                    const float* pb = (const float*)p.in + (size_t)n * p.in_ns + (inside ? h * p.Wi + w : 0);
                    for (int ci = g * 16; ci < g * 16 + 16 && ci < p.Ci; ++ci)
                        sum = __builtin_fmaf(ci < f.lim ? ((const float*)p.wt)[(size_t)f.fixed + (size_t)ci * f.stride] : 0.0f,
                                             inside ? pb[(size_t)ci * p.HiWi] : 0.0f, sum);
                }
            }
            replace_element<TM, TN>(hi, idx, sum);
        }
    }
    store_tile<float, D2S, FUSED, TM, TN, !MINUS>(p, (float*)p.out + (size_t)split * q.split_stride, hi, i0 + wm * TM * 32,
                                                  j0 + wn * TN * 32 + (lane & 31), khalf, bias_s, i0);
}

// Second pass of a split reduction: partial[split][n][row][position] added in split order, then the
// epilogue of the pass. One thread per element, lanes along positions.
template <bool D2S, bool FWD>
__global__ __launch_bounds__(256) void packets_reduce_kernel(const PixParams p, const float* __restrict__ partial, int splits, size_t stride) {
    const long long total = (long long)p.N * p.Co * p.HoWo;
    for (long long t = (long long)blockIdx.x * 256 + threadIdx.x; t < total; t += (long long)gridDim.x * 256) {
        float v = 0.0f;
        for (int s = 0; s < splits; ++s) v += partial[(size_t)s * stride + t];
        const int ni = fastdiv((int)t, p.div_howo), rem = (int)t - ni * p.HoWo;
        const int n = ni / p.Co, i = ni - n * p.Co;
        const TileAddr<float, D2S> addr(p, n, rem);
        bool ok;
        const int off = addr.at(i, ok);
        if (!ok) continue;
        float* out = (float*)p.out;
        if (FWD && p.bias) v += ((const float*)p.bias)[i];
        if (FWD && p.relu) v = v > 0.0f ? v : 0.0f;
        if (!FWD && p.mask) v = ((const float*)p.mask)[off] > 0.0f ? v : 0.0f;
        if (!FWD && p.beta != 0.0f) v += out[off];
        out[off] = v;
    }
}

template <bool MINUS, bool D2S, bool FUSED, int TM, int TN, int WM, int WN>
hipError_t launch_main(const PixParams& p, const PacketParams& q, hipStream_t st) {
    typedef Tile<TM, TN, WM, WN> T;
    const long long total = (long long)p.tiles_i * p.tiles_pix * q.splits;
    if (total <= 0 || total > 0x7fffffffLL) return hipErrorInvalidValue;
    if (T::LDS > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&igemm_packets_kernel<MINUS, D2S, FUSED, TM, TN, WM, WN>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS);
        if (e != hipSuccess) return e;
    }
    (void)hipGetLastError();   // drop stale status left by earlier, unrelated runtime calls
    hipLaunchKernelGGL((igemm_packets_kernel<MINUS, D2S, FUSED, TM, TN, WM, WN>), dim3((unsigned)total), dim3(WM * WN * 64), T::LDS, st, p, q);
    return hipGetLastError();
}

template <bool MINUS, bool D2S, bool FUSED>
hipError_t by_tile(const PixParams& p, const PacketParams& q, int bm, int bn, hipStream_t st) {
#define CALL(TM, TN, WM, WN) launch_main<MINUS, D2S, FUSED, TM, TN, WM, WN>(p, q, st)
    PACKET_TILES(CALL)
#undef CALL
}

}  // namespace

// How the layer would run on this kernel, and the time that is expected to take (k.us; the caller
// compares it with the fp32 MFMA kernels'). Pure host arithmetic on p's geometry.
//
// The model. A CU works on two workgroups at a time; x workgroups per CU cost (x + ceil(x)) / 2
// workgroup times (the busiest CU sets the pace, but the clock, which the power limit holds at 1.9 -
// 2.0 GHz on a full chip, rises as the others run dry: 338 tiles measured 0.82 of 507), a lone
// workgroup 1.45. Splitting the reduction writes and reads one partial output per split, mostly from
// the last-level cache, and costs a launch; the depth-to-space epilogue scatters single elements.
// Against sweeps of all tiles and split counts on twelve layers the choice is within 5 % of the best
// on most and 10 % on the worst.
PacketPlan plan_packets(const PixParams& p, bool d2s, bool any_taps) {
    PacketPlan k{};
    const long long steps = (long long)((p.Ci + 15) / 16) * p.Rt * p.St;
    const long long cb = (p.Ci + 15) / 16 * 2;
    const long long b_bytes = (long long)p.N * cb * p.HiWi * 16 * PLANES;
    if ((p.Rt * p.St < 2 && !any_taps) || p.Ci < 8 || b_bytes >= 0x7fffffffLL || p.in_bytes == 0) return k;
    // a copy of the gathered tensor in the scratch: only for strided gathers and for launches too small to
    // fill the chip without a split reduction
    const bool strided = p.g_mul_h > 1 || p.g_mul_w > 1;
    if (!strided && !any_taps && !split_packets_forced() && ((p.Co + 127) / 128) * (((long long)p.M + 255) / 256) >= 128) return k;
    const double ghz = 2.2e3;                             // cycles per microsecond
    const double out_bytes = (double)p.M * p.Co * 4.0;
    for (const PacketTile& t : kTiles) {
        const long long ti = (p.Co + t.bm - 1) / t.bm, tp = ((long long)p.M + t.bn - 1) / t.bn, tiles = ti * tp;
        const long long a_bytes = ti * steps * PLANES * 2 * t.bm * 16;
        if (a_bytes >= 0x7fffffffLL) continue;
        // laying out the operands: 10 bytes per packed element, and a launch
        const double pack_us = 5.0 + ((double)b_bytes + (double)a_bytes) / 6.0 * 10.0 / 4.5e6;
        // no split, or split counts that fill the chip to 1/2, 1, 3/2 .. 4 workgroups per CU
        long long last = -1;
        for (int half_fill = 0; half_fill <= 8; ++half_fill) {
            long long sp = half_fill * 128 / tiles;
            if (sp < 1) sp = 1;
            if (sp > 64) sp = 64;
            const long long per = (steps + sp - 1) / sp;
            sp = (steps + per - 1) / per;
            if (per == last) continue;
            last = per;
            if (sp > 1 && sp * out_bytes >= 128.0 * (1 << 20)) break;
            const double x = (double)(tiles * sp) / 256.0;
            const double load = x <= 1.0 ? 1.45 : 0.5 * (x + (double)((tiles * sp + 255) / 256));
            double us = load * ((double)per * t.cycles / t.eff + (d2s && sp == 1 ? 40000.0 : 4000.0)) / ghz + 4.0 + pack_us;
            if (sp > 1) us += 6.0 + 2.0 * sp * out_bytes / 8e6;
            if (!k.use || us < k.us) {
                k.use = true; k.us = us;
                k.bm = t.bm; k.bn = t.bn; k.tiles_i = (int)ti; k.tiles_pix = (int)tp;
                k.splits = (int)sp; k.steps_per_split = (int)per;
                k.a_bytes = (size_t)a_bytes;
            }
        }
    }
    if (!k.use) return k;
    k.steps = (int)steps; k.Cb = (int)cb;
    k.b_offset = (k.a_bytes + 255) / 256 * 256;
    k.b_bytes = (size_t)b_bytes;
    k.part_offset = (k.b_offset + k.b_bytes + 255) / 256 * 256;
    k.ws_bytes = k.splits > 1 ? k.part_offset + (size_t)k.splits * p.M * p.Co * 4 : k.part_offset;
    return k;
}

hipError_t launch_packets(PixParams p, const PacketPlan& k, int mode, const void* w, int K, int C, void* ws, hipStream_t st) {
    if (!ws) return hipErrorInvalidValue;
    ProbeScope whole_op(st);             // layout pass, products, second pass
    unsigned char* base = (unsigned char*)ws;
    PackParams a{};
    a.x = (const float*)p.in; a.xp = base + k.b_offset;
    a.Ci = p.Ci; a.HW = p.HiWi; a.Cb = k.Cb; a.in_ns = p.in_ns;
    a.x_total = p.N * k.Cb * p.HiWi; a.x_blocks = (a.x_total + 255) / 256;
    a.div_hw = make_fastdiv(p.HiWi); a.div_cb = make_fastdiv(k.Cb);
    a.plane_bytes = k.b_bytes / PLANES;
    a.w = (const float*)w; a.wp = base;
    a.mode = mode; a.K = K; a.C = C; a.R = p.R; a.S = p.S; a.sh = p.sh; a.sw = p.sw; a.St = p.St; a.Co = p.Co;
    a.bm = k.bm; a.steps = k.steps; a.taps = p.Rt * p.St;
    a.w_total = k.tiles_i * k.steps * 2 * k.bm;
    a.div_bm = make_fastdiv(k.bm); a.div_steps = make_fastdiv(k.steps); a.div_taps = make_fastdiv(a.taps); a.div_st = make_fastdiv(p.St);
    a.div_phases = make_fastdiv(p.sh * p.sw); a.div_sw = make_fastdiv(p.sw);
    (void)hipGetLastError();
    hipLaunchKernelGGL(pack_operands_kernel, dim3((unsigned)(a.x_blocks + (a.w_total + 255) / 256)), dim3(256), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;

    PacketParams q{};
    q.a = base; q.b = base + k.b_offset;
    q.a_bytes = (unsigned)k.a_bytes; q.b_bytes = (unsigned)k.b_bytes; q.plane_bytes = (int)(k.b_bytes / PLANES);
    q.Cb = k.Cb; q.taps = a.taps; q.steps = k.steps; q.splits = k.splits; q.steps_per_split = k.steps_per_split;
    q.mode = mode; q.div_taps = a.div_taps; q.div_st = a.div_st;
    p.wt = w; p.C = C;
    p.tiles_i = k.tiles_i; p.tiles_pix = k.tiles_pix;
    const bool fused = p.bias || p.relu || p.mask;
    if (k.splits > 1) {
        PixParams r = p;
        float* partial = (float*)(base + k.part_offset);
        q.split_stride = (size_t)p.M * p.Co;
        p.out = partial; p.out_ns = p.Co * p.HoWo; p.bias = nullptr; p.mask = nullptr; p.relu = 0; p.beta = 0.0f;
        p.out_bytes = (unsigned)(q.split_stride * 4);
        e = mode == 0 ? by_tile<false, false, false>(p, q, k.bm, k.bn, st) : by_tile<true, false, false>(p, q, k.bm, k.bn, st);
        if (e != hipSuccess) return e;
        const long long total = (long long)r.M * r.Co;
        const unsigned blocks = (unsigned)((total + 255) / 256 > 8192 ? 8192 : (total + 255) / 256);
        if (mode == 0) hipLaunchKernelGGL((packets_reduce_kernel<false, true>), dim3(blocks), dim3(256), 0, st, r, partial, k.splits, q.split_stride);
        else if (mode == 1) hipLaunchKernelGGL((packets_reduce_kernel<false, false>), dim3(blocks), dim3(256), 0, st, r, partial, k.splits, q.split_stride);
        else hipLaunchKernelGGL((packets_reduce_kernel<true, false>), dim3(blocks), dim3(256), 0, st, r, partial, k.splits, q.split_stride);
        return hipGetLastError();
    }
    if (mode == 0) return fused ? by_tile<false, false, true>(p, q, k.bm, k.bn, st) : by_tile<false, false, false>(p, q, k.bm, k.bn, st);
    if (mode == 1) return fused ? by_tile<true, false, true>(p, q, k.bm, k.bn, st) : by_tile<true, false, false>(p, q, k.bm, k.bn, st);
    return fused ? by_tile<true, true, true>(p, q, k.bm, k.bn, st) : by_tile<true, true, false>(p, q, k.bm, k.bn, st);
}

// out[rows][cols] = beta * out + sum over k of a[k][row] * b[k][col], dense (the fully-connected weight
// gradient: k runs over the batch): the single-tap backward-data pass over one image of K channels.
static PixParams matrix_params(long long rows, long long cols, long long K) {
    PixParams p{};
    p.N = 1; p.Ci = (int)K; p.Hi = 1; p.Wi = p.HiWi = (int)cols; p.Co = (int)rows; p.Ho = 1; p.Wo = p.HoWo = p.M = (int)cols;
    p.Rt = p.St = p.R = p.S = p.sh = p.sw = p.g_mul_h = p.g_mul_w = p.phases = 1;
    p.div_howo = p.div_wo = make_fastdiv((uint32_t)cols); p.div_phases = p.div_sw = make_fastdiv(1);
    p.in_ns = (int)(K * cols); p.out_ns = (int)(rows * cols);
    p.in_bytes = (unsigned)(K * cols * 4); p.out_bytes = (unsigned)(rows * cols * 4);      // both below 2^31 (the caller's check)
    return p;
}
PacketPlan plan_packets_matrix(long long rows, long long cols, long long K) { return plan_packets(matrix_params(rows, cols, K), false, true); }
hipError_t launch_packets_matrix(const PacketPlan& k, const void* a, const void* b, void* out, float beta, long long rows, long long cols, long long K,
                                 void* ws, hipStream_t st) {
    PixParams p = matrix_params(rows, cols, K);
    p.in = b; p.out = out; p.beta = beta;
    return launch_packets(p, k, 1, a, (int)K, (int)rows, ws, st);
}

}  // namespace pix
}  // namespace purine

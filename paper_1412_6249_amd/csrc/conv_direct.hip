// Convolutions of small launches in one kernel: forward and backward-data, fp32 and bf16, any stride.
//
//     out[i, pixel] = sum over t of A[i][t] * in[pixel, t],  t = (channel, filter row, filter column) as the filter lies in memory
//
// The general kernels lay the filter (and some the activations) out first and then walk the whole reduction in a few workgroups: two to three
// launches and a chain of slabs, 16 - 20 us for 38 -> 42 channels 3x3 of two 8x9 images. Here a workgroup owns 32 rows x 32 pixels, its
// wavefronts take the steps of the reduction (16 elements) in turn, loading their MFMA fragments straight from memory (the next
// step's while one is multiplied; bf16 as they are, fp32 as three bf16 parts with six products and two accumulator sets, see
// conv_packets.hip), and the wavefronts' sums are added through LDS in order. No scratch, no layout pass, no second launch. Where element t of
// every pixel lies, and which filter row and column it belongs to, is a table in LDS that the workgroup makes first; a pixel's taps
// that fall outside are two bit masks in registers. A strided backward pass multiplies the taps that do not reach a pixel as zeros.
//
// Bound: the chain of loads of a few steps (0.8 us each forward, 1.7 backward, whose filter elements lie R * S apart), and with many of
// them the VALU work of gathering and splitting. us, general kernels / here: fp32 38 -> 42 3x3 of two 8x9 images forward 19.2 / 6.9, backward-data
// 20.4 / 8.8; 64 -> 64 3x3 at 56x56, N = 1 17.8 / 8.4, 17.5 / 10.4; 64 -> 8 5x5 at 8x9, N = 4 61 / 13, 19.6 / 7.0; 384 -> 384 3x3 at 13x13,
// N = 2 28.5 / 31.5, 27.8 / 42.4 (stays).
#include <cmath>
#include <type_traits>
#include "packets.h"
#include "pix_common.h"

namespace purine {
namespace {

using namespace packets;

struct ConvDirectParams {
    const void* in; const void* w; void* out; const void* bias; const void* mask;
    unsigned in_bytes, w_bytes;
    int rows, M, T, steps, tiles_j;
    int C, RS, S, sh, sw, ph, pw;
    int Hi, Wi, HiWi, Wo, HoWo, in_ns, out_ns;
    int relu;
    float beta;
    FastDiv div_howo, div_wo, div_rs, div_s, div_sh, div_sw;
};
constexpr unsigned NOWHERE = 0x80000000u;

// One element of the reduction: offset of the gathered value from a pixel's, of the filter's from a row's (backward), shifts that bring
// the filter row's and column's bits of a pixel's masks to the sign.
struct __attribute__((aligned(16))) Element { int in, w, row, col; };

// FAR: images so far apart that the gathered tensor spans 2^31 bytes or more: plain loads instead of range-checked ones.
template <int PL, bool BWD, bool FAR, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void conv_direct_kernel(const ConvDirectParams q) {
    constexpr int ES = PL == 1 ? 2 : 4, NT = WAVES * 64;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    Element* table = reinterpret_cast<Element*>(smem);
    float (*sums)[16][64] = reinterpret_cast<float (*)[16][64]>(smem);       // (after the table has been used)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int khalf = lane >> 5, l31 = lane & 31;
    const int it = blockIdx.x / q.tiles_j, jt = blockIdx.x - it * q.tiles_j;
    const int row = it * 32 + l31, col = jt * 32 + l31;
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(q.w), (short)0, (int)q.w_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(q.in), (short)0, (int)q.in_bytes, 0x00020000);

    // the pixel: offset of its gathered window, bit r / s: filter row r / column s reaches an input that exists
    const int R = q.RS / q.S;
    typename std::conditional<FAR, long long, unsigned>::type b_base = 0;
    unsigned rows_ok = 0, cols_ok = 0;
    if (col < q.M) {
        const int n = fastdiv(col, q.div_howo), pix = col - n * q.HoWo, ho = fastdiv(pix, q.div_wo), wo = pix - ho * q.Wo;
        if (!BWD) {
            const int h0 = ho * q.sh - q.ph, w0 = wo * q.sw - q.pw;
            for (int r = 0; r < R; ++r) rows_ok |= (unsigned)((unsigned)(h0 + r) < (unsigned)q.Hi) << r;
            for (int s = 0; s < q.S; ++s) cols_ok |= (unsigned)((unsigned)(w0 + s) < (unsigned)q.Wi) << s;
            b_base = (decltype(b_base))n * q.in_ns + h0 * q.Wi + w0;
        } else {
            const int hq = fastdiv(ho + q.ph, q.div_sh), a = ho + q.ph - hq * q.sh, wq = fastdiv(wo + q.pw, q.div_sw), b = wo + q.pw - wq * q.sw;
            for (int r = a, p = hq; r < R; r += q.sh, --p) rows_ok |= (unsigned)((unsigned)p < (unsigned)q.Hi) << r;
            for (int s = b, p = wq; s < q.S; s += q.sw, --p) cols_ok |= (unsigned)((unsigned)p < (unsigned)q.Wi) << s;
            b_base = (decltype(b_base))n * q.in_ns + hq * q.Wi + wq;
        }
    }
    for (int t = tid; t < q.steps * 16; t += NT) {
        const int c = fastdiv(t, q.div_rs), rs = t - c * q.RS, r = fastdiv(rs, q.div_s), s = rs - r * q.S;
        Element e;
        e.in = BWD ? c * q.HiWi - fastdiv(r, q.div_sh) * q.Wi - fastdiv(s, q.div_sw) : c * q.HiWi + r * q.Wi + s;
        e.w = t < q.T ? (c * q.C * q.RS + rs) : 0x40000000;
        e.row = t < q.T ? 31 - r : 0;           // (bit 31 is never set)
        e.col = 31 - s;
        table[t] = e;
    }
    __syncthreads();

    floatx16 hi, lo;
#pragma unroll
    for (int e = 0; e < 16; ++e) { hi[e] = 0.0f; lo[e] = 0.0f; }
    struct Frag { unsigned a[PL == 1 && !BWD ? 5 : 8], b[8]; };
    auto load = [&](int s, Frag& f) {
        const bool live = s < q.steps;
        const int t = live ? s * 16 + khalf * 8 : 0;
        if constexpr (!BWD) {
            typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
            const unsigned o = live && row < q.rows ? (unsigned)(row * q.T + t) * ES & ~3u : NOWHERE;
            const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(ra, o, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) f.a[e] = x[e];
            if constexpr (PL == 1) {
                f.a[4] = __builtin_amdgcn_raw_buffer_load_b32(ra, o == NOWHERE ? o : o + 16, 0, 0);
            } else {
                const u32x4 y = __builtin_amdgcn_raw_buffer_load_b128(ra, o == NOWHERE ? o : o + 16, 0, 0);
#pragma unroll
                for (int e = 0; e < 4; ++e) f.a[4 + e] = y[e];
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const Element k = table[t + e];
            const bool ok = live && (int)((rows_ok << k.row) & (cols_ok << k.col)) < 0;
            if constexpr (FAR) {
                const long long o = ok ? b_base + k.in : 0;
                const unsigned v = PL == 1 ? (unsigned)((const uint16_t*)q.in)[o] : ((const unsigned*)q.in)[o];
                f.b[e] = ok ? v : 0u;
            } else {
                const unsigned o = ok ? (b_base + (unsigned)k.in) * ES : NOWHERE;
                f.b[e] = PL == 1 ? (unsigned)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rb, o, 0, 0) : (unsigned)__builtin_amdgcn_raw_buffer_load_b32(rb, o, 0, 0);
            }
            if constexpr (BWD) {
                const unsigned w = live && row < q.rows && k.w != 0x40000000 ? (unsigned)(k.w + row * q.RS) * ES : NOWHERE;
                f.a[e] = PL == 1 ? (unsigned)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(ra, w, 0, 0) : (unsigned)__builtin_amdgcn_raw_buffer_load_b32(ra, w, 0, 0);
            }
        }
    };
    auto multiply = [&](int s, Frag& f) {
        const int t = s * 16 + khalf * 8;
        if constexpr (PL == 1) {
            unsigned a[4], b[4];
            if constexpr (BWD) {
#pragma unroll
                for (int e = 0; e < 4; ++e) a[e] = f.a[2 * e] | f.a[2 * e + 1] << 16;
            } else {
                const unsigned sh = ((unsigned)row * (unsigned)q.T + (unsigned)t) & 1 ? 16u : 0u;
#pragma unroll
                for (int e = 0; e < 4; ++e) a[e] = __builtin_amdgcn_alignbit(f.a[e + 1], f.a[e], sh);
                if (t + 8 > q.T) {                 // (past the end of the reduction lies the next row)
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[e] &= (t + 2 * e < q.T ? 0xffffu : 0u) | (t + 2 * e + 1 < q.T ? 0xffff0000u : 0u);
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) b[e] = f.b[2 * e] | f.b[2 * e + 1] << 16;
            multiply_loaded<PL>(a, b, hi, lo);
        } else {
            if (!BWD && t + 8 > q.T) {
#pragma unroll
                for (int e = 0; e < 8; ++e) f.a[e] = t + e < q.T ? f.a[e] : 0u;
            }
            multiply_loaded<PL>(f.a, f.b, hi, lo);
        }
    };
    Frag f0, f1;
    load(wave, f0);
    for (int s = wave; s < q.steps; s += 2 * WAVES) {
        load(s + WAVES, f1);
        multiply(s, f0);
        load(s + 2 * WAVES, f0);
        multiply(s + WAVES, f1);             // (past the last step: zeros)
    }
    __syncthreads();
    put_sums<PL>(sums[wave], lane, hi, lo);
    __syncthreads();

    auto value = [](const void* t, size_t i) { return PL == 1 ? __uint_as_float((unsigned)((const uint16_t*)t)[i] << 16) : ((const float*)t)[i]; };
    for (int o = tid; o < 1024; o += NT) {
        const int e = o >> 6, l = o & 63;
        const int i = it * 32 + (e >> 2) * 8 + (l >> 5) * 4 + (e & 3), j = jt * 32 + (l & 31);
        float v = all_sums<WAVES>(sums, e, l);
        if (i >= q.rows || j >= q.M) continue;
        const int n = fastdiv(j, q.div_howo), pix = j - n * q.HoWo;
        if ((PL == 3 || BWD) && !(__builtin_fabsf(v) <= 3.402823466e38f)) {
            // infinities and NaNs: again, as a plain fp32 sum of the taps that reach the pixel (padding as zeros)
            const int ho = fastdiv(pix, q.div_wo), wo = pix - ho * q.Wo;
            v = 0.0f;
            for (int t = 0; t < q.T && v == v; ++t) {
                const int c = fastdiv(t, q.div_rs), rs = t - c * q.RS, r = fastdiv(rs, q.div_s), s = rs - r * q.S;
                int h, w;
                if (BWD) {
                    h = ho + q.ph - r; w = wo + q.pw - s;
                    if (h % q.sh || w % q.sw) continue;
                    h /= q.sh; w /= q.sw;
                } else {
                    h = ho * q.sh - q.ph + r; w = wo * q.sw - q.pw + s;
                }
                const bool in = (unsigned)h < (unsigned)q.Hi && (unsigned)w < (unsigned)q.Wi;
                v = __builtin_fmaf(value(q.w, BWD ? ((size_t)c * q.C + i) * q.RS + rs : (size_t)i * q.T + t),
                                   in ? value(q.in, (size_t)n * q.in_ns + (size_t)c * q.HiWi + (size_t)h * q.Wi + w) : 0.0f, v);
            }
        }
        const size_t at = (size_t)n * q.out_ns + (size_t)i * q.HoWo + pix;
        if (q.bias) v += value(q.bias, i);
        if (q.relu) v = v > 0.0f ? v : 0.0f;
        if (q.mask) v = value(q.mask, at) > 0.0f ? v : 0.0f;
        if (q.beta != 0.0f) v += value(q.out, at);
        if constexpr (PL == 1) ((__bf16*)q.out)[at] = (__bf16)v;
        else ((float*)q.out)[at] = v;
    }
}

template <int PL, bool BWD, bool FAR, int WAVES>
hipError_t launch(const ConvDirectParams& q, hipStream_t st) {
    const long long tiles = (long long)((q.rows + 31) / 32) * q.tiles_j;
    if (tiles <= 0 || tiles > 0x7fffffffLL) return hipErrorInvalidValue;
    const int table = q.steps * 16 * (int)sizeof(Element), sums = WAVES * 4096, lds = table > sums ? table : sums;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_direct_kernel<PL, BWD, FAR, WAVES>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
    }
    ProbeScope probe(st);
    (void)hipGetLastError();   // drop stale status left by earlier, unrelated runtime calls
    hipLaunchKernelGGL((conv_direct_kernel<PL, BWD, FAR, WAVES>), dim3((unsigned)tiles), dim3(WAVES * 64), lds, st, q);
    return hipGetLastError();
}
template <int PL, bool BWD>
hipError_t by_waves(const ConvDirectParams& q, hipStream_t st) {
    if (q.in_bytes == 0) {
        if (q.steps > 16) return launch<PL, BWD, true, 16>(q, st);
        if (q.steps > 4) return launch<PL, BWD, true, 8>(q, st);
        return launch<PL, BWD, true, 2>(q, st);
    }
    if (q.steps > 16) return launch<PL, BWD, false, 16>(q, st);
    if (q.steps > 4) return launch<PL, BWD, false, 8>(q, st);
    return launch<PL, BWD, false, 2>(q, st);
}

}  // namespace

// Expected time (fitted to 1143 passes of 4 - 100 us: 0.5 - 1.7 of the measured ones), or a negative number where the kernel does not apply.
double conv_direct_us(const ConvGeom& g, bool bwd, int dtype) {
    const long long es = dtype == PURINE_F32 ? 4 : 2, T = (long long)(bwd ? g.K : g.C) * g.R * g.S;
    const long long rows = bwd ? g.C : g.K, M = (long long)g.N * (bwd ? (long long)g.H * g.W : (long long)g.P * g.Q);
    // (by the extents alone: a slice of a larger tensor gets the bits of a dense one)
    const long long in = (long long)g.N * (bwd ? g.K : g.C) * (bwd ? (long long)g.P * g.Q : (long long)g.H * g.W) * es;
    if (T > 8192 || g.R > 31 || g.S > 31 || in >= (1ll << 31) - 64 || (long long)g.K * g.C * g.R * g.S * es >= (1ll << 30) || g.ph > 4096 || g.pw > 4096) return -1.0;
    const double steps = (double)((T + 15) / 16), tiles = (double)((rows + 31) / 32) * (double)((M + 31) / 32);
    const double waves = steps > 16 ? 16 : steps > 4 ? 8 : 2, chain = std::ceil(steps / waves);
    const double work = tiles * steps * 1e-3;
    if (bwd) return dtype == PURINE_F32 ? 2.8 + 1.72 * chain + 0.47 * work + 5.7e-3 * tiles : 2.7 + 1.62 * chain + 0.417 * work + 3.07e-3 * tiles;
    const double apart = g.sw > 1 ? 1.2 : 1.0;       // lanes on every other element ask for twice the lines
    return apart * (dtype == PURINE_F32 ? 3.9 + 0.76 * chain + 0.556 * work + 3.13e-3 * tiles : 2.9 + 0.99 * chain + 0.313 * work + 1.55e-3 * tiles);
}

hipError_t launch_conv_direct(int dtype, const ConvGeom& g, bool bwd, const void* in, const void* wt, void* out, float beta, const PixEpilogue& epi, hipStream_t st) {
    const int es = dtype == PURINE_F32 ? 4 : 2;
    ConvDirectParams q{};
    q.in = in; q.w = wt; q.out = out; q.bias = epi.bias; q.mask = epi.mask; q.relu = epi.relu; q.beta = beta;
    q.rows = bwd ? g.C : g.K; q.T = (bwd ? g.K : g.C) * g.R * g.S; q.steps = (q.T + 15) / 16;
    q.C = g.C; q.RS = g.R * g.S; q.S = g.S; q.sh = g.sh; q.sw = g.sw; q.ph = g.ph; q.pw = g.pw;
    q.Hi = bwd ? g.P : g.H; q.Wi = bwd ? g.Q : g.W; q.HiWi = q.Hi * q.Wi;
    q.Wo = bwd ? g.W : g.Q; q.HoWo = (bwd ? g.H : g.P) * q.Wo;
    q.in_ns = bwd ? g.y_ns : g.x_ns; q.out_ns = bwd ? g.x_ns : g.y_ns;
    q.M = g.N * q.HoWo; q.tiles_j = (q.M + 31) / 32;
    const long long span = ((long long)(g.N - 1) * q.in_ns + (long long)(bwd ? g.K : g.C) * q.HiWi) * es;
    q.in_bytes = span < (1ll << 31) - 64 ? (unsigned)span : 0u;
    q.w_bytes = (unsigned)(((long long)g.K * g.C * q.RS * es + 3) & ~3ll);
    q.div_howo = make_fastdiv(q.HoWo); q.div_wo = make_fastdiv(q.Wo); q.div_rs = make_fastdiv(q.RS); q.div_s = make_fastdiv(g.S);
    q.div_sh = make_fastdiv(g.sh); q.div_sw = make_fastdiv(g.sw);
    if (dtype == PURINE_F32) return bwd ? by_waves<3, true>(q, st) : by_waves<3, false>(q, st);
    return bwd ? by_waves<1, true>(q, st) : by_waves<1, false>(q, st);
}

}  // namespace purine

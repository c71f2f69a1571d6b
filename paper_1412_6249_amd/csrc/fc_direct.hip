// Fully-connected passes in one launch: small matrices, whose time is launches and chains of loads.
//
//     out[row][column] = sum over k of A[row][k] * B[k][column]       (plus a bias per column; or times nothing, added to out)
//
// A workgroup owns a 32 x 32 tile and its wavefronts take the steps of the reduction (16 elements) in turn: each loads its MFMA
// fragments straight from memory (two steps ahead of their use), multiplies them (bf16 as they are; fp32 as three bf16
// parts with six products and two accumulator sets, see conv_packets.hip), and the wavefronts' sums are added through LDS in
// order. No scratch, no layout pass, no second launch; the bias and its gradient ride along. An operand's reduction axis is its
// inner one (16-byte loads, for bf16 rows of odd length from the dword before) or its outer one (eight loads, lanes along rows / columns).
//
// Bound: the chain of a few loads, and one launch's 3 us. All three passes together, us, before / now: bf16 3 x 222 x 37 (images,
// inputs, outputs) 30 / 13, 4 x 957 x 93 33 / 15; fp32 3 x 222 x 37 25 / 14, 226 x 853 x 271 42 / 23.
#include <cmath>
#include "packets.h"
#include "pix_common.h"

namespace purine {
namespace {

using namespace packets;

struct FcDirectParams {
    const void* a; const void* b; void* out;
    const void* bias;                // per column, of the operands' type; or null
    float* db;                       // per row: the sums of A over k; or null
    unsigned a_bytes, b_bytes;
    int rows, cols, K, a_ld, b_ld, tiles_j, steps;
    float beta;
};

constexpr unsigned NOWHERE = 0x80000000u;

// Eight reduction elements of a row / column, as they are in memory: bf16 in v[0 .. 3] (pairs), fp32 in v[0 .. 7].
template <int PL, bool IN>
__device__ __forceinline__ void fetch8(const __amdgpu_buffer_rsrc_t r, int i, bool ok, int k, int K, int ld, unsigned (&v)[PL == 1 ? 5 : 8]) {
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    constexpr int ES = PL == 1 ? 2 : 4;
    if (IN) {
        const unsigned off = (unsigned)((size_t)i * ld + k) * ES;
        const unsigned o = ok && k < K ? off & ~3u : NOWHERE;
        const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(r, o, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = x[e];
        if constexpr (PL == 1) {
            v[4] = __builtin_amdgcn_raw_buffer_load_b32(r, o == NOWHERE ? o : o + 16, 0, 0);
        } else {
            const u32x4 y = __builtin_amdgcn_raw_buffer_load_b128(r, o == NOWHERE ? o : o + 16, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 + e] = y[e];
        }
    } else {
        unsigned t[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const unsigned o = ok && k + e < K ? (unsigned)((size_t)(k + e) * ld + i) * ES : NOWHERE;
            t[e] = PL == 1 ? (unsigned)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, o, 0, 0) : (unsigned)__builtin_amdgcn_raw_buffer_load_b32(r, o, 0, 0);
        }
        if constexpr (PL == 1) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = t[2 * e] | t[2 * e + 1] << 16;
            v[4] = 0;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = t[e];
        }
    }
}
// ... lined up, and zeros past the end of the reduction (an inner axis goes on with the next row there)
template <int PL, bool IN>
__device__ __forceinline__ void finish8(unsigned (&v)[PL == 1 ? 5 : 8], int i, int k, int K, int ld) {
    if (!IN) return;
    if constexpr (PL == 1) {
        const unsigned sh = ((unsigned)i * (unsigned)ld + (unsigned)k) & 1 ? 16u : 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = __builtin_amdgcn_alignbit(v[e + 1], v[e], sh);
    }
    if (k + 8 > K) {
        constexpr int PER = PL == 1 ? 2 : 1;
#pragma unroll
        for (int e = 0; e < 8 / PER; ++e) {
            if (PL == 1) v[e] &= (k + 2 * e < K ? 0xffffu : 0u) | (k + 2 * e + 1 < K ? 0xffff0000u : 0u);
            else v[e] = k + e < K ? v[e] : 0u;
        }
    }
}

template <int PL, bool A_IN, bool B_IN, bool OUT16, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void fc_direct_kernel(const FcDirectParams q) {
    constexpr int V = PL == 1 ? 5 : 8;
    __shared__ float sums[WAVES][16][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int khalf = lane >> 5, l31 = lane & 31;
    const int it = blockIdx.x / q.tiles_j, jt = blockIdx.x - it * q.tiles_j;
    const int row = it * 32 + l31, col = jt * 32 + l31;
    const bool a_ok = row < q.rows, b_ok = col < q.cols;
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(q.a), (short)0, (int)q.a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(q.b), (short)0, (int)q.b_bytes, 0x00020000);

    floatx16 hi, lo;
#pragma unroll
    for (int e = 0; e < 16; ++e) { hi[e] = 0.0f; lo[e] = 0.0f; }
    float dsum = 0.0f;
    struct Frag { unsigned a[V], b[V]; };
    auto load = [&](int s, Frag& f) {
        const int k = s * 16 + khalf * 8;
        fetch8<PL, A_IN>(ra, row, a_ok && s < q.steps, k, q.K, q.a_ld, f.a);
        fetch8<PL, B_IN>(rb, col, b_ok && s < q.steps, k, q.K, q.b_ld, f.b);
    };
    auto multiply = [&](int s, Frag& f) {
        const int k = s * 16 + khalf * 8;
        finish8<PL, A_IN>(f.a, row, k, q.K, q.a_ld);
        finish8<PL, B_IN>(f.b, col, k, q.K, q.b_ld);
        if (q.db) {
#pragma unroll
            for (int e = 0; e < (PL == 1 ? 4 : 8); ++e)
                dsum += PL == 1 ? __uint_as_float(f.a[e] << 16) + __uint_as_float(f.a[e] & 0xffff0000u) : __uint_as_float(f.a[e]);
        }
        multiply_loaded<PL>(f.a, f.b, hi, lo);
    };
    // (both axes inner: two or four 16-byte loads a step, so four steps are in flight; else two)
    constexpr int AHEAD = A_IN && B_IN ? 4 : 2;
    Frag f[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) load(wave + u * WAVES, f[u]);
    for (int s = wave; s < q.steps; s += AHEAD * WAVES) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {            // (past the last step: zeros)
            multiply(s + u * WAVES, f[u]);
            load(s + (AHEAD + u) * WAVES, f[u]);
        }
    }

    put_sums<PL>(sums[wave], lane, hi, lo);
    __syncthreads();
    for (int o = tid; o < 1024; o += WAVES * 64) {
        const int e = o >> 6, l = o & 63;
        const int i = it * 32 + (e >> 2) * 8 + (l >> 5) * 4 + (e & 3), j = jt * 32 + (l & 31);
        float t = all_sums<WAVES>(sums, e, l);
        if (i >= q.rows || j >= q.cols) continue;
        if (PL == 3 && !(__builtin_fabsf(t) <= 3.402823466e38f)) {
            // infinities and NaNs: again, as a plain fp32 sum
            const float* a = (const float*)q.a;
            const float* b = (const float*)q.b;
            t = 0.0f;
            for (int k = 0; k < q.K && t == t; ++k)
                t = __builtin_fmaf(a[A_IN ? (size_t)i * q.a_ld + k : (size_t)k * q.a_ld + i], b[B_IN ? (size_t)j * q.b_ld + k : (size_t)k * q.b_ld + j], t);
        }
        const size_t at = (size_t)i * q.cols + j;
        if (q.bias) t += PL == 1 ? __uint_as_float((unsigned)((const uint16_t*)q.bias)[j] << 16) : ((const float*)q.bias)[j];
        if constexpr (OUT16) {
            ((__bf16*)q.out)[at] = (__bf16)t;
        } else {
            float* out = (float*)q.out;
            out[at] = q.beta != 0.0f ? out[at] + t : t;
        }
    }
    if (q.db && jt == 0) {
        __syncthreads();
        float* rows = &sums[0][0][0];
        rows[wave * 64 + lane] = dsum;
        __syncthreads();
        if (tid < 32 && it * 32 + tid < q.rows) {
            double all = 0.0;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) all += (double)rows[w * 64 + tid] + (double)rows[w * 64 + 32 + tid];
            const float t = (float)all;
            float* d = q.db + it * 32 + tid;
            *d = q.beta != 0.0f ? *d + t : t;
        }
    }
}

template <int PL, bool A_IN, bool B_IN, bool OUT16>
hipError_t launch(const FcDirectParams& q, hipStream_t st) {
    const long long tiles = (long long)((q.rows + 31) / 32) * q.tiles_j;
    if (tiles <= 0 || tiles > 0x7fffffffLL) return hipErrorInvalidValue;
    ProbeScope probe(st);
    (void)hipGetLastError();   // drop stale status left by earlier, unrelated runtime calls
    if (q.steps > 32) hipLaunchKernelGGL((fc_direct_kernel<PL, A_IN, B_IN, OUT16, 16>), dim3((unsigned)tiles), dim3(1024), 0, st, q);
    else if (q.steps > 4) hipLaunchKernelGGL((fc_direct_kernel<PL, A_IN, B_IN, OUT16, 8>), dim3((unsigned)tiles), dim3(512), 0, st, q);
    else hipLaunchKernelGGL((fc_direct_kernel<PL, A_IN, B_IN, OUT16, 2>), dim3((unsigned)tiles), dim3(128), 0, st, q);
    return hipGetLastError();
}

}  // namespace

// Whether a pass goes here: its time (fitted to 260 layers drawn from 1 - 256 images, 64 - 9216 inputs, 10 - 4096 outputs: 0.6 - 1.5 of
// the measured ones) against that of the kernels it would take otherwise (their launches, operands at 4.5 TB/s, and the arithmetic they reach).
// us, otherwise / here: y fp32 185 x 499 x 1333 (images, inputs, outputs) 14.6 / 7.2, 64 x 4096 x 1000 17.6 / 34 (stays); dx bf16 34 x 2243 x 2795
// 66 / 18, 128 x 9216 x 4096 38 / 125 (stays); dw bf16 3 x 3273 x 2559 35 / 24, 281 x 2011 x 2591 43 / 55 and 16 x 4096 x 4096 21 / 40 (stay).
// other_splits (weight gradients of more than 256 images): the kernel it would take otherwise has its reduction over workgroups. A wavefront here
// walks N / 256 steps by itself, which more images than the layers above had make the longer way (both sides again fitted to 425
// layers of 257 - 262144 images without db; half of db's time counts against the other kernel, which has a launch of its own for it; the bits
// of dw must not depend on db). us without db, otherwise / here: fp32 32 x 32 at 1024 images 14.4 / 11.9, at 8192 19.6 / 49, at 65536
// 69 / 344; bf16 43 x 33 at 225580 56 / 1062 (these but the first stay). Where the other kernel does not split, it is the slower one at any
// length: fp32 53 x 49 at 752 25 / 11, bf16 512 x 512 at 262144 4962 / 1179.
bool fc_direct_faster(int pass, int64_t N, int64_t C, int64_t K, int dtype, bool other_splits) {
    const bool f32 = dtype == PURINE_F32;
    const int64_t es = f32 ? 4 : 2, most = (1ll << 30) / es;
    if (buffer_loads_disabled() || N >= most || C >= most || K >= most || N * C >= most || K * C >= most / 2 || N * K >= most || small_kernels_disabled()) return false;
    if (direct_forced()) return true;
    const bool grad = pass >= PURINE_CONV_BWD_WEIGHT;
    const int64_t rows = grad ? K : N, cols = pass == PURINE_CONV_FWD ? K : C, len = pass == PURINE_CONV_FWD ? C : grad ? N : K;
    const double steps = (double)((len + 15) / 16), tiles = (double)((rows + 31) / 32) * (double)((cols + 31) / 32), work = tiles * steps * 1e-3;
    const double chain = steps > 32 ? (steps + 15) / 16 : steps > 4 ? (steps + 7) / 8 : (steps + 1) / 2;      // steps of a wavefront
    const double bytes = (grad ? 4.0 : (double)es) * K * C, flops = 2e-6 * (double)N * C * K;
    // (bf16 rows that are whole lines apart: the 32 rows of a load ask few channels. 64 x 1664 x 64 16 us here, 9.5 otherwise; of 47 such layers of up to
    // 256 images and more than 700 inputs 12 went here and were slower, by up to 1.7.)
    const double lines = C % 64 == 0 && steps > 32 ? 1.3 : 1.0;
    if (pass == PURINE_CONV_FWD)
        return f32 ? 1.1 * (3.5 + 1.17 * chain + 1.4e-3 * tiles + 0.44 * work) < 9.0 + bytes / 4.5e6 + flops / 150.0
                   : 1.15 * (2.5 + 0.88 * lines * chain + 0.35 * work) < 9.4 + 0.02 * (double)(N < 80 ? N : 80) + bytes / 4.5e6 + flops / 400.0;
    if (!grad) {
        if (f32) return K > 16 && 1.1 * (3.5 + 0.86 * chain + 2.25e-3 * tiles + 0.42 * work) < 9.5 + bytes / 4.5e6 + flops / 120.0;
        if (C % 8 == 0) return 1.1 * (3.4 + 0.55 * chain + 0.73e-3 * tiles + 0.31 * work) < 6.3 + bytes / 4.5e6 + flops / 400.0;
        // Rows of w that are no whole packets run the general forward convolution otherwise: a chain of slabs of 32 outputs over tiles of 128 x 128, dy
        // copied as its filter bank. Both sides fitted to 301 layers of 1 - 262144 images (0.64 - 1.4 of the measured times). us, otherwise / here:
        // 142 x 30 x 3186 51 / 19, 211369 x 30 x 310 192 / 57; 7405 x 2645 x 108 36 / 123, 8975 x 3409 x 91 41 / 167 (stay).
        const double slabs = (double)((K + 31) / 32), big = (double)((N + 127) / 128) * (double)((C + 127) / 128), rounds = std::ceil(big / 256.0);
        const double here = 3.0 + 0.7 * chain + tiles * (steps > 32 ? 13.3e-3 : steps > 4 ? 4.0e-3 : 1.7e-3) + 0.186 * work;
        return here < 5.2 + 0.5 * slabs + 7.7e-3 * rounds * slabs + 12.1e-3 * big + 2.2e-3 * big * slabs + 2.06e-6 * (double)N * K;
    }
    if (other_splits) {
        const double big = (double)((K + 127) / 128) * (double)((C + 127) / 128), db = 0.6e-6 * (double)N * K;
        const double here = 2.4 + (f32 ? 1.2 : 0.98) * chain + 5.9e-3 * tiles + (f32 ? 0.3 : 0.2) * work;
        const double split = f32 ? 11.7 + 0.57e-3 * (double)N + 2.5e-6 * (double)K * C + 0.23e-3 * big * (double)N
                                 : 15.9 + 1.2e-6 * (double)N * (double)(C + K) + 17.5e-6 * (double)K * C + 0.091e-3 * big * (double)N;
        if (here > split + db) return false;
    }
    if (f32) return 5.5 + 1.3 * (1.97e-3 * tiles + 0.69 * work) < (N <= 32 ? 7.0 : 10.0) + bytes / 4.5e6 + flops / 120.0;
    // (whose operands there are transposed first, and read in pieces if their rows then are no whole packets)
    const double pieces = N % 8 != 0 ? 1.5 + 2.1e-6 * (double)K * C : 0.0;
    return 1.1 * (4.7 + 1.41e-3 * tiles + 0.72 * work) < 11.0 + 0.022 * (double)N + bytes / 4.5e6 + flops / 400.0 + pieces;
}

hipError_t launch_fc_direct(int pass, int dtype, const void* a, const void* b, void* out, const void* bias, float* db, float beta, int64_t N, int64_t C,
                            int64_t K, hipStream_t st) {
    const bool f32 = dtype == PURINE_F32;
    const int es = f32 ? 4 : 2;
    const int64_t rows = pass >= PURINE_CONV_BWD_WEIGHT ? K : N, cols = pass == PURINE_CONV_FWD ? K : C;
    const int64_t len = pass == PURINE_CONV_FWD ? C : pass == PURINE_CONV_BWD_DATA ? K : N;
    FcDirectParams q{};
    q.a = a; q.b = b; q.out = out; q.bias = bias; q.db = db; q.beta = beta;
    q.rows = (int)rows; q.cols = (int)cols; q.K = (int)len;
    q.a_ld = (int)(pass >= PURINE_CONV_BWD_WEIGHT ? rows : len);
    q.b_ld = (int)(pass == PURINE_CONV_FWD ? len : cols);
    q.a_bytes = (unsigned)((rows * len * es + 3) & ~3ll); q.b_bytes = (unsigned)((cols * len * es + 3) & ~3ll);
    q.tiles_j = (int)((cols + 31) / 32); q.steps = (int)((len + 15) / 16);
    if (f32) {
        if (pass == PURINE_CONV_FWD) return launch<3, true, true, false>(q, st);
        if (pass == PURINE_CONV_BWD_DATA) return launch<3, true, false, false>(q, st);
        return launch<3, false, false, false>(q, st);
    }
    if (pass == PURINE_CONV_FWD) return launch<1, true, true, true>(q, st);
    if (pass == PURINE_CONV_BWD_DATA) return launch<1, true, false, true>(q, st);
    return launch<1, false, false, false>(q, st);
}

}  // namespace purine

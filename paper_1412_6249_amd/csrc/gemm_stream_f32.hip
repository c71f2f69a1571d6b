// fp32 GEMMs with an operand that is used (almost) once: the passes of the fully-connected layer, on the bf16
// matrix cores (three exact bf16 parts per operand, six products, two accumulator sets: see conv_packets.hip
// for the arithmetic and its error).
//
//     out[row][column] = sum over k of A[row][k] * B[k][column]
//
// Bound: HBM (the weight matrix: 151 MB at 9216 x 4096) and MFMA about equally at a batch of 128. Nothing is laid out beforehand and
// nothing but the operands is read: a thread loads 8 consecutive reduction elements of one row (A) and of
// one column (B), splits them in registers and stores three 16-byte packets to LDS, two steps of 16 ahead in
// two register sets. An operand's reduction axis is either its inner one (two 16-byte loads per packet) or its outer one (eight 4-byte loads, lanes
// along rows / columns). Two workgroups of four wavefronts per CU, one barrier per step.
//
// 9216 x 4096, batch 128 (58 GFLOP as 6 products: 27 us at 2.1 PFLOP/s; 158 MB: 31 us at 5.1 TB/s), against the
// general fp32 kernels over the same layer: y 118 -> 77 us (the kernel 72), dx 119 -> 86 (69 + 8 for adding the
// splits); the weight gradient 114 -> 90. The rest is the split itself, done again by every tile that shares a
// row or column, and one barrier per 16 elements of the reduction.
#include "packets.h"
#include "pix_common.h"

namespace purine {
namespace pix {
namespace {

using namespace packets;

constexpr int COLS = 128, NT = 256;      // columns and threads of a workgroup's tile

struct StreamParams {
    const float* a; const float* b;
    unsigned a_bytes, b_bytes;
    int a_ld, b_ld;              // elements between rows of the operand as it lies in memory
    int K;                       // reduction length
    int steps, splits, steps_per_split;
    size_t split_stride;         // elements between the splits' partial outputs
};

template <int TM, int TN, int WM, int WN>
struct StreamTile {
    static constexpr int BM = TM * WM * 32, BN = COLS;
    static constexpr int A_BYTES = PLANES * 2 * BM * 16, B_BYTES = PLANES * 2 * BN * 16, STAGE = A_BYTES + B_BYTES;
    static constexpr int LDS = 2 * STAGE;
    static_assert(TN * WN * 32 == BN && WM * WN * 64 == NT && BM * 2 <= NT, "");
};

// A_IN / B_IN: the reduction is the operand's inner axis. Buffer loads of 16 bytes need 4-byte alignment only and
// are range-checked by the dword, so rows need not be whole packets.
template <bool A_IN, bool B_IN, int TM, int TN, int WM, int WN>
__global__ __launch_bounds__(NT, 2) void gemm_stream_f32_kernel(const PixParams p, const StreamParams q) {
    typedef StreamTile<TM, TN, WM, WN> T;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int BN = COLS;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int khalf = lane >> 5;
    const int wm = wave / WN, wn = wave % WN;
    const int id = xcd_tile(blockIdx.x, gridDim.x);
    const int per_split = p.tiles_i * p.tiles_pix;
    const int split = id / per_split, tile = id - split * per_split;
    const int pt = tile / p.tiles_i, rt = tile - pt * p.tiles_i;
    const int i0 = rt * T::BM, j0 = pt * BN;
    const int s0 = split * q.steps_per_split, s1 = min(s0 + q.steps_per_split, q.steps);

    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(q.a), (short)0, (int)q.a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(q.b), (short)0, (int)q.b_bytes, 0x00020000);

    // this thread's packet of each tile: byte offset of its first element at step 0, LDS place
    const int a_row = A_IN ? tid >> 1 : tid % T::BM, a_half = A_IN ? tid & 1 : tid / T::BM;
    const bool a_mine = T::BM * 2 == NT || tid < T::BM * 2;
    const bool a_ok = a_mine && i0 + a_row < p.Co;
    const unsigned a_off = (unsigned)(A_IN ? (i0 + a_row) * q.a_ld + a_half * 8 : a_half * 8 * q.a_ld + i0 + a_row) * 4u;
    const int a_dst = (a_half * T::BM + a_row) * 16;
    const int b_col = B_IN ? tid >> 1 : tid & (BN - 1), b_half = B_IN ? tid & 1 : tid >> 7;
    const int col = j0 + b_col;
    const bool b_ok = col < p.M;
    unsigned b_off = 0;
    if (B_IN) b_off = (unsigned)((b_ok ? col : 0) * q.b_ld + b_half * 8) * 4u;
    else b_off = (unsigned)((b_ok ? col : 0) + b_half * 8 * q.b_ld) * 4u;
    const int b_dst = T::A_BYTES + (b_half * BN + b_col) * 16;

    struct Regs { float a[8], b[8]; };
    // Elements past the end of the reduction: A's are made zeros in store(). B's are zeros, or (whole packets of
    // an inner axis) whatever lies there: the next row, or past the tensor the range check's zeros; should it be
    // infinite or NaN, the output is computed again below. The range check subtracts the scalar offset from the
    // tensor's size, so that offset has to lie inside the tensor: in a step that is not whole the elements'
    // offsets are the lanes' own.
    auto fetch = [&](const __amdgpu_buffer_rsrc_t& r, bool inner, unsigned off, bool ok, int k0, int kt, int ld, float (&v)[8]) {
        const int soff = inner ? k0 * 4 : k0 * ld * 4;
        if (inner) {
            const unsigned o = ok ? off : 0x80000000u;
            const floatx4 lo4 = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, o, soff, 0));
            const floatx4 hi4 = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, o + 16, soff, 0));
#pragma unroll
            for (int e = 0; e < 4; ++e) { v[e] = lo4[e]; v[4 + e] = hi4[e]; }
        } else if (k0 + 16 <= q.K) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                v[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, ok ? off : 0x80000000u, soff + e * ld * 4, 0));
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                v[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, ok && kt + e < q.K ? off + (unsigned)(e * ld * 4) : 0x80000000u, soff, 0));
        }
    };
    auto load = [&](int s, Regs& g) {
        const bool live = s < s1;
        const int k0 = live ? s * 16 : 0;
        fetch(ra, A_IN, a_off, a_ok && live, k0, k0 + a_half * 8, q.a_ld, g.a);
        fetch(rb, B_IN, b_off, b_ok && live, k0, k0 + b_half * 8, q.b_ld, g.b);
    };
    auto put = [&](const float (&v)[8], unsigned char* dst, int plane) {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        u32x4 pk[PLANES];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t part[PLANES];
            split_pair(v[2 * e], v[2 * e + 1], part);
#pragma unroll
            for (int pl = 0; pl < PLANES; ++pl) pk[pl][e] = part[pl];
        }
#pragma unroll
        for (int pl = 0; pl < PLANES; ++pl) *reinterpret_cast<u32x4*>(dst + pl * plane) = pk[pl];
    };
    auto store = [&](int s, Regs& g, int slot) {
        const int lim = q.K - s * 16 - a_half * 8;        // elements of this thread's A packet that exist
#pragma unroll
        for (int e = 0; e < 8; ++e) g.a[e] = e < lim ? g.a[e] : 0.0f;
        if (a_mine) put(g.a, smem + slot * T::STAGE + a_dst, 2 * T::BM * 16);
        __builtin_amdgcn_sched_barrier(0);         // (one packet's parts at a time: the registers are full)
        put(g.b, smem + slot * T::STAGE + b_dst, 2 * BN * 16);
    };

    floatx16 hi[TM][TN], lo[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) { hi[a][b][e] = 0.0f; lo[a][b][e] = 0.0f; }
    const int a_frag = (khalf * T::BM + wm * TM * 32 + (lane & 31)) * 16;
    const int b_frag = T::A_BYTES + (khalf * BN + wn * TN * 32 + (lane & 31)) * 16;

    Regs g0, g1;
    load(s0, g0);
    load(s0 + 1, g1);
    store(s0, g0, 0);
    load(s0 + 2, g0);
    // step s: its tiles are in slot s & 1; the next step's wait in registers, the one after that is on its way
    auto step = [&](int s, Regs& next) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xc07f);        // lgkmcnt(0): this wavefront's LDS traffic is done; loads stay in flight
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const int slot = (s - s0) & 1;
        multiply_step<T, TM, TN>(smem + slot * T::STAGE, a_frag, b_frag, hi, lo);
        __builtin_amdgcn_sched_barrier(0);
        store(s + 1, next, slot ^ 1);
        load(s + 3, next);
        __builtin_amdgcn_sched_barrier(0);
    };
    // (an odd last step is followed by one of zeros: a tail of its own makes the compiler copy every accumulator
    // in every turn of the loop)
    for (int s = s0; s < s1; s += 2) {
        step(s, g1);
        step(s + 1, g0);
    }

    // infinities and NaNs: again, as plain fp32 sums
    unsigned long long bad = join_sets<TM, TN>(hi, lo);
    if (__builtin_expect(__any(bad != 0), 0)) {
        while (bad) {
            const int idx = __ffsll((long long)bad) - 1;
            bad &= bad - 1;
            const int ab = idx >> 4, e = idx & 15;
            const int row = i0 + wm * TM * 32 + (ab / TN) * 32 + (e >> 2) * 8 + khalf * 4 + (e & 3);
            const int c = j0 + wn * TN * 32 + (ab % TN) * 32 + (lane & 31);
            float sum = 0.0f;
            if (row < p.Co && c < p.M) {
                const float* pb = q.b + (B_IN ? (size_t)c * q.b_ld : (size_t)c);
                const int k1 = min(s1 * 16, q.K);
                for (int k = s0 * 16; k < k1 && sum == sum; ++k)
                    sum = __builtin_fmaf(q.a[A_IN ? (size_t)row * q.a_ld + k : (size_t)k * q.a_ld + row],
                                         pb[B_IN ? (size_t)k : (size_t)k * q.b_ld], sum);
            }
            replace_element<TM, TN>(hi, idx, sum);
        }
    }
    store_tile<float, false, false, TM, TN, false>(p, (float*)p.out + (size_t)split * q.split_stride, hi, i0 + wm * TM * 32,
                                                 j0 + wn * TN * 32 + (lane & 31), khalf, nullptr, i0);
}

// Second pass of a split reduction over a dense matrix [rows][cols]: partial sums added in split order, plus a
// bias per column (or null). Four columns per thread where the rows are whole packets.
template <int V>
__global__ __launch_bounds__(256) void stream_reduce_kernel(const float* __restrict__ partial, float* __restrict__ out, const float* __restrict__ bias,
                                                            int splits, size_t total, int cols, float beta) {
    for (size_t t = ((size_t)blockIdx.x * 256 + threadIdx.x) * V; t < total; t += (size_t)gridDim.x * 256 * V) {
        float v[V];
#pragma unroll
        for (int e = 0; e < V; ++e) v[e] = 0.0f;
#pragma unroll 4
        for (int s = 0; s < splits; ++s) {
            if (V == 4) {
                const floatx4 x = *reinterpret_cast<const floatx4*>(partial + (size_t)s * total + t);
#pragma unroll
                for (int e = 0; e < V; ++e) v[e] += x[e];
            } else {
                v[0] += partial[(size_t)s * total + t];
            }
        }
        const int c = (int)(t % (size_t)cols);
#pragma unroll
        for (int e = 0; e < V; ++e) {
            if (bias) v[e] += bias[c + e];
            if (beta != 0.0f) v[e] += out[t + e];
            out[t + e] = v[e];
        }
    }
}

template <bool A_IN, bool B_IN, int TM, int TN, int WM, int WN>
hipError_t launch_main(const PixParams& p, const StreamParams& q, hipStream_t st) {
    typedef StreamTile<TM, TN, WM, WN> T;
    const long long total = (long long)p.tiles_i * p.tiles_pix * q.splits;
    if (total <= 0 || total > 0x7fffffffLL) return hipErrorInvalidValue;
    ProbeScope probe(st);
    (void)hipGetLastError();   // drop stale status left by earlier, unrelated runtime calls
    hipLaunchKernelGGL((gemm_stream_f32_kernel<A_IN, B_IN, TM, TN, WM, WN>), dim3((unsigned)total), dim3(NT), T::LDS, st, p, q);
    return hipGetLastError();
}

// Row tiles of a form. Eight 4-byte loads per packet need more registers than two 16-byte ones: with both operands
// read along their outer axis 128 rows spill 208 registers and 96 rows 52, with one of them 96 rows spill 32 (weight
// gradient 3140 x 1780 of 33 images, 128 rows: 49 us, the general kernel 17; backward-data 9216 x 4096 of 131
// images, 96 rows: 175 us, the general kernel 121).
constexpr bool has_tile(bool a_in, bool b_in, int bm) { return bm <= 64 || (a_in && (b_in || bm == 128)); }

template <bool A_IN, bool B_IN>
hipError_t by_tile(const PixParams& p, const StreamParams& q, int bm, hipStream_t st) {
    switch (bm) {
        case 128: if constexpr (has_tile(A_IN, B_IN, 128)) return launch_main<A_IN, B_IN, 2, 2, 2, 2>(p, q, st); return hipErrorInvalidValue;
        case 96:  if constexpr (has_tile(A_IN, B_IN, 96)) return launch_main<A_IN, B_IN, 3, 1, 1, 4>(p, q, st); return hipErrorInvalidValue;
        case 64:  return launch_main<A_IN, B_IN, 1, 2, 2, 2>(p, q, st);
        case 32:  return launch_main<A_IN, B_IN, 1, 1, 1, 4>(p, q, st);
        default: return hipErrorInvalidValue;
    }
}

struct RowTile { int bm, cycles; float eff; };
constexpr RowTile kTilesS[] = {{128, 768, 0.62f}, {96, 576, 0.58f}, {64, 384, 0.52f}, {32, 192, 0.35f}};

}  // namespace

// rows x cols over K; a_in, b_in as in launch_stream_gemm. Model as in plan_packets, with the memory's time as a
// second floor: operands and output once, partial outputs twice.
StreamPlan plan_stream(long long rows, long long cols, long long K, bool a_in, bool b_in) {
    StreamPlan k{};
    const long long steps = (K + 15) / 16;
    if (rows < 1 || cols < 1 || K < 1 || steps > (1 << 26)) return k;
    const double mem_us = 4.0 * ((double)rows * K + (double)cols * K + (double)rows * cols) / 4.5e6;
    for (const RowTile& t : kTilesS) {
        const long long ti = (rows + t.bm - 1) / t.bm, tp = (cols + COLS - 1) / COLS, tiles = ti * tp;
        if (tiles > 0x7fffffffLL || !has_tile(a_in, b_in, t.bm)) continue;
        // B along its outer axis and too large for the caches, read again by every row tile: 9216 x 4096, 131 images on three
        // tiles of 64 rows 153 us, on five of 32 rows 135 - 155, 200 images on two of 128 rows 115
        const double eff = a_in && !b_in && t.bm <= 64 && ti > 2 && (double)cols * K * 4.0 > 60e6 ? 0.77 * t.eff : t.eff;
        long long last = -1;
        for (int half_fill = 0; half_fill <= 8; ++half_fill) {
            long long sp = half_fill * 128 / tiles;
            if (sp < 1) sp = 1;
            if (sp > 64) sp = 64;
            const long long per = (steps + sp - 1) / sp;
            sp = (steps + per - 1) / per;
            if (per == last) continue;
            last = per;
            const double part = sp > 1 ? 4.0 * sp * rows * cols : 0.0;
            if (part > 128.0 * (1 << 20)) break;
            const double x = (double)(tiles * sp) / 256.0;
            // 512 workgroups are resident (of the smallest tile 1024): a few more than a whole number of rounds
            // cost almost another round
            const int resident = t.bm == 32 ? 4 : 2;          // per CU
            const double rounds = (double)((tiles * sp + 256 * resident - 1) / (256 * resident));
            const double ragged = x > resident ? 0.5 + 0.5 * rounds * resident / x : 1.0;
            const double load = x <= 1.0 ? 1.45 : x <= 2.0 ? 0.5 * (x + 2.0) : x * ragged;
            // B along its outer axis, one workgroup for the whole sum: a step takes its time however little there is to
            // multiply, 16 loads, their split and a barrier (247 x 169, 128 images, backward-data: 16 steps 16.2 us, split
            // one by one 8.6 with the second pass; weight gradient 64 x 10 of 128: 8 steps of 32 rows 10 us, of 64 12)
            const double chain_us = b_in || sp > 1 ? 0.0 : (t.bm == 32 ? 0.7 : 0.95) * (double)per;
            double mma_us = load * ((double)per * t.cycles / eff + 3000.0) / 2.2e3;
            if (mma_us < chain_us) mma_us = chain_us;
            // fewer than two workgroups per CU (of the smallest tile three) do not keep enough loads in flight
            const double mem = mem_us * ragged / (x >= (t.bm == 32 ? 2.6 : 1.9) ? 1.0 : x >= 1.0 ? 0.8 : 0.8 * x);
            const double us = (mma_us > mem ? mma_us + 0.3 * mem : mem + 0.3 * mma_us) + 6.0 + (sp > 1 ? 6.0 + 2.0 * part / 7e6 : 0.0);
            if (!k.use || us < k.us) {
                k.use = true; k.us = us;
                k.bm = t.bm; k.tiles_i = (int)ti; k.tiles_pix = (int)tp;
                k.steps = (int)steps; k.splits = (int)sp; k.steps_per_split = (int)per;
                k.part_bytes = (size_t)part;
            }
        }
    }
    return k;
}

// Dense matrices: out[rows][cols] (+)= A * B, A [rows][K] (a_in) or [K][rows], B [cols][K] (b_in) or
// [K][cols]; bias: per column, or null. (a_in, b_in) = (1, 1), (1, 0) or (0, 0).
hipError_t launch_stream_gemm(const StreamPlan& k, const void* a, bool a_in, const void* b, bool b_in, void* out, const void* bias, float beta,
                              long long rows, long long cols, long long K, void* ws, hipStream_t st) {
    PixParams p{};
    p.N = 1; p.Co = (int)rows; p.Ci = (int)K; p.HoWo = p.HiWi = p.Wo = (int)cols; p.Ho = 1; p.M = (int)cols;
    p.out_ns = (int)(rows * cols);
    p.div_howo = make_fastdiv((uint32_t)cols); p.div_wo = p.div_howo;
    p.out_bytes = rows * cols * 4 < 0x7fffffffLL && !buffer_loads_disabled() ? (unsigned)(rows * cols * 4) : 0u;
    p.tiles_i = k.tiles_i; p.tiles_pix = k.tiles_pix;
    p.out = out; p.beta = beta;
    StreamParams q{};
    q.a = (const float*)a; q.b = (const float*)b;
    q.a_bytes = (unsigned)(rows * K * 4); q.b_bytes = (unsigned)(cols * K * 4);
    q.a_ld = (int)(a_in ? K : rows); q.b_ld = (int)(b_in ? K : cols);
    q.K = (int)K; q.steps = k.steps; q.splits = k.splits; q.steps_per_split = k.steps_per_split;
    const bool second = k.splits > 1;
    if (second) {
        if (!ws) return hipErrorInvalidValue;
        p.out = ws; p.beta = 0.0f;
        q.split_stride = (size_t)rows * cols;
    }
    hipError_t e;
    if (a_in && b_in) e = by_tile<true, true>(p, q, k.bm, st);
    else if (a_in) e = by_tile<true, false>(p, q, k.bm, st);
    else if (!b_in) e = by_tile<false, false>(p, q, k.bm, st);
    else return hipErrorInvalidValue;
    if (e != hipSuccess || !second) return e;
    const size_t total = (size_t)rows * cols;
    const bool v4 = cols % 4 == 0;
    const size_t threads = v4 ? total / 4 : total;
    const unsigned blocks = (unsigned)((threads + 255) / 256 > 4096 ? 4096 : (threads + 255) / 256);
    if (v4) hipLaunchKernelGGL((stream_reduce_kernel<4>), dim3(blocks), dim3(256), 0, st, (const float*)ws, (float*)out, (const float*)bias, k.splits, total, (int)cols, beta);
    else hipLaunchKernelGGL((stream_reduce_kernel<1>), dim3(blocks), dim3(256), 0, st, (const float*)ws, (float*)out, (const float*)bias, k.splits, total, (int)cols, beta);
    return hipGetLastError();
}

}  // namespace pix
}  // namespace purine

// Weight gradients whose operands are laid out inside LDS (bf16, and fp32 as three exact bf16 parts with six products and two
// accumulator sets: see conv_packets.hip for the arithmetic and its measured error).
//
// dw[k, (r, s, c)] = sum over (image, output position) of dy[k, position] * x[c, position shifted by the tap]. The MFMA wants
// eight consecutive reduction elements per lane; they are EIGHT IMAGES at one position, as in conv_wgrad_packets.hip, so that a tap
// is a whole number of 16-byte packets away whatever its offset, the stride, the padding or the width of a row. There the
// packets are made in scratch memory by a pass of their own (ten bytes per fp32 element, which layers of few channels or
// one tap do not earn back); here a workgroup makes them on the way into LDS: a chunk is PR x QS output positions of a
// group of eight images, its dy as [part][position][k] and the patch of x that its taps touch as [part][row][column][c].
// Each tap then reads the patch at an offset of its own: a lane's offset is fixed for its column (r, s, c), a step's is one
// scalar. Batches that are no multiple of eight images are cut into bands of output rows (1, 2, 4 or 8 per image), eight
// bands to a group. 1x1 layers as they lie in memory (FLAT) need no such exchange: there a packet is eight consecutive elements
// of a plane, and a chunk 64 of them.
//
// Bound: none of the roofs. conv1 of the five-layer stack (3 -> 96 channels 11x11 / 4 at 227x227, N = 128) has its matrix pipes 41 % busy (when it
// took a quarter longer 32 %, the address units 65 %, VALU and LDS a third each). What sets the pace is a chunk's chain of loads, packing and multiplication
// (2.5 - 4 us), so it is taken apart: four wavefronts request and pack dy, four x, one chunk ahead and with the loads of the next in
// flight, into two LDS buffers in turn; the others only multiply. (The same wavefronts doing both in turn, two workgroups per CU: 290 us
// for that layer; loads and packing on wavefronts of their own, a lane loading one position of eight images: 278; four positions, 16 bytes per
// load, neighbouring lanes on neighbouring columns: 247. Loads with lanes along channels ask for each line once per lane: 8800 cycles a
// chunk to issue them instead of 3000.)
//
// Whole operator with the bias gradient, general kernel / here, us (three sets of tensors in turn): that layer 294 / 218; 3 -> 170 7x7 / 2 at
// 174x175, N = 88 672 / 321; 3 -> 344 7x7 / 2 at 199x199, N = 10 266 / 112; 272 -> 126 1x1 at 26x26, N = 1 15.6 / 10.3; 16 -> 32 5x5 at
// 28x28, N = 128 59 / 42; bf16 3 -> 139 7x7 / 2 at 184x186, N = 106 638 / 179; 3 -> 220 7x7 / 2 at 65x66, N = 140 152 / 60.
#include <type_traits>
#include "packets.h"
#include "pix_common.h"

namespace purine {
namespace {

using namespace packets;

struct StagedParams {
    const void* x; const void* dy;
    float* out;                      // partial sums [split][K][channel tile][r][s][c of the tile], or dw itself (direct)
    float* db_out;                   // [split][K], or db itself; or null
    unsigned x_bytes, dy_bytes;
    int N, C, H, W, K, P, Q, R, S, sh, sw, ph, pw, x_ns, dy_ns;
    int RS, J;                       // taps; columns in all
    int Ct, CtP;                     // channels of a tile; packets between the columns of the patch
    int tiles_i, tiles_j, c_tiles;   // row tiles, column tiles of a channel tile, channel tiles
    int band_shift, PB;              // bands per image (log2), output rows of a band
    int Qc;                          // packets along a row of dy: Q, or (flat) a plane's eighths
    int PR, QS, qsegs, pchunks, chunks, splits;
    int PW, XR, lead;                // patch: columns, rows at most; columns before the first that counts
    int dquads, xquads;              // units of a row of dy and of x
    int d_plane, x_off, x_plane;     // LDS: bytes between parts; where the patch begins
    int buf_bytes;                   // ... of one chunk
    int direct;
    float beta;
    FastDiv div_dquads, div_pr, div_xquads, div_xr, div_qsegs, div_pchunks, div_s, div_ct, div_cl;
};

// Lanes that load each of the two tensors, and units that a lane holds for a chunk: a unit is four positions (columns) of one
// channel of the group's eight images, four packets.
constexpr int LOADERS = 256;
constexpr int units_of(int PL) { return PL == 1 ? 2 : 1; }
constexpr unsigned NOWHERE = 0x80000000u;      // offset of what does not exist: beyond any tensor of less than 2^31 bytes

struct Chunk { int p0, q0, pr_n, qn, grp; };
__device__ __forceinline__ Chunk chunk_at(const StagedParams& q, int ch) {
    const int t = fastdiv(ch, q.div_qsegs), grp = fastdiv(t, q.div_pchunks);
    Chunk c;
    c.q0 = (ch - t * q.qsegs) * q.QS; c.p0 = (t - grp * q.pchunks) * q.PR; c.grp = grp;
    c.pr_n = min(q.PR, q.PB - c.p0); c.qn = min(q.QS, q.Qc - c.q0);
    if (ch >= q.chunks) c.pr_n = c.qn = 0;       // nothing of it is there
    return c;
}

// (a bare barrier: a fence would wait for the loads in flight as well)
__device__ __forceinline__ void meet() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);      // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The wavefronts that load dy (X = false) or x: chunk after chunk into the two buffers in turn, its loads requested one chunk ahead of
// their packing. Rows of a tile: BM channels of dy from k0, cw channels of x from c0.
// FAR: images so far apart that a tensor spans 2^31 bytes or more. x_bytes and dy_bytes are an image's, and each image is read through a
// descriptor of its own (of whole dwords: images of a dense bf16 tensor beside a far one may begin in the middle of one).
template <int PL, bool X, bool FLAT, bool FAR, int BM>
__device__ __forceinline__ void load_chunks(const StagedParams& q, unsigned char* smem, int lt, int k0, int c0, int cw, int r_first, int nr, int split, int n, bool do_db) {
    static_assert(!FLAT || PL == 3, "bf16 planes as they lie in memory: the general kernel");
    constexpr int ES = PL == 1 ? 2 : 4, U = units_of(PL), DW = PL == 1 ? 3 : 4, DP = BM + 1;
    unsigned char* const from = static_cast<unsigned char*>(const_cast<void*>(X ? q.x : q.dy));
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(from, (short)0, (int)(X ? q.x_bytes : q.dy_bytes), 0x00020000);
    const int Ws = X ? q.W : q.Q, Hs = X ? q.H : q.P, ns = X ? q.x_ns : q.dy_ns, bands = 1 << q.band_shift;
    const int stride = (X ? q.CtP : DP) * 16, plane = X ? q.x_plane : q.d_plane;

    // the lane's units: offset from the chunk's (its patch's) first element, and place in LDS (/ 16), column / 4 and row in one.
    // Neighbouring lanes take neighbouring columns, so that a line is asked for once.
    // (FLAT: a packet is eight consecutive elements of a plane; a unit's four belong to channels LOADERS / 8 apart, and
    // neighbouring lanes take neighbouring packets: 256 bytes of fp32 in a row.)
    constexpr int B = FLAT ? 4 : 1;
    unsigned base[U * B], where[U * B];
#pragma unroll
    for (int u = 0; u < U * B; ++u) {
        if (FLAT) {
            const int oct = lt & 7, ch = (lt >> 3) + u * (LOADERS / 8);
            const bool in = ch < (X ? cw : BM);
            base[u] = in && (X || k0 + ch < q.K) ? (unsigned)(((X ? c0 : k0) + ch) * Ws + oct * 8) * ES : NOWHERE;
            where[u] = in ? (unsigned)(X ? (q.x_off >> 4) + oct * q.CtP + ch : oct * DP + ch) | (unsigned)(oct * 8) << 14 : 0xffffffffu;
            continue;
        }
        const int i = lt + u * LOADERS;
        const int v = fastdiv(i, X ? q.div_xquads : q.div_dquads), quad = i - v * (X ? q.xquads : q.dquads);
        const int ch = fastdiv(v, X ? q.div_xr : q.div_pr), row = v - ch * (X ? q.XR : q.PR);
        const bool in = ch < (X ? cw : BM), there = X ? in : in && k0 + ch < q.K;
        base[u] = there ? (unsigned)((((X ? c0 : k0) + ch) * Hs + row) * Ws + quad * 4) * ES : NOWHERE;
        where[u] = in ? (unsigned)(X ? (q.x_off >> 4) + (row * q.PW + quad * 4) * q.CtP + ch : (row * q.QS + quad * 4) * DP + ch) | (unsigned)quad << 14 |
                            (unsigned)row << 24 : 0xffffffffu;
    }
    // a chunk's loads, and what is to be known when they have landed
    struct Units {
        unsigned v[U][8][DW];
        int c0, c1;                      // columns that exist
        bool cut;                        // ... and those outside can meet an operand that counts
        unsigned odd;                    // bf16: images whose first element lies in the upper half of a dword
    };
    auto request = [&](int ch, Units& t) {
        const Chunk c = chunk_at(q, ch);
        unsigned vo[U][8];
        size_t image[8] = {};                              // FAR: where the image begins
        if (FLAT) {
            const int first = c.q0 * 8;
            const unsigned off = (unsigned)((FAR ? 0 : c.grp * ns) + first) * ES;
#pragma unroll
            for (int e = 0; e < 8; ++e) image[e] = FAR && c.pr_n ? (size_t)c.grp * ns * ES : 0;
            t.c0 = 0; t.c1 = c.pr_n ? min(c.qn * 8, Ws - first) : 0;
            t.cut = t.c1 & 7;
            t.odd = 0;
#pragma unroll
            for (int u = 0; u < U * B; ++u) {
                const int col = (where[u] >> 14) & 1023;
                const unsigned o = base[u] + off;
                const bool ok = col < t.c1 && base[u] != NOWHERE;
                vo[u / 4][u % 4 * 2] = ok ? o : NOWHERE;
                vo[u / 4][u % 4 * 2 + 1] = ok && col + 4 < t.c1 ? o + 4 * ES : NOWHERE;
            }
        } else {
            const int w0 = X ? c.q0 * q.sw - q.pw - q.lead : c.q0;
            const int rows = X ? (c.pr_n - 1) * q.sh + nr : c.pr_n;
            t.c0 = X ? -w0 : 0; t.c1 = X ? q.W - w0 : c.qn;
            const int u0 = X ? max(q.lead, t.c0) : 0, u1 = X ? min(q.lead + (c.qn - 1) * q.sw + q.S, t.c1) : c.qn;      // ... and are used
            // (dy: the position after an odd number of them is multiplied, too, and a unit's four go into the bias gradient)
            t.cut = X ? t.c0 > q.lead || t.c1 < q.lead + (c.qn - 1) * q.sw + q.S : c.qn & 3;
            t.odd = 0;
            // (The loads themselves stay out of the branch: a register loaded on one side only would be waited for where the sides meet.)
            if (!FAR && q.band_shift == 0 && c.grp * 8 + 8 <= q.N) {
                // eight whole images: the same rows exist in all of them
                const int h0 = X ? c.p0 * q.sh - q.ph + r_first : c.p0, b0 = X ? max(0, -h0) : 0, b1 = min(rows, Hs - h0);
                const unsigned lo = (unsigned)b0 << 24, len = (unsigned)max(0, b1 - b0) << 24;
                const unsigned off = (unsigned)(c.grp * 8 * ns + h0 * Ws + w0) * ES, step = (unsigned)ns * ES;
                if (PL == 1) t.odd = (off & 2 ? 0xffu : 0u) ^ (step & 2 ? 0xaau : 0u);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int col = (where[u] >> 12) & 4092;
                    const bool ok = where[u] - lo < len && col + 3 >= u0 && col < u1 && base[u] != NOWHERE;
                    unsigned o = ok ? base[u] + off : NOWHERE;
                    const unsigned s = ok ? step : 0u;
#pragma unroll
                    for (int e = 0; e < 8; ++e, o += s) vo[u][e] = PL == 1 ? o & ~3u : o;
                }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int im = c.grp * 8 + e, im_n = im >> q.band_shift, p = (im & (bands - 1)) * q.PB + c.p0;
                    const bool there = im_n < q.N && p < q.P;
                    const int h0 = X ? p * q.sh - q.ph + r_first : p, b0 = X ? max(0, -h0) : 0, b1 = there ? min(rows, Hs - h0) : 0;
                    const unsigned lo = (unsigned)b0 << 24, len = (unsigned)max(0, b1 - b0) << 24;
                    const size_t at = FAR && there ? (size_t)im_n * ns * ES : 0;
                    image[e] = at;
                    const unsigned off = there ? (unsigned)((FAR ? 0 : im_n * ns) + h0 * Ws + w0) * ES + (unsigned)(at & 3) : 0u;
                    if (PL == 1) t.odd |= (off >> 1 & 1) << e;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int col = (where[u] >> 12) & 4092;
                        const bool ok = where[u] - lo < len && col + 3 >= u0 && col < u1 && base[u] != NOWHERE;
                        const unsigned o = base[u] + off;
                        vo[u][e] = ok ? PL == 1 ? o & ~3u : o : NOWHERE;
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                typedef unsigned u32x3 __attribute__((ext_vector_type(3)));
                typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
                const __amdgpu_buffer_rsrc_t re = FAR ? __builtin_amdgcn_make_buffer_rsrc(from + (image[e] & ~(size_t)3), (short)0, (int)(((X ? q.x_bytes : q.dy_bytes) + (unsigned)(image[e] & 3) + 3) & ~3u), 0x00020000) : r;
                if constexpr (PL == 1) {
                    const u32x3 l = __builtin_amdgcn_raw_buffer_load_b96(re, vo[u][e], 0, 0);
#pragma unroll
                    for (int j = 0; j < DW; ++j) t.v[u][e][j] = l[j];
                } else {
                    const u32x4 l = __builtin_amdgcn_raw_buffer_load_b128(re, vo[u][e], 0, 0);
#pragma unroll
                    for (int j = 0; j < DW; ++j) t.v[u][e][j] = l[j];
                }
            }
    };
    // The four packets of every unit. What was read outside the columns that exist belongs to another row: zero.
    float db_sum[U * B];
#pragma unroll
    for (int u = 0; u < U * B; ++u) db_sum[u] = 0.0f;
    auto commit = [&](Units& t, unsigned char* buf) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!FLAT && where[u] == 0xffffffffu) continue;
            unsigned (&v)[8][DW] = t.v[u];
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int j = 0; j < DW; ++j) asm volatile("" : "+v"(v[e][j]));      // here, not where the loads were requested
            if constexpr (PL == 1) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const unsigned s0 = (base[u] & 2) * 8, s = t.odd >> e & 1 ? 16 - s0 : s0;
                    v[e][0] = __builtin_amdgcn_alignbit(v[e][1], v[e][0], s);
                    v[e][1] = __builtin_amdgcn_alignbit(v[e][2], v[e][1], s);
                }
            }
            constexpr int PER = PL == 1 ? 2 : 1;      // elements of a dword
            if (t.cut) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
#pragma unroll
                    for (int j = 0; j < 4 / PER; ++j) {
                        const int a = FLAT ? (int)((where[FLAT ? u * 4 + e / 2 : u] >> 14) & 1023) + e % 2 * 4 + j * PER : (int)((where[u] >> 12) & 4092) + j * PER;
                        if (PL == 1) v[e][j] &= (a >= t.c0 && a < t.c1 ? 0xffffu : 0u) | (a + 1 >= t.c0 && a + 1 < t.c1 ? 0xffff0000u : 0u);
                        else v[e][j] = a >= t.c0 && a < t.c1 ? v[e][j] : 0u;
                    }
            }
            // fused bias gradient: of fp32 values, before they are split
            if (!X && do_db) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float s;
                    if (PL == 1) s = (__uint_as_float(v[e][0] << 16) + __uint_as_float(v[e][0] & 0xffff0000u)) + (__uint_as_float(v[e][1] << 16) + __uint_as_float(v[e][1] & 0xffff0000u));
                    else s = (__uint_as_float(v[e][0]) + __uint_as_float(v[e][1])) + (__uint_as_float(v[e][2]) + __uint_as_float(v[e][DW - 1]));
                    db_sum[FLAT ? u * 4 + e / 2 : u] += s;
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const unsigned to = where[FLAT ? u * 4 + j : u];
                unsigned char* dst = buf + (to & 16383u) * 16 + (FLAT ? 0 : j * stride);
                if (FLAT && to == 0xffffffffu) continue;
                if constexpr (PL == 1) {
                    const unsigned pick = j & 1 ? 0x07060302u : 0x05040100u;
                    const uint4 w = make_uint4(__builtin_amdgcn_perm(v[1][j >> 1], v[0][j >> 1], pick), __builtin_amdgcn_perm(v[3][j >> 1], v[2][j >> 1], pick),
                                               __builtin_amdgcn_perm(v[5][j >> 1], v[4][j >> 1], pick), __builtin_amdgcn_perm(v[7][j >> 1], v[6][j >> 1], pick));
                    *reinterpret_cast<uint4*>(dst) = w;
                } else {
                    float f[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) f[e] = __uint_as_float(FLAT ? v[2 * j + e / 4][e % 4] : v[e][j]);
                    store_split8(f, dst, plane);
                }
            }
        }
    };
    Units even, odd;
    for (int i = 0; i <= n; i += 2) {
        request(split + i * q.splits, even);
        if (i > 0) {
            commit(odd, smem + q.buf_bytes);
            meet();
        }
        if (i == n) break;
        request(split + (i + 1) * q.splits, odd);
        commit(even, smem);
        meet();
    }
    // the bias gradient's sums of a channel lie in neighbouring places; the first buffer is free (n is even)
    if (!X && do_db) {
        float* sums = reinterpret_cast<float*>(smem);
#pragma unroll
        for (int u = 0; u < U * B; ++u) sums[lt + u * LOADERS] = db_sum[u];
    }
    meet();
    if (!X && do_db) {
        const float* sums = reinterpret_cast<const float*>(smem);
        const int per = FLAT ? 8 : q.PR * q.dquads;
        if (lt < BM && k0 + lt < q.K) {
            float t = 0.0f;
            for (int i = 0; i < per; ++i) t += sums[lt * per + i];
            float* d = q.db_out + (size_t)split * q.K + k0 + lt;
            *d = q.direct && q.beta != 0.0f ? *d + t : t;
        }
    }
}

template <int PL, bool FLAT, bool FAR, int TM, int TN, int WM, int WN>
__global__ __launch_bounds__(WM * WN * 64 + 2 * LOADERS, 2) void wgrad_staged_kernel(const StagedParams q) {
    constexpr int BM = TM * WM * 32, BN = TN * WN * 32, DP = BM + 1;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int khalf = lane >> 5;
    const int wm = wave / WN, wn = wave % WN;

    // the tiles of one split read the same images: contiguous ids, one XCD's L2
    const int id = pix::xcd_tile(blockIdx.x, gridDim.x);
    const int per = q.tiles_i * q.tiles_j * q.c_tiles;
    const int split = id / per, tile = id - split * per;
    const int it = tile % q.tiles_i, jct = tile / q.tiles_i;
    const int jt = jct % q.tiles_j, ct = jct / q.tiles_j;
    const int k0 = it * BM, c0 = ct * q.Ct, cw = min(q.Ct, q.C - c0), cols = q.RS * cw, j0 = jt * BN;
    if (j0 >= cols) return;
    const FastDiv div_c = cw == q.Ct ? q.div_ct : q.div_cl;
    const int r_first = fastdiv(fastdiv(j0, div_c), q.div_s);
    const int r_last = fastdiv(fastdiv(min(j0 + BN, cols) - 1, div_c), q.div_s);

    const int bands = 1 << q.band_shift;
    // Splits take chunks in turn: those that run side by side on an XCD read neighbouring ends of the same lines.
    const int n = split < q.chunks ? ((q.chunks - split + q.splits - 1) / q.splits + 1) / 2 * 2 : 0;      // (the last of an odd number: none)
    if (wave >= WM * WN) {
        const int lt = tid - WM * WN * 64, nr = r_last - r_first + 1;
        if (lt < LOADERS) load_chunks<PL, false, FLAT, FAR, BM>(q, smem, lt, k0, c0, cw, r_first, nr, split, n, q.db_out != nullptr && jct == 0);
        else load_chunks<PL, true, FLAT, FAR, BM>(q, smem, lt - LOADERS, k0, c0, cw, r_first, nr, split, n, false);
        return;
    }

    const int a_lane = (khalf * DP + wm * TM * 32 + (lane & 31)) * 16;
    int b_lane[TN];
#pragma unroll
    for (int b = 0; b < TN; ++b) {
        const int j = min(j0 + wn * TN * 32 + b * 32 + (lane & 31), cols - 1);      // (columns past the last: read, never written)
        const int tap = fastdiv(j, div_c), c = j - tap * cw;
        const int r = fastdiv(tap, q.div_s), s = tap - r * q.S;
        b_lane[b] = q.x_off + (((r - r_first) * q.PW + q.lead + s + khalf * q.sw) * q.CtP + c) * 16;
    }

    constexpr int LM = PL == 3 ? TM : 1, LN = PL == 3 ? TN : 1;
    floatx16 hi[TM][TN], lo[LM][LN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                hi[a][b][e] = 0.0f;
                if (PL == 3) lo[a][b][e] = 0.0f;
            }
    bf16x8 av[PL][TM], bv[PL][TN];
    auto fetch_a = [&](const unsigned char* from, int pl) {
#pragma unroll
        for (int a = 0; a < TM; ++a) av[pl][a] = *reinterpret_cast<const bf16x8*>(from + a_lane + pl * q.d_plane + a * 512);
    };
    auto fetch_b = [&](const unsigned char* from, int pl) {
#pragma unroll
        for (int b = 0; b < TN; ++b) bv[pl][b] = *reinterpret_cast<const bf16x8*>(from + b_lane[b] + pl * q.x_plane);
    };
    auto mul = [&](int i, int j, auto& acc) {
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[i][a], bv[j][b], acc[a][b], 0, 0, 0);
    };
    for (int i = 0; i < n; ++i) {
        meet();
        const Chunk now = chunk_at(q, split + i * q.splits);
        const unsigned char* buf = smem + (i & 1) * q.buf_bytes;
        const int per_row = (now.qn + 1) / 2, steps = now.pr_n * per_row;
        const unsigned char* pa = buf;
        const unsigned char* pb = buf;
        int left = per_row;
        // the next pair of positions (of the last one: the same again)
        auto next = [&](int st) {
            if (st + 1 >= steps) return;
            pa += 2 * DP * 16; pb += 2 * q.sw * q.CtP * 16;
            if (--left == 0) {
                left = per_row;
                pa += (q.QS - 2 * per_row) * DP * 16; pb += (q.sh * q.PW - 2 * per_row * q.sw) * q.CtP * 16;
            }
        };
        if constexpr (PL == 3) {
            // an operand's part is fetched for the next step as soon as its last product is under way
            fetch_a(pa, 1); fetch_b(pb, 1); fetch_a(pa, 0); fetch_b(pb, 0); fetch_b(pb, 2); fetch_a(pa, 2);
#pragma unroll 1
            for (int st = 0; st < steps; ++st) {
                next(st);
                mul(1, 1, lo);
                mul(0, 1, lo);
                mul(1, 0, lo);
                __builtin_amdgcn_sched_barrier(0);
                fetch_a(pa, 1); fetch_b(pb, 1);
                __builtin_amdgcn_sched_barrier(0);
                mul(0, 0, hi);
                mul(0, 2, lo);
                mul(2, 0, lo);
                __builtin_amdgcn_sched_barrier(0);
                fetch_a(pa, 0); fetch_b(pb, 0); fetch_b(pb, 2); fetch_a(pa, 2);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            bf16x8 av2[TM], bv2[TN];
            fetch_a(pa, 0); fetch_b(pb, 0);
#pragma unroll 1
            for (int st = 0; st < steps; st += 2) {
                next(st);
#pragma unroll
                for (int a = 0; a < TM; ++a) av2[a] = *reinterpret_cast<const bf16x8*>(pa + a_lane + a * 512);
#pragma unroll
                for (int b = 0; b < TN; ++b) bv2[b] = *reinterpret_cast<const bf16x8*>(pb + b_lane[b]);
                __builtin_amdgcn_sched_barrier(0);
                mul(0, 0, hi);
                if (st + 1 == steps) break;
                next(st + 1);
                __builtin_amdgcn_sched_barrier(0);
                fetch_a(pa, 0); fetch_b(pb, 0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int a = 0; a < TM; ++a)
#pragma unroll
                    for (int b = 0; b < TN; ++b) hi[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av2[a], bv2[b], hi[a][b], 0, 0, 0);
            }
        }
        // (The sums stay where they are from chunk to chunk: used element by element after the loop, they were copied element by element at the
        // end of every chunk, and 27 of 96 went through memory: 182 MB written beside conv1's 12 MB of partial sums, 254 us instead of 218.)
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b) {
                asm volatile("" : "+v"(hi[a][b]));
                if constexpr (PL == 3) asm volatile("" : "+v"(lo[a][b]));
            }
    }
    meet();

    // infinities and NaNs (also of zero times an x that a position or image without a dy met): again, over the positions that exist
    auto again = [&](int k, int j) {
        float sum = 0.0f;
        auto value = [](const void* t, size_t i) { return PL == 1 ? __uint_as_float((unsigned)((const uint16_t*)t)[i] << 16) : ((const float*)t)[i]; };
        const int tap = fastdiv(j, div_c), c = j - tap * cw, r = fastdiv(tap, q.div_s), s = tap - r * q.S;
        for (int ch = split; ch < q.chunks && sum == sum; ch += q.splits) {
            const Chunk at = chunk_at(q, ch);
            if (FLAT) {
                for (int m = at.q0 * 8; at.pr_n && m < min((at.q0 + at.qn) * 8, q.W); ++m)
                    sum = __builtin_fmaf(value(q.dy, (size_t)at.grp * q.dy_ns + (size_t)k * q.W + m), value(q.x, (size_t)at.grp * q.x_ns + (size_t)(c0 + c) * q.W + m), sum);
                continue;
            }
            for (int m = 0; m < at.pr_n * at.qn; ++m) {
                const int pr = m / at.qn, pc = at.q0 + m - pr * at.qn;
                for (int e = 0; e < 8; ++e) {
                    const int im = at.grp * 8 + e, n = im >> q.band_shift, p = (im & (bands - 1)) * q.PB + at.p0 + pr;
                    if (n >= q.N || p >= q.P) continue;
                    const int h = p * q.sh - q.ph + r, w = pc * q.sw - q.pw + s;
                    const bool inside = (unsigned)h < (unsigned)q.H && (unsigned)w < (unsigned)q.W;
                    const float f = inside ? value(q.x, (size_t)n * q.x_ns + ((size_t)(c0 + c) * q.H + h) * q.W + w) : 0.0f;
                    sum = __builtin_fmaf(value(q.dy, (size_t)n * q.dy_ns + ((size_t)k * q.P + p) * q.Q + pc), f, sum);
                }
            }
        }
        return sum;
    };
    auto place = [&](int k, int j) {
        const int tap = fastdiv(j, div_c), c = j - tap * cw;
        return q.out + ((size_t)split * q.K + k) * q.J + (q.direct ? (c0 + c) * q.RS + tap : ct * q.RS * q.Ct + j);
    };
    constexpr int WORDS = (TM * TN * 16 + 63) / 64;
    unsigned long long bad[WORDS] = {};
#pragma unroll
    for (int b = 0; b < TN; ++b) {
        const int j = j0 + wn * TN * 32 + b * 32 + (lane & 31);
        if (j >= cols) continue;
        float* dst = place(0, j);
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int k = k0 + wm * TM * 32 + a * 32 + (e >> 2) * 8 + khalf * 4 + (e & 3), idx = (a * TN + b) * 16 + e;
                float v = hi[a][b][e];
                if constexpr (PL == 3) v += lo[a][b][e];
                if (k < q.K) {
                    float* d = dst + (size_t)k * q.J;
                    if (__builtin_fabsf(v) <= 3.402823466e38f) {
                        if (PL == 3) v *= JOIN_SCALE;
                        *d = q.direct && q.beta != 0.0f ? *d + v : v;
                    } else bad[idx >> 6] |= 1ull << (idx & 63);
                }
            }
    }
    for (;;) {
        int idx = -1;
#pragma unroll
        for (int w = WORDS - 1; w >= 0; --w) idx = bad[w] ? w * 64 + __ffsll((long long)bad[w]) - 1 : idx;
        if (idx < 0) break;
#pragma unroll
        for (int w = 0; w < WORDS; ++w) bad[w] = idx >> 6 == w ? bad[w] & (bad[w] - 1) : bad[w];
        const int ab = idx >> 4, e = idx & 15;
        const int k = k0 + wm * TM * 32 + (ab / TN) * 32 + (e >> 2) * 8 + khalf * 4 + (e & 3), j = j0 + wn * TN * 32 + (ab % TN) * 32 + (lane & 31);
        const float v = again(k, j);
        float* d = place(k, j);
        *d = q.direct && q.beta != 0.0f ? *d + v : v;
    }
}

template <int PL, bool FLAT, bool FAR, int TM, int TN, int WM, int WN>
hipError_t launch_one(const StagedParams& q, int lds, int splits, hipStream_t st) {
    const long long total = (long long)q.tiles_i * q.tiles_j * q.c_tiles * splits;
    if (total <= 0 || total > 0x7fffffffLL) return hipErrorInvalidValue;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&wgrad_staged_kernel<PL, FLAT, FAR, TM, TN, WM, WN>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
    }
    ProbeScope probe(st);
    (void)hipGetLastError();   // drop stale status left by earlier, unrelated runtime calls
    hipLaunchKernelGGL((wgrad_staged_kernel<PL, FLAT, FAR, TM, TN, WM, WN>), dim3((unsigned)total), dim3(WM * WN * 64 + 2 * LOADERS), lds, st, q);
    return hipGetLastError();
}

struct StagedTile { bool f32; int bm, bn; };
constexpr StagedTile kStagedTiles[] = {{true, 128, 128}, {true, 96, 128}, {true, 64, 256}, {true, 64, 128}, {true, 32, 256}, {true, 32, 128},
                                       {false, 128, 128}, {false, 96, 128}, {false, 64, 256}, {false, 64, 128}, {false, 32, 256}, {false, 32, 128}};
template <bool FAR>
hipError_t by_tile(int dtype, bool flat, const StagedParams& q, int bm, int bn, int lds, int splits, hipStream_t st) {
#define ONE(PL, TM, TN, WM, WN) return flat ? launch_one<PL, true, FAR, TM, TN, WM, WN>(q, lds, splits, st) : launch_one<PL, false, FAR, TM, TN, WM, WN>(q, lds, splits, st)
#define TWO(PL, TM, TN, WM, WN) return launch_one<PL, false, FAR, TM, TN, WM, WN>(q, lds, splits, st)
    if (dtype == PURINE_F32) {
        switch (bm * 1000 + bn) {
            case 128128: ONE(3, 2, 1, 2, 4);
            case 96128:  ONE(3, 3, 1, 1, 4);
            case 64256:  ONE(3, 2, 1, 1, 8);
            case 64128:  ONE(3, 2, 1, 1, 4);
            case 32256:  ONE(3, 1, 2, 1, 4);
            case 32128:  ONE(3, 1, 1, 1, 4);
        }
    } else {
        switch (bm * 1000 + bn) {
            case 128128: TWO(1, 2, 2, 2, 2);
            case 96128:  TWO(1, 3, 1, 1, 4);
            case 64256:  TWO(1, 2, 2, 1, 4);
            case 64128:  TWO(1, 2, 1, 1, 4);
            case 32256:  TWO(1, 1, 2, 1, 4);
            case 32128:  TWO(1, 1, 1, 1, 4);
        }
    }
#undef TWO
#undef ONE
    return hipErrorInvalidValue;
}

}  // namespace

// How the layer would run on this kernel and the time expected for it: tile, channels of a column tile, chunk, splits. Nothing
// comes back that is not expected under budget_us. `limit` (0: none) bounds the partial sums.
WgradStagedPlan plan_wgrad_staged(const ConvGeom& g, int dtype, size_t limit, double budget_us) {
    WgradStagedPlan best{};
    const bool f32 = dtype == PURINE_F32;
    const int es = f32 ? 4 : 2, PL = f32 ? 3 : 1, U = units_of(PL), max_units = LOADERS * U;
    // (by the extents alone: views get the bits of dense tensors, however far apart their images lie)
    const long long xs = (long long)g.N * g.C * g.H * g.W, dys = (long long)g.N * g.K * g.P * g.Q;
    if ((xs + 8) * es >= (1LL << 31) || (dys + 8) * es >= (1LL << 31) || (long long)g.K * g.C * g.R * g.S >= (1LL << 31)) return best;
    const int RS = g.R * g.S;
    const bool flat = RS == 1 && g.sh == 1 && g.sw == 1 && g.ph == 0 && g.pw == 0;
    const int P = flat ? 1 : g.P, Qc = flat ? (int)(((long long)g.P * g.Q + 7) / 8) : g.Q;
    if (flat && !f32) return best;     // (the general kernel is the faster: 93 -> 62 channels at 19x20, N = 14: 12.4 us, 13.6 here)
    // (Planes as they lie in memory, 16 MB and more of them: alone a little faster than the general kernel (96 -> 96 channels at 54x54, N = 64 57 and
    // 51 us), but its workgroups want a CU to themselves, and beside another stream's kernels the two wait for each other: the NIN
    // block of 43 images 593 us with it, 529 without. A plan does not know what runs beside it.)
    if (flat && (long long)g.N * ((long long)g.C * g.H * g.W + (long long)g.K * g.P * g.Q) * 4 >= (16ll << 20)) return best;   // (of views as of dense tensors)
    if (P > (1 << 20) || Qc > (1 << 20) || g.S > 64 || g.sw > 16 || g.sh > 16 || g.ph > 4096 || g.pw > 4096) return best;
    int shift = 0;                     // bands: as many as fill a group of eight, or do not cost more than they bring
    if (!flat)
        while (shift < 3 && (g.N << shift) % 8 != 0 && (g.P >> (shift + 1)) >= 1) ++shift;
    const int lead = flat ? 0 : (4 - g.pw % 4) % 4;
    const double dw_bytes = (double)g.K * g.C * RS * 4.0;
    const int PB = (P + (1 << shift) - 1) >> shift, groups = flat ? g.N : (int)((((long long)g.N << shift) + 7) / 8);
    const double positions = (double)groups * PB * Qc;
    for (const StagedTile& t : kStagedTiles) {
        if (t.f32 != f32 || (staged_wgrad_tile() > 0 && staged_wgrad_tile() != t.bm * 1000 + t.bn)) continue;
        const int tiles_i = (g.K + t.bm - 1) / t.bm;
        // channels of a column tile: all, or as many as make about one tile of columns
        const int most = t.bn / RS > 0 ? t.bn / RS : 1;
        const int c_tiles0 = (long long)RS * g.C <= 4 * t.bn && g.C <= 16 ? 1 : (g.C + most - 1) / most;
        const int Ct = (g.C + c_tiles0 - 1) / c_tiles0, c_tiles = (g.C + Ct - 1) / Ct, tiles_j = (RS * Ct + t.bn - 1) / t.bn, CtP = Ct | 1;
        const long long tiles = (long long)tiles_i * tiles_j * c_tiles;
        if (tiles > 4096) continue;
        // A tile is left out whose positions alone take longer, by the least of the terms below on all CUs all the time, than what is to be
        // beaten: most calls end here, and the search is 1.1 us of the others.
        const double least = f32 ? 0.069 + 0.00129 * (t.bm + Ct) : 0.0155 + 0.00099 * t.bm + 0.00012 * Ct;
        if (!flat && 5.0 + (double)tiles * positions * least / 256.0 >= (best.use ? best.us : budget_us)) continue;
        const unsigned most_splits = tiles < 256 ? 256u / (unsigned)tiles : 1u;
        int nr = 1;                    // filter rows that the columns of a tile span, at most
        if (RS > 1)
            for (int cw = Ct, last = 0; !last; cw = g.C % Ct ? g.C % Ct : Ct, last = 1)
                for (int j0 = 0; j0 < RS * cw; j0 += t.bn) {
                    const int j1 = (j0 + t.bn < RS * cw ? j0 + t.bn : RS * cw) - 1, n = j1 / cw / g.S - j0 / cw / g.S + 1;
                    if (n > nr) nr = n;
                }
        // chunks: the widest that fits LDS and the loaders, then as many rows
        for (int qs = flat ? 8 : 32, last = 0; qs >= (flat ? 8 : 4); qs = qs > 16 ? qs - 8 : qs - 4) {
            int QS = qs;
            if (!flat) {
                const int segs = (Qc + qs - 1) / qs;
                QS = ((Qc + segs - 1) / segs + 3) / 4 * 4;
                if (QS > qs || QS == last) continue;      // (short rows: the same again)
                last = QS;
            }
            const int PW = flat ? 8 : (lead + (QS - 1) * g.sw + g.S + 3) / 4 * 4;
            int PR = 0, XR = 0, lds = 0, units = 0;
            for (int pr = 1; pr <= 8 && pr <= PB; pr *= 2) {
                const int xr = (pr - 1) * g.sh + nr;
                const long long l = 2LL * (PL * ((long long)pr * QS * (t.bm + 1) + (long long)xr * PW * CtP) * 16 + g.sw * CtP * 16);
                const long long du = flat ? t.bm * 2 : (long long)t.bm * pr * QS / 4, xu = flat ? Ct * 2 : (long long)Ct * xr * PW / 4;
                if (l > 160 * 1024 || du > max_units || xu > max_units || xr > 255 || PW > 1020) break;
                PR = pr; XR = xr; lds = (int)l; units = (int)(du + xu);
            }
            if (!PR) continue;
            const long long chunks = (long long)((Qc + QS - 1) / QS) * ((PB + PR - 1) / PR) * groups;
            if (chunks > (1 << 28)) continue;
            // Time of a chunk: its packing, its MFMA steps, and the lines that its loads ask for. Planes as they lie in memory: whole lines,
            // the packing alone. Fitted to 50 layers; of 950 with each fp32 tile nine in ten take 0.76 - 1.37 times the expected time (up
            // to 1.9 below 20 us, where a chunk's chain of loads counts), and the tile chosen is 5 % from the best.
            const double lines = 8.0 * ((double)t.bm * PR * ((QS * es + 63) / 64) + (double)Ct * XR * ((PW * es + 63) / 64 + 0.5));
            const double chunk_us = flat ? 0.006 * units : f32 ? 0.0035 * units + 0.069 * PR * QS + 0.00084 * lines : 1.8 + 0.0155 * PR * QS + 0.00048 * lines;
            if (5.0 + (double)tiles * (double)chunks * chunk_us / 256.0 * 0.999999 >= (best.use ? best.us : budget_us)) continue;
            // one workgroup per CU at a time: one round of the CUs, or one workgroup for each tile where that costs no second pass
            for (int round = 0; round < 2; ++round) {
                unsigned splits = round ? 1 : most_splits;
                if (splits > (unsigned)chunks) splits = (unsigned)chunks;
                const unsigned per = ((unsigned)chunks + splits - 1) / splits;
                splits = ((unsigned)chunks + per - 1) / per;
                if (limit && splits > 1 && splits * (dw_bytes + g.K * 4.0) + 512 > limit) continue;
                double us = 5.0 + (double)((tiles * splits + 255) / 256) * per * chunk_us;
                if (splits > 1) us += 5.0 + 2.0 * splits * dw_bytes / 4e6;
                if (us < (best.use ? best.us : budget_us)) {
                    best.use = true; best.us = us; best.flat = flat;
                    best.bm = t.bm; best.bn = t.bn; best.Ct = Ct; best.tiles_i = tiles_i; best.tiles_j = tiles_j; best.c_tiles = c_tiles;
                    best.band_shift = shift; best.PB = PB; best.PR = PR; best.QS = QS; best.PW = PW; best.XR = XR;
                    best.chunks = (int)chunks; best.splits = (int)splits; best.lds = lds;
                }
            }
        }
    }
    return best;
}

// Partial sums at ws (with one split: dw and db themselves), db's partial rows at db_partial.
hipError_t launch_wgrad_staged(int dtype, const ConvGeom& g, const WgradStagedPlan& k, const void* x, const void* dy, float* dw, float* db, float beta,
                               void* ws, float* db_partial, hipStream_t st) {
    const int es = dtype == PURINE_F32 ? 4 : 2, PL = dtype == PURINE_F32 ? 3 : 1;
    StagedParams q{};
    q.x = x; q.dy = dy;
    q.direct = k.splits == 1; q.beta = beta;
    q.out = q.direct ? dw : (float*)ws;
    q.db_out = q.direct ? db : db ? db_partial : nullptr;
    q.N = g.N; q.C = g.C; q.K = g.K; q.R = g.R; q.S = g.S; q.sh = g.sh; q.sw = g.sw; q.ph = g.ph; q.pw = g.pw;
    q.x_ns = g.x_ns; q.dy_ns = g.y_ns;
    q.H = k.flat ? 1 : g.H; q.W = k.flat ? g.H * g.W : g.W; q.P = k.flat ? 1 : g.P; q.Q = k.flat ? g.P * g.Q : g.Q;
    const int Q = k.flat ? (q.Q + 7) / 8 : q.Q;
    const long long xi = (long long)g.C * g.H * g.W, dyi = (long long)g.K * g.P * g.Q;
    const long long xspan = (g.N - 1) * (long long)g.x_ns + xi, dyspan = (g.N - 1) * (long long)g.y_ns + dyi;
    const bool far = (xspan + 8) * es >= (1LL << 31) || (dyspan + 8) * es >= (1LL << 31);
    q.x_bytes = (unsigned)((far ? xi : xspan) * es); q.dy_bytes = (unsigned)((far ? dyi : dyspan) * es);
    if (!far) { q.x_bytes = (q.x_bytes + 3) & ~3u; q.dy_bytes = (q.dy_bytes + 3) & ~3u; }      // whole dwords (the tensors begin at one)
    q.RS = g.R * g.S; q.J = q.RS * g.C;
    q.Ct = k.Ct; q.CtP = k.Ct | 1;
    q.tiles_i = k.tiles_i; q.tiles_j = k.tiles_j; q.c_tiles = k.c_tiles;
    q.band_shift = k.band_shift; q.PB = k.PB;
    q.Qc = Q; q.PR = k.PR; q.QS = k.QS; q.qsegs = (Q + k.QS - 1) / k.QS; q.pchunks = (k.PB + k.PR - 1) / k.PR; q.chunks = k.chunks; q.splits = k.splits;
    q.PW = k.PW; q.XR = k.XR;
    q.d_plane = k.PR * k.QS * (k.bm + 1) * 16; q.x_off = PL * q.d_plane; q.x_plane = k.XR * k.PW * q.CtP * 16; q.buf_bytes = k.lds / 2;
    const int cl = g.C % k.Ct ? g.C % k.Ct : k.Ct;
    q.lead = (4 - g.pw % 4) % 4; q.dquads = k.QS / 4; q.xquads = k.PW / 4;
    q.div_dquads = make_fastdiv(q.dquads); q.div_pr = make_fastdiv(k.PR); q.div_xquads = make_fastdiv(q.xquads); q.div_xr = make_fastdiv(k.XR);
    q.div_qsegs = make_fastdiv(q.qsegs); q.div_pchunks = make_fastdiv(q.pchunks); q.div_s = make_fastdiv(g.S);
    q.div_ct = make_fastdiv(k.Ct); q.div_cl = make_fastdiv(cl);
    return far ? by_tile<true>(dtype, k.flat, q, k.bm, k.bn, k.lds, k.splits, st) : by_tile<false>(dtype, k.flat, q, k.bm, k.bn, k.lds, k.splits, st);
}

}  // namespace purine

// fp32 weight gradients on the bf16 matrix cores (three exact bf16 parts per operand, six products,
// two accumulator sets: see conv_packets.hip for the arithmetic and its measured error).
//
// dw[k, (tap, c)] = sum over (image, output position) of dy[k, position] * x[c, position shifted by the
// tap]. Bound: MFMA. The MFMA wants 8 consecutive reduction elements per lane. Taking them along a
// row, as NCHW has them, would make every column tap a misaligned window; here they are EIGHT IMAGES
// at one position, so that a tap is a whole number of 16-byte packets away whatever its offset, the
// stride or the padding. Operands are laid out as
//     [plane][group of 8 images][position][channel][8 images]
// with the padding of x written out, so a reduction step (two positions of a group: 16 elements) is
// two contiguous runs of channels per operand and tap, the offsets of a lane never change and a
// step's address is one scalar: the main loop holds no VALU work besides the MFMAs. Batches that
// are not a multiple of 8 are cut into bands of output rows (1, 2, 4 or 8 per image; each band brings
// its own halo rows of x) and the group is 8 bands.
//
// dy is read once for both parameter gradients: the layout pass sums it per channel on the way.
#include "packets.h"
#include "pix_common.h"

namespace purine {
namespace {

using namespace packets;

constexpr int PT = 32, CT = 16, PITCH = CT + 1;     // layout pass: positions x channels of a tile; packets per LDS row

// One tensor of the layout pass.
struct BandPack {
    const float* src; unsigned char* dst;
    float* sums;                     // dy: per (group, position tile) and channel, sum over the tile; or null
    int ch, Hs, Ws, ns;              // channels; source plane; elements between images
    int WD, PD, real;                // band row width; packed positions per group; those that hold data
    int rows_step, ph, pw;           // source row of band row 0 = band * rows_step - ph; column 0 = -pw
    int p_tiles, c_tiles, groups0;   // tiles per group; first group of this launch
    size_t plane;                    // bytes between planes
    FastDiv div_wd, div_ct, div_pt;
    int blocks;
};
struct BandPackPair { BandPack t[2]; int bands, N; };

__global__ __launch_bounds__(256) void pack_bands_kernel(const BandPackPair q) {
    __shared__ __attribute__((aligned(16))) unsigned char tile[PLANES * PT * PITCH * 16];
    const bool second = (int)blockIdx.x >= q.t[0].blocks;
    const BandPack& b = q.t[second ? 1 : 0];
    const int blk = blockIdx.x - (second ? q.t[0].blocks : 0);
    const int rest = fastdiv(blk, b.div_ct), c0 = (blk - rest * b.c_tiles) * CT;
    const int lg = fastdiv(rest, b.div_pt), pt = rest - lg * b.p_tiles;
    const int group = b.groups0 + lg;
    const int tid = threadIdx.x;

    const int pos = pt * PT + (tid & 31);
    const int row = fastdiv(pos, b.div_wd), col = pos - row * b.WD;
    const int w = col - b.pw;
    const bool pos_ok = pos < b.real && (unsigned)w < (unsigned)b.Ws;
    // the eight virtual images of the group: image and source row of this position
    long long off[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int v = group * 8 + e, n = v / q.bands, band = v - n * q.bands;
        const int h = band * b.rows_step - b.ph + row;
        const bool ok = pos_ok && n < q.N && (unsigned)h < (unsigned)b.Hs;
        off[e] = ok ? (long long)n * b.ns + (long long)h * b.Ws + w : -1;
    }
#pragma unroll
    for (int i = 0; i < CT / 8; ++i) {
        const int c = (tid >> 5) + i * 8;
        float v[8];
        float sum = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            v[e] = off[e] >= 0 && c0 + c < b.ch ? b.src[off[e] + (long long)(c0 + c) * b.Hs * b.Ws] : 0.0f;
            sum += v[e];
        }
        store_split8(v, tile + ((tid & 31) * PITCH + c) * 16, PT * PITCH * 16);
        if (b.sums) {
#pragma unroll
            for (int m = 16; m >= 1; m >>= 1) sum += __shfl_xor(sum, m);
            if ((tid & 31) == 0 && c0 + c < b.ch) b.sums[(size_t)(group * b.p_tiles + pt) * b.ch + c0 + c] = sum;
        }
    }
    __syncthreads();
    const int c = tid & (CT - 1);
    if (c0 + c < b.ch) {
#pragma unroll
        for (int pl = 0; pl < PLANES; ++pl)
#pragma unroll
            for (int i = 0; i < PT * CT / 256; ++i) {
                const int j = (tid >> 4) + i * (256 / CT), p = pt * PT + j;
                if (p < b.PD)
                    *reinterpret_cast<bf16x8*>(b.dst + pl * b.plane + ((size_t)((size_t)lg * b.PD + p) * b.ch + c0 + c) * 16) =
                        *reinterpret_cast<const bf16x8*>(tile + ((pl * PT + j) * PITCH + c) * 16);
            }
    }
}

// Second pass: dw[k][c][tap] = beta * dw + the partial sums [split][tap][k][c], added in split order. A
// workgroup owns 64 channels of one row k and all taps: it reads runs of 64 channels and writes one
// contiguous run of dw, through LDS (written element by element as the sums come, at a distance of
// R * S floats, the pass took 18.5 us for 384 x 256 x 9 instead of 12). Workgroups past dw_blocks
// add the bias gradient's rows (some thousand of them on large planes): 8 channels each, 32 row lanes deep,
// in a fixed order.
constexpr int RC = 64, RTAPS = 32, DB_COLS = 8, DB_LANES = 256 / DB_COLS;
__global__ __launch_bounds__(256) void reduce_taps_kernel(const float* __restrict__ partial, float* __restrict__ dw, int splits, float beta,
                                                          int K, int C, int taps, int c_blocks, int dw_blocks,
                                                          const float* __restrict__ db_partial, float* __restrict__ db, int db_rows) {
    __shared__ float buf[RTAPS * (RC + 1)];
    const int c = threadIdx.x & (RC - 1), lane4 = threadIdx.x >> 6;
    if ((int)blockIdx.x >= dw_blocks) {
        const int col = threadIdx.x & (DB_COLS - 1), lane = threadIdx.x / DB_COLS;
        const int k = (blockIdx.x - dw_blocks) * DB_COLS + col;
        float a = 0.0f;
        if (k < K) {
#pragma unroll 8
            for (int r = lane; r < db_rows; r += DB_LANES) a += db_partial[(size_t)r * K + k];
        }
        buf[lane * DB_COLS + col] = a;
        __syncthreads();
        if (lane == 0 && k < K) {
            float t = beta != 0.0f ? db[k] : 0.0f;
#pragma unroll
            for (int l = 0; l < DB_LANES; ++l) t += buf[l * DB_COLS + col];
            db[k] = t;
        }
        return;
    }
    const int k = blockIdx.x / c_blocks, c0 = (blockIdx.x - k * c_blocks) * RC;
    const int nc = min(RC, C - c0);
    const size_t stride = (size_t)taps * K * C;
    for (int t0 = 0; t0 < taps; t0 += RTAPS) {
        const int nt = min(RTAPS, taps - t0);
        if (c < nc)
            for (int t = lane4; t < nt; t += 4) {
                const float* src = partial + ((size_t)(t0 + t) * K + k) * C + c0 + c;
                float a = 0.0f;
#pragma unroll 4
                for (int s = 0; s < splits; ++s) a += src[(size_t)s * stride];
                buf[t * (RC + 1) + c] = a;
            }
        __syncthreads();
        for (int i = threadIdx.x; i < nc * nt; i += 256) {
            const int cc = i / nt, t = i - cc * nt;
            float* dst = dw + ((size_t)k * C + c0 + cc) * taps + t0 + t;
            *dst = beta != 0.0f ? *dst + buf[t * (RC + 1) + cc] : buf[t * (RC + 1) + cc];
        }
        __syncthreads();
    }
}

struct WgradPacketParams {
    const void* dy; const void* x;       // packed operands of groups groups0 ..
    float* out;                          // partial sums [split][tap][K][C]
    unsigned dy_bytes, x_bytes;
    int dy_plane, x_plane;               // bytes between planes
    int K, C, J, S;                      // J = taps * C columns, S filter columns
    int pairs, real, PD, XD;             // steps per group, positions per group (real, padded), x positions per group
    int Q, WB, sh, sw;
    int tiles_i, tiles_j, split0, steps, steps_per_split, groups0;
    int bands, N, P, PB;
    // the fp32 operands, for outputs that are computed again
    const float* dy_src; const float* x_src;
    int dy_ns, x_ns, H, W, ph, pw;
    FastDiv div_pairs, div_q, div_c, div_s;
};

template <int TM, int TN, int WM, int WN>
__global__ __launch_bounds__(WM * WN * 64, 2) void wgrad_packets_kernel(const WgradPacketParams q) {
    typedef Tile<TM, TN, WM, WN> T;
    constexpr int LOADS = T::RA + T::RBL;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char* spare = smem + T::NS * T::STAGE;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int khalf = lane >> 5;
    const int wm = wave / WN, wn = wave % WN;

    // the tiles of one split read the same range of images: contiguous ids, one XCD's L2
    const int id = pix::xcd_tile(blockIdx.x, gridDim.x);
    const int per_split = q.tiles_i * q.tiles_j;
    const int split = q.split0 + id / per_split, tile = id % per_split;
    const int jt = tile / q.tiles_i, it = tile - jt * q.tiles_i;
    const int k0 = it * T::BM, j0 = jt * T::BN;
    const int s0 = split * q.steps_per_split, s1 = min(s0 + q.steps_per_split, q.steps);

    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(q.dy), (short)0, (int)q.dy_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(q.x), (short)0, (int)q.x_bytes, 0x00020000);

    // the lane's part of every load's address: fixed for the whole reduction
    unsigned va[T::RA], vb[T::RBL];
#pragma unroll
    for (int j = 0; j < T::RA; ++j) {
        const int t = j * T::NW + wave, pk = t * 64 + lane;         // packet of the A tile: [plane][half][row]
        const int ph = pk / T::BM, row = pk - ph * T::BM;
        const bool ok = t < T::LA && k0 + row < q.K;
        va[j] = ok ? (unsigned)((ph >> 1) * q.dy_plane + ((ph & 1) * q.K + k0 + row) * 16) : 0x80000000u;
    }
#pragma unroll
    for (int j = 0; j < T::RBL; ++j) {
        const int t = j * T::NW + wave, ph = t / T::PG;             // the load's (plane, half)
        const int col = j0 + (t % T::PG) * 64 + lane;
        const bool ok = t < T::LB && col < q.J;
        const int tap = fastdiv(ok ? col : 0, q.div_c), c = (ok ? col : 0) - tap * q.C;
        const int r = fastdiv(tap, q.div_s), s = tap - r * q.S;
        vb[j] = ok ? (unsigned)((ph >> 1) * q.x_plane + ((r * q.WB + s) * q.C + c) * 16) : 0x80000000u;
    }
    auto request = [&](int st, int slot) {
        const bool exists = st < s1;
        unsigned char* sa = smem + slot * T::STAGE;
        unsigned char* sb = sa + T::A_BYTES;
        // positions m and m + 1 of a group (an odd plane is padded with a zero position of dy, for which
        // x is read at position 0: initialised data, times zero)
        const int sc = exists ? st : s0;
        const int grp = fastdiv(sc, q.div_pairs), m = (sc - grp * q.pairs) * 2, m1 = m + 1 < q.real ? m + 1 : 0;
        const int lg = grp - q.groups0;
        const int p0 = fastdiv(m, q.div_q), p1 = fastdiv(m1, q.div_q);
        const int soff_a = (lg * q.PD + m) * q.K * 16;
        const int soff_b0 = (lg * q.XD + p0 * q.sh * q.WB + (m - p0 * q.Q) * q.sw) * q.C * 16;
        const int soff_b1 = (lg * q.XD + p1 * q.sh * q.WB + (m1 - p1 * q.Q) * q.sw) * q.C * 16;
#pragma unroll
        for (int j = 0; j < T::RA; ++j) {
            const int t = j * T::NW + wave;
            const bool live = T::LA % T::NW == 0 || t < T::LA;
            unsigned v = exists ? va[j] : 0x80000000u;
            asm volatile("" : "+v"(v));        // a select, not a load on either side of a branch
            __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (__attribute__((address_space(3))) void*)(live ? sa + t * 1024 : spare), 16, v, soff_a, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < T::RBL; ++j) {
            const int t = j * T::NW + wave;
            const bool live = T::LB % T::NW == 0 || t < T::LB;
            unsigned v = exists ? vb[j] : 0x80000000u;
            asm volatile("" : "+v"(v));
            const int soff_b = (t / T::PG) & 1 ? soff_b1 : soff_b0;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (__attribute__((address_space(3))) void*)(live ? sb + t * 1024 : spare), 16, v, soff_b, 0, 0);
        }
    };

    floatx16 hi[TM][TN], lo[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) { hi[a][b][e] = 0.0f; lo[a][b][e] = 0.0f; }

#pragma unroll
    for (int k = 0; k < T::NS - 1; ++k) request(s0 + k, k);
    const int a_off = (khalf * T::BM + wm * TM * 32 + (lane & 31)) * 16;
    const int b_off = T::A_BYTES + (khalf * T::BN + wn * TN * 32 + (lane & 31)) * 16;
    int slot = 0;
    for (int st = s0; st < s1; ++st) {
        packets_landed<LOADS * (T::NS - 2)>();
        request(st + T::NS - 1, slot == 0 ? T::NS - 1 : slot - 1);
        multiply_step<T, TM, TN>(smem + slot * T::STAGE, a_off, b_off, hi, lo);
        slot = slot + 1 == T::NS ? 0 : slot + 1;
    }
    // the last requests must not outlive the workgroup's LDS
    __builtin_amdgcn_s_waitcnt(0x0070);

    // infinities and NaNs: again, as plain fp32 sums of the fp32 operands over the positions that exist
    unsigned long long bad = join_sets<TM, TN>(hi, lo);
    if (__builtin_expect(__any(bad != 0), 0)) {
        while (bad) {
            const int idx = __ffsll((long long)bad) - 1;
            bad &= bad - 1;
            const int ab = idx >> 4, e = idx & 15;
            const int k = k0 + wm * TM * 32 + (ab / TN) * 32 + (e >> 2) * 8 + khalf * 4 + (e & 3);
            const int col = j0 + wn * TN * 32 + (ab % TN) * 32 + (lane & 31);
            float sum = 0.0f;
            if (k < q.K && col < q.J) {
                const int tap = fastdiv(col, q.div_c), c = col - tap * q.C;
                const int r = fastdiv(tap, q.div_s), s = tap - r * q.S;
                for (int st = s0; st < s1 && sum == sum; ++st) {
                    const int grp = fastdiv(st, q.div_pairs);
                    for (int half = 0; half < 2; ++half) {
                        const int m = (st - grp * q.pairs) * 2 + half;
                        if (m >= q.real) continue;
                        const int pr = fastdiv(m, q.div_q), pc = m - pr * q.Q;
                        const float* pa = q.dy_src + (size_t)k * q.P * q.Q + pc;
                        const float* pb = q.x_src + (size_t)c * q.H * q.W;
                        const int w = pc * q.sw - q.pw + s;
                        for (int im = 0; im < 8; ++im) {
                            const int v = grp * 8 + im, n = v / q.bands, band = v - n * q.bands, p = band * q.PB + pr;
                            if (n >= q.N || p >= q.P) continue;
                            const int h = p * q.sh - q.ph + r;
                            const bool inside = (unsigned)h < (unsigned)q.H && (unsigned)w < (unsigned)q.W;
                            sum = __builtin_fmaf(pa[(size_t)n * q.dy_ns + (size_t)p * q.Q], inside ? pb[(size_t)n * q.x_ns + (size_t)h * q.W + w] : 0.0f, sum);
                        }
                    }
                }
            }
            replace_element<TM, TN>(hi, idx, sum);
        }
    }
    // partial tile [split][tap][k][c]: lanes along the channels of a tap
    float* __restrict__ out = q.out + (size_t)split * q.K * q.J;
#pragma unroll
    for (int b = 0; b < TN; ++b) {
        const int col = j0 + wn * TN * 32 + b * 32 + (lane & 31);
        if (col >= q.J) continue;
        const int tap = fastdiv(col, q.div_c), c = col - tap * q.C;
        float* dst = out + (size_t)tap * q.K * q.C + c;
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int k = k0 + wm * TM * 32 + a * 32 + (e >> 2) * 8 + khalf * 4 + (e & 3);
                if (k < q.K) dst[(size_t)k * q.C] = hi[a][b][e];
            }
    }
}

template <int TM, int TN, int WM, int WN>
hipError_t launch_main(const WgradPacketParams& q, int splits, hipStream_t st) {
    typedef Tile<TM, TN, WM, WN> T;
    const long long total = (long long)q.tiles_i * q.tiles_j * splits;
    if (total <= 0 || total > 0x7fffffffLL) return hipErrorInvalidValue;
    if (T::LDS > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&wgrad_packets_kernel<TM, TN, WM, WN>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS);
        if (e != hipSuccess) return e;
    }
    (void)hipGetLastError();   // drop stale status left by earlier, unrelated runtime calls
    hipLaunchKernelGGL((wgrad_packets_kernel<TM, TN, WM, WN>), dim3((unsigned)total), dim3(WM * WN * 64), T::LDS, st, q);
    return hipGetLastError();
}

hipError_t by_tile(const WgradPacketParams& q, int bm, int bn, int splits, hipStream_t st) {
#define CALL(TM, TN, WM, WN) launch_main<TM, TN, WM, WN>(q, splits, st)
    PACKET_TILES(CALL)
#undef CALL
}

size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }

// Expected times (us) of the two second passes, less the 2.6 us that either takes at least. reduce_taps_kernel reads
// whole lines only where there are channels enough, and a thread walks ceil(taps / 4) * splits loads one after the other,
// 0.036 us each while the partial sums stay in the L2s and 0.078 beyond; wgrad_reduce_kernel (splits over lanes,
// elements in the partials' order) scatters single floats into dw. Measured, us, taps / lanes: 55 x 3 x 11x11 with 64
// splits 155 / 5, 256 x 48 x 5x5 with 64 40 / 16, 128 x 96 x 3x3 with 16 4.1 / 5.4, 384 x 256 x 3x3 with 1 4.5 / 13.4
// and with 64 34 / 45.
double reduce_taps_us(double dw_bytes, long long splits, int taps) {
    const double bytes = (double)splits * dw_bytes, chain = (bytes < 16e6 ? 0.036 : 0.078) * ((taps + 3) / 4) * (double)splits, mem = bytes / 6e6;
    return chain > mem ? chain : mem;
}
double reduce_lanes_us(double dw_bytes, long long splits) {
    const double scatter = dw_bytes / 4.0 * 1e-5, mem = (double)splits * dw_bytes / ((long long)(dw_bytes / 4.0) % 4 == 0 ? 6e6 : 2.5e6);
    return 2.2 + (scatter > mem ? scatter : mem);
}

}  // namespace

// How the layer would run on this kernel and the time expected for it; `limit` (0: none): the scratch
// of purine_conv_bwd_weight_static, which must be able to hold the partial sums and the packed groups
// that one split reads (it then works through the splits one after the other). No plan comes back that is not
// expected under `budget_us`, and none of those that cannot be is looked at: the search runs on every call (256 <- 96
// channels 5x5, 128 images: 3.9 us of host time without the bounds, 1.3 with them).
WgradPacketPlan plan_wgrad_packets(const ConvGeom& g, size_t limit, double budget_us) {
    WgradPacketPlan best{};
    const long long J = (long long)g.R * g.S * g.C;
    const long long xspan = (long long)(g.N - 1) * g.x_ns + (long long)g.C * g.H * g.W, dyspan = (long long)(g.N - 1) * g.y_ns + (long long)g.K * g.P * g.Q;
    if (J < 32 || g.K < 16 || xspan >= (1LL << 31) || dyspan >= (1LL << 31)) return best;
    for (int bands = 1; bands <= 8; bands *= 2) {
        if (bands > 1 && (g.P < 2 * bands || (long long)g.N * bands > (1 << 24))) break;
        WgradPacketPlan k{};
        k.bands = bands;
        k.PB = (g.P + bands - 1) / bands;
        k.groups = (int)(((long long)g.N * bands + 7) / 8);
        const long long real = (long long)k.PB * g.Q, pd = (real + 1) / 2 * 2;
        const long long wb = (long long)(g.Q - 1) * g.sw + g.S, hb = (long long)(k.PB - 1) * g.sh + g.R;
        if (wb > (1 << 20) || hb > (1 << 20) || real > (1 << 26)) continue;
        const long long dy_group = pd * g.K * 16, x_group = wb * hb * g.C * 16;      // bytes of a plane
        if (dy_group * k.groups * PLANES >= 0x7fffffffLL || x_group * k.groups * PLANES >= 0x7fffffffLL) continue;
        k.real = (int)real; k.PD = (int)pd; k.WB = (int)wb; k.XD = (int)(wb * hb);
        k.pairs = (int)(pd / 2);
        k.dy_group = (size_t)dy_group; k.x_group = (size_t)x_group;
        const long long steps = (long long)k.pairs * k.groups;
        if (steps > (1 << 28)) continue;
        k.steps = (int)steps;
        // (the layout pass works through CT channels at a time, there or not: an image of three costs about three times
        // its bytes)
        const auto dead_lanes = [](int ch) { return 0.5 + 0.5 * (double)((ch + CT - 1) / CT * CT) / (double)ch; };
        const double packed = ((double)dy_group * dead_lanes(g.K) + (double)x_group * dead_lanes(g.C)) * k.groups * PLANES;
        const double pack_us = 5.0 + packed / 6.0 * 10.0 / 4.0e6;
        const double dw_bytes = (double)g.K * J * 4.0;
        const double least_us = pack_us + 10.0 + 2.0 * dw_bytes / 5e6;       // whatever the tile and the splits
        for (const PacketTile& t : kTiles) {
            const long long ti = (g.K + t.bm - 1) / t.bm, tj = (J + t.bn - 1) / t.bn, tiles = ti * tj;
            // (no split shares the multiplication out better than evenly)
            if (least_us + (double)tiles * steps * t.cycles / t.eff_w / (256.0 * 2.2e3) >= (best.use ? best.us : budget_us)) continue;
            // split counts that fill the chip to 1/2, 1, 3/2 .. 6 workgroups per CU
            const int all = (int)steps, few = tiles < 2048 ? (int)tiles : 2048;
            int last = -1;
            for (int half_fill = 1; half_fill <= 12; ++half_fill) {
                int sp = half_fill * 128 / few;
                if (sp < 1) sp = 1;
                if (sp > 512) sp = 512;
                const int per = (all + sp - 1) / sp;
                if (per == last) continue;
                last = per;
                sp = (all + per - 1) / per;
                if (sp > 1 && sp * dw_bytes > 256.0 * (1 << 20)) break;
                const double part_us = sp * dw_bytes / 5e6;                        // the partial sums written
                const double x = (double)tiles * sp / 256.0;
                const double load = x <= 1.0 ? 1.45 : 0.5 * (x + (double)((tiles * sp + 255) / 256));
                double us = load * ((double)per * t.cycles / t.eff_w + 5000.0) / 2.2e3 + 4.0 + pack_us + 6.0 + part_us;
                if (us + part_us >= (best.use ? best.us : budget_us)) continue;
                const double taps_us = reduce_taps_us(dw_bytes, sp, g.R * g.S), lanes_us = reduce_lanes_us(dw_bytes, sp);
                const bool lanes = lanes_us < taps_us;
                const double red = lanes ? lanes_us : taps_us;
                us += red > part_us ? red : part_us;
                // groups that one split touches at most
                const int span = (per + k.pairs - 2) / k.pairs + 1;
                const size_t one = up256((size_t)(sp * dw_bytes)) + up256((size_t)((span < k.groups ? span : k.groups) * dy_group * PLANES)) +
                                   up256((size_t)((span < k.groups ? span : k.groups) * x_group * PLANES));
                if (limit && one > limit) continue;
                if (us < (best.use ? best.us : budget_us)) {
                    k.use = true; k.us = us;
                    k.bm = t.bm; k.bn = t.bn; k.tiles_i = (int)ti; k.tiles_j = (int)tj;
                    k.splits = (int)sp; k.steps_per_split = (int)per; k.reduce_lanes = lanes;
                    best = k;
                }
            }
        }
    }
    if (!best.use) return best;
    best.db_rows = best.groups * ((best.PD + PT - 1) / PT);
    best.part_bytes = up256((size_t)best.splits * g.K * J * 4);
    best.ws_bytes = best.part_bytes + up256(best.dy_group * best.groups * PLANES) + up256(best.x_group * best.groups * PLANES);
    // Scratch is asked for in whole copies of dw, and a row of K sums per copy for the fused bias gradient,
    // as for the general kernels; the packed operands and the bias sums of the layout pass take up as
    // many of the copies as they need.
    const size_t dw_bytes = (size_t)g.K * J * 4;
    best.db_offset = best.ws_bytes;
    best.copies = (best.ws_bytes + up256((size_t)best.db_rows * g.K * 4) + dw_bytes - 1) / dw_bytes;
    return best;
}

// Partial sums [split][tap][K][C] at ws, packed operands behind them, then (db != null: the whole scratch
// is there) the bias sums per (group, position tile) and channel. ws_bytes below k.ws_bytes: the splits are taken a few at a time, as
// many as the scratch holds the groups of.
hipError_t launch_wgrad_packets(const ConvGeom& g, const WgradPacketPlan& k, const void* x, const void* dy, float* dw, float* db, float beta, void* ws,
                                size_t ws_bytes, hipStream_t st) {
    ProbeScope whole_op(st);             // layout pass, products, second pass
    unsigned char* base = (unsigned char*)ws;
    float* db_sums = db ? (float*)(base + k.db_offset) : nullptr;
    WgradPacketParams q{};
    q.out = (float*)ws;
    q.K = g.K; q.C = g.C; q.J = g.R * g.S * g.C; q.S = g.S;
    q.pairs = k.pairs; q.real = k.real; q.PD = k.PD; q.XD = k.XD; q.Q = g.Q; q.WB = k.WB; q.sh = g.sh; q.sw = g.sw;
    q.tiles_i = k.tiles_i; q.tiles_j = k.tiles_j; q.steps = k.steps; q.steps_per_split = k.steps_per_split;
    q.bands = k.bands; q.N = g.N; q.P = g.P; q.PB = k.PB;
    q.dy_src = (const float*)dy; q.x_src = (const float*)x; q.dy_ns = g.y_ns; q.x_ns = g.x_ns; q.H = g.H; q.W = g.W; q.ph = g.ph; q.pw = g.pw;
    q.div_pairs = make_fastdiv(k.pairs); q.div_q = make_fastdiv(g.Q); q.div_c = make_fastdiv(g.C); q.div_s = make_fastdiv(g.S);

    BandPackPair b{};
    b.bands = k.bands; b.N = g.N;
    BandPack& d = b.t[0];
    d.src = (const float*)dy; d.sums = db_sums; d.ch = g.K; d.Hs = g.P; d.Ws = g.Q; d.ns = g.y_ns;
    d.WD = g.Q; d.PD = k.PD; d.real = k.real; d.rows_step = k.PB; d.ph = 0; d.pw = 0;
    BandPack& v = b.t[1];
    v.src = (const float*)x; v.sums = nullptr; v.ch = g.C; v.Hs = g.H; v.Ws = g.W; v.ns = g.x_ns;
    v.WD = k.WB; v.PD = k.XD; v.real = k.XD; v.rows_step = k.PB * g.sh; v.ph = g.ph; v.pw = g.pw;
    for (int i = 0; i < 2; ++i) {
        BandPack& t = b.t[i];
        t.p_tiles = (t.PD + PT - 1) / PT; t.c_tiles = (t.ch + CT - 1) / CT;
        t.div_wd = make_fastdiv(t.WD); t.div_ct = make_fastdiv(t.c_tiles); t.div_pt = make_fastdiv(t.p_tiles);
    }
    for (int split = 0; split < k.splits;) {
        const int g0 = split * k.steps_per_split / k.pairs;
        int end = k.splits, g1 = k.groups;
        if (ws_bytes < k.ws_bytes) {
            for (end = split + 1;; ++end) {
                const long long next_step = (long long)(end + 1) * k.steps_per_split;       // one past the steps of `end`, if it were taken too
                const int ng1 = end >= k.splits ? 0 : (int)(((next_step < k.steps ? next_step : k.steps) + k.pairs - 1) / k.pairs);
                if (end >= k.splits || k.part_bytes + up256((size_t)(ng1 - g0) * k.dy_group * PLANES) + up256((size_t)(ng1 - g0) * k.x_group * PLANES) > ws_bytes) break;
            }
            const long long last = (long long)end * k.steps_per_split;
            g1 = (int)(((last < k.steps ? last : k.steps) + k.pairs - 1) / k.pairs);
        }
        const size_t dyb = (size_t)(g1 - g0) * k.dy_group, xb = (size_t)(g1 - g0) * k.x_group;      // bytes of a plane
        unsigned char* pdy = base + k.part_bytes;
        unsigned char* px = pdy + up256(dyb * PLANES);
        if (px + xb * PLANES > base + ws_bytes) return hipErrorInvalidValue;
        d.dst = pdy; d.plane = dyb; v.dst = px; v.plane = xb;
        long long blocks = 0;
        for (int i = 0; i < 2; ++i) {
            BandPack& t = b.t[i];
            const long long nb = (long long)(g1 - g0) * t.p_tiles * t.c_tiles;
            t.groups0 = g0; t.blocks = (int)nb;
            blocks += nb;
        }
        if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
        (void)hipGetLastError();
        hipLaunchKernelGGL(pack_bands_kernel, dim3((unsigned)blocks), dim3(256), 0, st, b);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        q.dy = pdy; q.x = px; q.dy_plane = (int)dyb; q.x_plane = (int)xb;
        q.dy_bytes = (unsigned)(dyb * PLANES); q.x_bytes = (unsigned)(xb * PLANES);
        q.split0 = split; q.groups0 = g0;
        e = by_tile(q, k.bm, k.bn, end - split, st);
        if (e != hipSuccess) return e;
        split = end;
    }
    if (k.reduce_lanes)
        return launch_wgrad_reduce((const float*)ws, dw, k.splits, beta, true, g.K, g.C, g.R * g.S, (const float*)db_sums, db, k.db_rows, st);
    const int c_blocks = (g.C + RC - 1) / RC, db_blocks = db ? (g.K + DB_COLS - 1) / DB_COLS : 0;
    const long long dw_blocks = (long long)g.K * c_blocks;
    if (dw_blocks + db_blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(reduce_taps_kernel, dim3((unsigned)(dw_blocks + db_blocks)), dim3(256), 0, st, (const float*)ws, dw, k.splits, beta, g.K, g.C,
                       g.R * g.S, c_blocks, (int)dw_blocks, (const float*)db_sums, db, k.db_rows);
    return hipGetLastError();
}

}  // namespace purine

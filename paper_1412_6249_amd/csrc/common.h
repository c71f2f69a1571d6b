// Internal declarations shared by the host entry points and the gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "purine.h"

namespace purine {

// Division of 0 <= n < 2^31 by a divisor fixed on the host, done with one high multiply, one masked
// add and a shift, with no branch (round-up reciprocal: m = ceil(2^(32+s)/d) with
// s = ceil(log2 d) - 1 fits 32 bits, and the error term n*e/2^(32+s) stays below 1/d for every
// n < 2^31; d = 1 has no such m, so it takes q = (0 + n) >> 0 through the add mask).
struct FastDiv {
    uint32_t m, s, add;
};

inline FastDiv make_fastdiv(uint32_t d) {
    FastDiv f{0u, 0u, 0xffffffffu};
    if (d <= 1) return f;
    uint32_t l = 0;
    while ((1ull << l) < d) ++l;           // l = ceil(log2 d) >= 1
    f.s = l - 1;
    f.add = 0u;
    const unsigned __int128 one = 1;
    const unsigned __int128 num = one << (32 + f.s);
    f.m = (uint32_t)((num + d - 1) / d);
    return f;
}

__host__ __device__ inline uint32_t fastdiv(uint32_t n, const FastDiv& f) {
#if defined(__HIP_DEVICE_COMPILE__)
    return (__umulhi(n, f.m) + (n & f.add)) >> f.s;
#else
    return ((uint32_t)(((uint64_t)n * f.m) >> 32) + (n & f.add)) >> f.s;
#endif
}

// Problem description of the weight-gradient implicit GEMM:
//   partial[split][k][(c,r,s)] = sum over pixels (n,p,q) of the split of dy[n,k,p,q] * x[n,c,p*sh-ph+r,q*sw-pw+s]
struct WgradParams {
    const void* x;
    const void* dy;
    float* out;        // partial sums [splits][K][CRS], or dw itself when splits == 1 and beta == 0
    int N, C, H, W, K, P, Q, R, S, sh, sw, ph, pw;
    int PQ, M, CRS, RS, HW;
    FastDiv div_pq, div_q, div_rs, div_s;
    int chunk;         // pixels per split, a multiple of the slab depth
    int tiles_i, tiles_j, splits;
    int c_tiles;       // per-tap column mode: channel tiles per tap (tiles_j = R*S*c_tiles)
    int x_ns, dy_ns;   // elements between consecutive images of x and of dy
    unsigned x_bytes, dy_bytes;   // tensor spans when the kernels may read them as raw buffers, else 0
    float* db_out;     // fused bias gradient: partial sums [splits][K], or null
};


struct ConvGeom {
    int N, C, H, W, K, R, S, P, Q, sh, sw, ph, pw;
    // elements between consecutive images of the x-shaped tensors (x, dx, the ReLU mask of dx) and
    // of the y-shaped ones (y, dy): C*H*W and K*P*Q unless the tensor is a channel-slice view
    int x_ns, y_ns;
};

// Part of the plan below: the fp32 kernel on packed bf16 parts (conv_packets.hip).
struct PacketPlan {
    bool use;
    int bm, bn, tiles_i, tiles_pix;
    int steps, splits, steps_per_split;    // reduction steps (16 channels of one tap each), split over workgroups
    int Cb;                                // packed channel groups of 8 per image
    size_t a_bytes, b_offset, b_bytes, part_offset, ws_bytes;   // scratch: filter, activations, partial outputs
    double us;                             // expected time
};

// ... and the one that splits a patch of the gathered tensor in LDS (conv_patch_f32.hip).
struct PatchF32Plan {
    bool use, split;            // split: bf16 parts; else fp32 products in the tap kernel's order
    int bm, tiles_i, tiles_pix;
    int bands, Wb, PW;          // images are cut into bands of Wb columns; patch rows of PW positions
    int cgs;                    // groups of 16 gathered channels
    int full, parts, cg_part;   // tiles past the first `full` are summed by `parts` workgroups of cg_part groups each
    size_t a_bytes, part_offset, part_bytes;
    double us;
};

// ... and bf16 layers whose patch is staged in LDS whatever the width of its rows (conv_patch_any_bf16.hip).
struct PatchAnyPlan {
    bool use;
    int bm, bn, tiles_i, tiles_pix;
    int taps, cgs;                   // groups of 16 gathered channels
    int stage_taps, stages;          // taps per filter stage, stages per group
    int pw, h_base, w_base;          // patch columns; input row / column of patch position 0
    int c0, ncol, quads, rounds;     // input columns loaded, in fours; loads per thread
    int plane_bytes, lds;
    int rt;                          // square filter with a kernel of its own: its side, else 0
    bool ahead;                      // ... whose filter and patch are requested several groups ahead
    size_t a_bytes;
    double us;
};

// ... and fp32 1x1 layers on bf16 parts split in registers (conv_gemm1x1_split.hip).
struct Split1x1Plan {
    bool use;
    int tm, tiles_i, cgs;        // row tiles of 32 * tm; groups of 16 gathered channels
    int strips, groups, waves;   // strips of 32 pixels; workgroups per row tile, wavefronts of each that take strips
};

// Plan of the streaming fp32 GEMM on bf16 parts (gemm_stream_f32.hip): rows x columns of the output over a
// reduction, split over workgroups where scratch for partial outputs is at hand.
struct StreamPlan {
    bool use;
    int bm, tiles_i, tiles_pix, steps, splits, steps_per_split;
    size_t part_bytes;          // partial outputs (0 without a split)
    double us;                  // expected time
};
namespace pix {
StreamPlan plan_stream(long long rows, long long cols, long long K, bool a_in, bool b_in);
PacketPlan plan_packets_matrix(long long rows, long long cols, long long K);
hipError_t launch_packets_matrix(const PacketPlan& k, const void* a, const void* b, void* out, float beta, long long rows, long long cols, long long K,
                                 void* ws, hipStream_t st);
hipError_t launch_stream_gemm(const StreamPlan& k, const void* a, bool a_in, const void* b, bool b_in, void* out, const void* bias, float beta,
                              long long rows, long long cols, long long K, void* ws, hipStream_t st);
}

// Launch plan of the forward / backward-data implicit GEMM: same answer for the workspace query and
// for the launch.
struct PixPlan {
    int mode;          // 0 forward, 1 backward-data with unit stride, 2 backward-data phase-folded
    bool flat;         // forward with fewer than 16 input channels: flattened (c,r,s) reduction, no scratch
    int bm, bn, tiles_i, tiles_pix;
    int Co, Ci;        // GEMM rows and gathered channels
    int Rt, St;        // taps of the reduction
    int Ci_pad, i_pad; // extents of the repacked filter A[Rt*St][Ci_pad][i_pad]
    size_t ws_bytes;   // scratch: repacked filter, then (bf16 tap kernels) the channels-blocked input copy
    size_t blk_offset; // byte offset of that copy inside the scratch (0: none)
    bool patch;        // bf16: the kernel that stages the input patch in LDS runs (no blocked copy)
    // 1x1 / stride 1 / unpadded layers: streaming GEMM kernel (used when the pointers are aligned
    // to gemm_tn elements; the fields above stay valid for the general kernel otherwise)
    bool gemm1x1;
    int gemm_tm, gemm_tn, gemm_tiles_i, gemm_tiles_pix;
    // ... with a split reduction when its tiles alone would leave most of the chip idle (the
    // fully-connected backward-data shape: few rows, few pixels, a long reduction)
    int gemm_splits, gemm_split_ci;
    size_t gemm_part_offset;   // byte offset of the fp32 partial tiles inside the scratch
    PacketPlan pk;
    PatchF32Plan pf;
    PatchAnyPlan pa;
    Split1x1Plan ps;
    double us;                 // expected time of the general fp32 kernels
    bool direct;               // ... but a launch as small as this runs conv_direct.hip's kernel (the scratch stays as it is)
};
PixPlan plan_conv_pix(const ConvGeom& g, bool bwd_data, int dtype, bool fused, bool accumulate = false);
void force_pix_tile(int bm, int bn);
bool patch_any_forced();             // test hook: (-9, tile): bf16 layers run the patch kernel for rows of any width, with that tile (bm * 1000 + bn) or its own
bool split_1x1_forced();             // test hook: (-10, row tiles of 32, or 0): fp32 1x1 layers run the kernel on parts split in registers
bool split_patch_forced();           // test hook: (-6, parts): fp32 layers run the kernel that splits a patch in LDS wherever it applies (parts > 1: each last tile's channels over as many workgroups)
bool split_packets_forced();         // test hook: (-7, anything): ... the kernels on packed bf16 parts (forward, backward-data, weight gradient)
bool staged_wgrad_forced();          // test hook: (-11, tile): weight gradients run the kernel that lays its operands out in LDS, with that tile (bm * 1000 + bn) or its own
int staged_wgrad_tile();
bool direct_forced();                // test hook: (-12, anything): forward, backward-data and fully-connected passes run the kernels of small launches wherever they apply
bool small_kernels_disabled();       // test hook: (-13, anything): nothing runs them, the weight gradient inside LDS or the second pass of few splits
bool patch_split_roles_forced();     // test hook: (-5, anything) gives it layers of few tiles too
bool patch_split_roles_disabled();   // tuning hook: (-4, anything) keeps the bf16 patch kernel on its one-role form
bool buffer_loads_disabled();   // tuning hook: (anything, -1) given to force_pix_tile

// Split of the pixel reduction of the weight gradient: same answer for the workspace query and
// for the launch.
// Part of the plan below: the fp32 kernel on packed bf16 parts (conv_wgrad_packets.hip).
struct WgradPacketPlan {
    bool use;
    int bands, PB, groups;                 // bands of PB output rows per image; groups of 8 bands
    int real, PD, pairs, WB, XD;           // output positions of a band, padded to whole pairs; x positions (rows of WB)
    int bm, bn, tiles_i, tiles_j, steps, splits, steps_per_split;
    int db_rows;                           // rows of the bias gradient's partial sums
    bool reduce_lanes;                     // second pass: wgrad_reduce_kernel, splits over lanes (few channels, many splits)
    size_t dy_group, x_group;              // bytes of a packed group and plane
    size_t part_bytes, ws_bytes;           // scratch: partial sums of dw, then the packed operands,
    size_t db_offset, copies;              // then the bias sums; all of it in whole copies of dw
    double us;                             // expected time
};
WgradPacketPlan plan_wgrad_packets(const ConvGeom& g, size_t limit, double budget_us);
hipError_t launch_wgrad_packets(const ConvGeom& g, const WgradPacketPlan& k, const void* x, const void* dy, float* dw, float* db, float beta, void* ws,
                                size_t ws_bytes, hipStream_t st);
// ... and the kernel that lays its operands out inside LDS (conv_wgrad_staged.hip).
struct WgradStagedPlan {
    bool use;
    int bm, bn, Ct, tiles_i, tiles_j, c_tiles;   // tile; channels of a channel tile; row tiles, column tiles of a channel tile, channel tiles
    bool flat;                             // 1x1 layers as they lie in memory: one row per image
    int band_shift, PB, PR, QS, PW, XR;    // bands per image (log2) and their output rows; chunk of PR x QS positions, its patch
    int chunks, splits, lds;
    double us;                             // expected time
};
WgradStagedPlan plan_wgrad_staged(const ConvGeom& g, int dtype, size_t limit, double budget_us);
hipError_t launch_wgrad_staged(int dtype, const ConvGeom& g, const WgradStagedPlan& k, const void* x, const void* dy, float* dw, float* db, float beta,
                               void* ws, float* db_partial, hipStream_t st);
// Second pass of a split weight gradient: partial sums [split][k][c][tap], [split][tap][k][c] (tap_major) or
// [split][k][channel tile][tap][c] (tile > 0: its channels), into dw, and db_rows rows of K sums into db (db may be null). Reads in the partials' own order.
// finish (a layer of one tap): the product goes to a bf16 matrix y [K][C], rounded once after its column's bias (may be null) is added
struct WgradFinish { const uint16_t* bias; uint16_t* y; };
hipError_t launch_wgrad_reduce(const float* partial, float* dw, int splits, float beta, bool tap_major, int K, int C, int RS,
                               const float* db_partial, float* db, int db_rows, hipStream_t st, int tile = 0, const WgradFinish* finish = nullptr);
// scratch of purine_conv_bwd_weight_static
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;

struct WgradPlan {
    WgradPacketPlan pk;
    WgradStagedPlan sg;
    size_t static_bytes;  // what the layer has to fit into kStaticScratchBytes with: the general kernels' partial sums
    bool rows;         // bf16 3x3 layers: the row-staging kernel (one partial tile per persistent workgroup)
    bool cols;         // bf16 layers with C*R*S <= 160: whole-filter tiles per wavefront (conv_wgrad_cols_bf16.hip)
    bool taps;         // bf16 layers with C*R <= 32 and a known filter row shape: one tile per column tap (conv_wgrad_taps_bf16.hip)
    bool tap;          // columns are the channels of one tap (C >= 64) instead of flattened (c,r,s)
    int c_tiles;
    int bm, bn;        // tile extents along k and along the columns
    int tiles_i, tiles_j, splits, chunk;
    size_t ws_bytes;      // weight-gradient partials
    size_t db_ws_bytes;   // bias-gradient partials of the fused operator, placed behind them
};
WgradPlan plan_wgrad(const ConvGeom& g, int dtype);
bool wgrad_rows_bf16_applies(const ConvGeom& g, int* workers);
hipError_t launch_wgrad_rows_bf16(const ConvGeom& g, int workers, const void* x, const void* dy, float* partials,
                                  float* db_partials, hipStream_t st);
bool wgrad_taps_bf16_applies(const ConvGeom& g, int* workers);
hipError_t launch_wgrad_taps_bf16(const ConvGeom& g, const void* x, const void* dy, float* partials,
                                  float* db_partials, hipStream_t st);
bool wgrad_cols_bf16_applies(const ConvGeom& g, int* workers);
hipError_t launch_wgrad_cols_bf16(const ConvGeom& g, const void* x, const void* dy, float* partials,
                                  float* db_partials, hipStream_t st);
inline size_t wgrad_db_offset(const WgradPlan& pl) { return (pl.ws_bytes + 255) & ~(size_t)255; }

struct BiasBwdPlan {
    int parts;         // image groups per channel
    int imgs_per_part;
    size_t ws_bytes;
};
BiasBwdPlan plan_bias_bwd(int N, int K, int PQ);

// Maps a HIP status to a purine status and remembers the HIP error for purine_last_hip_error().
int hip_status(hipError_t e);

// One-shot event pair that brackets the main kernel of the next operator call of this host thread.
struct KernelProbe { hipEvent_t start, stop; };
KernelProbe take_kernel_probe();   // returns the pending pair (or NULLs) and clears it
struct ProbeScope {                 // records start on construction and stop on destruction
    KernelProbe p; hipStream_t st;
    explicit ProbeScope(hipStream_t s) : p(take_kernel_probe()), st(s) { if (p.start) (void)hipEventRecord(p.start, st); }
    // armed = false: an inert scope (the pending pair is left for an inner scope to take)
    ProbeScope(hipStream_t s, bool armed) : p(armed ? take_kernel_probe() : KernelProbe{nullptr, nullptr}), st(s) {
        if (p.start) (void)hipEventRecord(p.start, st);
    }
    ~ProbeScope() { if (p.stop) (void)hipEventRecord(p.stop, st); }
};

// Kernel launchers (defined in the .hip files). Each returns a hipError_t from the launch.
// Optional fused epilogue of the forward / backward-data kernels.
struct PixEpilogue {
    const void* bias = nullptr;   // forward: y = conv + bias[k]
    int relu = 0;                 // forward: y = max(y, 0)
    const void* mask = nullptr;   // backward-data: dx = mask > 0 ? dx : 0 (mask has dx's extents)
};
// forward / backward-data of small launches in one kernel without scratch (conv_direct.hip)
double conv_direct_us(const ConvGeom& g, bool bwd, int dtype);
hipError_t launch_conv_direct(int dtype, const ConvGeom& g, bool bwd, const void* in, const void* wt, void* out, float beta, const PixEpilogue& epi, hipStream_t st);
hipError_t launch_conv_pix(int dtype, const ConvGeom& g, const PixPlan& plan, const void* in,
                           const void* wt, void* out, float beta, void* ws, const PixEpilogue& epi,
                           hipStream_t st);
// db != null: also db = beta*db + sum of dy over pixels (fused BiasBwd), scratch behind dw's partials
hipError_t launch_conv_wgrad(int dtype, const ConvGeom& g, const WgradPlan& plan, const void* x,
                             const void* dy, float* dw, float* db, float beta, void* ws, size_t ws_bytes, hipStream_t st, const WgradFinish* finish = nullptr);
hipError_t launch_bias_fwd(int dtype, const void* b, void* y, int N, int K, int PQ, hipStream_t st);
hipError_t launch_bias_bwd(int dtype, const void* dy, float* db, float beta, int N, int K, int PQ,
                           const BiasBwdPlan& plan, void* ws, hipStream_t st);
hipError_t launch_relu_fwd(int dtype, const void* x, void* y, int64_t n, hipStream_t st);
hipError_t launch_relu_bwd(int dtype, const void* x, const void* dy, void* dx, int64_t n,
                           hipStream_t st);
hipError_t launch_bias_rows(const float* b, float* y, int N, int K, hipStream_t st);
// bf16 fully-connected data gradient: scratch bytes and slicing (SIZE_MAX: rows are not whole
// 16-byte packets, the kernel does not apply)
size_t fc_dgrad_bf16_plan(int64_t N, int64_t C, int64_t K, int* slices, int* k_per_slice);
hipError_t launch_fc_dgrad_bf16(const void* dy, const void* w, void* dx, int N, int K, int C, void* ws, hipStream_t st);
// db[k] = beta*db[k] + sum_n dy[n][k] for a dense [N][K] matrix (fixed summation order)
hipError_t launch_fc_bias_bwd(int dtype, const void* dy, float* db, int N, int K, float beta, hipStream_t st);
// out0 = in0^T and out1 = in1^T for dense 2-byte matrices of `rows` x cols0 / cols1 elements, one launch
hipError_t launch_transpose16_pair(const void* in0, void* out0, int cols0, const void* in1, void* out1, int cols1, int rows,
                                   hipStream_t st);
// bf16 fully-connected weight gradient on the transposed matrices (batches of a multiple of 8 samples)
bool fc_wgrad_bf16_applies(int64_t N, int64_t C, int64_t K);
hipError_t launch_fc_wgrad_bf16(const void* dyT, const void* xT, float* dw, int N, int K, int C, bool accumulate,
                                hipStream_t st);
// fully-connected passes in one launch without scratch (fc_direct.hip); db: the weight gradient's bias gradient
bool fc_direct_faster(int pass, int64_t N, int64_t C, int64_t K, int dtype, bool other_splits);
hipError_t launch_fc_direct(int pass, int dtype, const void* a, const void* b, void* out, const void* bias, float* db, float beta, int64_t N, int64_t C,
                            int64_t K, hipStream_t st);
hipError_t launch_relu_view(int dtype, bool bwd, const void* x, const void* dy, void* out, int N, int run,
                            int64_t x_ns, int64_t dy_ns, int64_t out_ns, hipStream_t st);
hipError_t launch_sgd_update(int dtype, const void* w, const float* dw, void* new_w, float lr,
                             int64_t n, hipStream_t st);
hipError_t launch_maxpool_fwd(int dtype, const void* x, void* y, int32_t* arg, int NC, int H, int W,
                              int P, int Q, int k, int stride, int pad, hipStream_t st);
hipError_t launch_maxpool_bwd(int dtype, const void* dy, const int32_t* arg, void* dx, const void* y, float beta,
                              int NC, int H, int W, int P, int Q, int k, int stride, int pad,
                              hipStream_t st);
hipError_t launch_copy_channels(int dtype, const void* src, void* dst, int N, int c_count,
                                int src_C, int src_c0, int dst_C, int dst_c0, int HW,
                                hipStream_t st);
hipError_t launch_sum(int dtype, const void* const* terms, int n_terms, void* out, int64_t n,
                      hipStream_t st);

}  // namespace purine

// launch.hpp -- host-side interface between the C-ABI shim and the kernel
// translation units.  Plain structs only; every launcher queues work on the
// given stream and returns the launch status.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.hpp"
#include "nnconv.h"

namespace nnconv {

constexpr int MAX_TAPS = 64;

// Filter taps visited by one implicit-GEMM launch.  Tap t moves the A-image
// read position by (dh[t], dw[t]) and starts at element boff[t] of a B row.
struct TapTable {
    int32_t n;
    int32_t dh[MAX_TAPS];
    int32_t dw[MAX_TAPS];
    int32_t boff[MAX_TAPS];
};

// One implicit GEMM  out[row, col] = alpha * sum_{tap, ch} A(row, tap, ch) * B[col, tap, ch]
// with channel-last operands, used for the forward pass (A = x, B = w) and
// for one stride phase of the backward-data pass (A = dy, B = w transposed
// to [R][S][Cg][Kg] per group).
//
// Row m decodes to (image n, i, j) with i < mi, j < mj.  A is read at pixel
// (i*ai_mul + ai_add + dh[t], j*aj_mul + aj_add + dw[t]) of image n (zero
// outside a_h x a_w), channels g*a_cg_ofs + ch.  B row `col` of group g
// starts at element g*b_g_ofs + col*b_ld.  The result goes to pixel
// (i*oi_mul + oi_add, j*oj_mul + oj_add) of an o_h x o_w image with o_c
// channels, channel g*o_cg_ofs + col.
// One output phase of a 64-channel-slice launch: rows m < M decode to
// (image n, i < mi, j < mj); the output pixel is (i*oi_mul + oi_add,
// j*oj_mul + oj_add); the phase uses taps [tap_start, tap_start + tap_count)
// of the tap table.  The forward pass has one phase; backward-data has one per
// stride phase, all in a single launch.
struct TNPhase {
    int32_t M, mi, mj;
    FastDiv div_mj, div_mi;
    int32_t oi_add, oj_add;
    int32_t tap_start, tap_count;
    int32_t tiles_m, block_start;  // filled by the launcher
};
constexpr int MAX_PHASES = 16;  // strides up to 4

struct TNParams {
    const void *a;
    uint32_t a_bytes;
    const void *b;
    uint32_t b_bytes;
    void *out;
    uint32_t o_bytes;     // size of the output tensor in bytes
    int32_t M;
    int32_t mi, mj;
    FastDiv div_mj, div_mi;
    int32_t a_h, a_w, a_c, a_cg_ofs;
    int32_t ai_mul, ai_add, aj_mul, aj_add;
    int32_t cr;            // reduction channels per tap (multiple of 8)
    FastDiv div_crv;       // division by cr / 8
    int32_t ncols;         // output columns per group (multiple of 8)
    int32_t b_ld, b_g_ofs;
    int32_t o_h, o_w, o_c, o_cg_ofs;
    int32_t oi_mul, oi_add, oj_mul, oj_add;
    float alpha;
    int32_t groups;
    int32_t group_inner;  // workgroup order: groups innermost
    int32_t diag32;  // igemm_wk only: 64x64 weight blocks, block-diagonal in 32x32 blocks
    int32_t tiles_m, tiles_n;  // per group; filled by the launcher
    TapTable taps;
    int32_t nphase;            // igemm_c64, igemm_wk: phases in ph[]
    TNPhase ph[MAX_PHASES];
};

// 64-element slices, of one tap where cr % 64 == 0 (the C64M tiles: of any
// taps).  pad: some (row, tap) pairs fall outside the A image and must read
// zeros.
enum C64Config { C64_256x256 = 0,   // 8 waves, 64-element slices, 2 stages
                 C64_128x128 = 1,   // 4 waves, 64-element slices, 2 stages
                 C64S_128x128 = 2,  // single stage (several workgroups per CU)
                 C64S_128x64 = 3,
                 C64W_256x256 = 4,    // 16 waves of 64x64, 2 stages
                 C64D_128x64 = 5,     // C64S_128x64 for block-diagonal 64x64 weights
                                      // (32x32 blocks): half the k-steps per wave
                 // LDS ring of 32-element slices with register-prefetched
                 // fragments (one wave per SIMD for 256x256: 128x128 per wave)
                 C64R_256x256 = 6,    // 4 waves of 128x128, 4 stages (128 KB)
                 C64R_256x128 = 7,    // 4 waves of 128x64, 3 stages (72 KB), 2 per CU
                 C64R_256x64 = 8,     // 4 waves of 64x64, 4 stages (80 KB), 2 per CU
                 C64E_128x128 = 36,   // 8 waves of 32x64, 2 stages
                 // any cr that is a multiple of 8: single stage, and two stages
                 C64M_128x64 = 32, C64M_128x128 = 33, C64M2_128x128 = 34 };
hipError_t launch_igemm_c64(int dtype, C64Config cfg, TNParams &p, bool pad, hipStream_t st);

// Small grids, any cr: the waves of a workgroup split the reduction of one
// small tile (igemm_wk.hip); phases as in the 64-channel-slice kernel.
// Names: pixels x channels, waves.
enum WKConfig { WK_32x32_4W = 0, WK_32x32_8W = 1, WK_64x64_4W = 2, WK_64x64_8W = 3 };
hipError_t launch_igemm_wk(int dtype, WKConfig cfg, TNParams &p, bool pad, hipStream_t st);

// Halo staging for stride-1 "same" geometries (igemm_halo.hip): single
// phase, one group, cr % 64 == 0, A image of the output's size, at most 32
// taps whose raster shifts span at most HALO_SPAN pixels (3x3 filters with
// padding 1 on images up to 63 pixels wide).  The single-slice
// register-weight tile also takes groups of 64 reduction channels into 64
// output columns (grouped convolution run as 64-channel super-groups).
constexpr int HALO_SPAN = 128;
enum HaloConfig { HALO_256x64 = 0,      // 4 waves of 64x64
                  HALO_256x128 = 1,     // 4 waves of 128x64
                  HALO_256x64_2T = 2,   // 256x64 with the B tiles of two taps per step
                  // igemm_hring.hip: weight fragments from L2 into registers,
                  // double-buffered halo (one workgroup per CU)
                  HALO_R256x128 = 3,    // 4 waves of 128x64, taps within 64 raster positions
                  HALO_R128x256 = 4,    // 4 waves of 128x64 side by side, taps within 128
                  HALO_R224x256 = 5,    // 4 waves of 224x64 side by side, taps within 32
                  HALO_R256x64S = 6 };  // 4 waves of 64x64, single 64-channel slice
                                        // (cr == 64), three workgroups per CU
// the register-weight configurations are the ones from HALO_R256x128 on
inline bool hring_config(int cfg) { return cfg >= HALO_R256x128 && cfg <= HALO_R256x64S; }
// grouped: also accept p.groups > 1 with groups of cr reduction channels
// into ncols output columns, side by side in the A and output pixels
bool halo_supported(const TNParams &p, bool grouped = false);
// largest minus smallest raster shift of the taps of phase 0
int halo_tap_span(const TNParams &p);
// raster span of the taps the configuration's halo buffer holds
int halo_cfg_span(HaloConfig cfg);
// whether configuration cfg runs p (geometry, tap count and span)
bool halo_cfg_supported(const TNParams &p, HaloConfig cfg);
// hipErrorInvalidValue when !halo_cfg_supported(p, cfg); `pack` is used by
// the register-weight configurations only (see launch_igemm_hring).  diag32:
// the per-tap 64x64 weight blocks are block-diagonal in 32x32 blocks
// (super-groups of groups of at most 32 channels); the single-slice tile then
// skips the zero blocks, the others ignore it.
struct PackSource;
hipError_t launch_igemm_halo(int dtype, HaloConfig cfg, TNParams &p, void *pack, bool diag32,
                             const PackSource *src, hipStream_t st);
// The register-weight halo tiles (igemm_hring.hip) take 3x3 filters (9
// taps) only, HALO_R256x64S a single 64-channel slice (cr == 64) too, and
// it alone more than one group (each of 64 output columns).  They read the
// B operand packed in fragment order: `pack` is caller-provided device
// memory of hring_pack_bytes(ncols, cr, groups) bytes, which
// launch_igemm_hring fills from p.b before the GEMM.
// With src they are packed straight from the caller's weights, without the
// re-laid (backward-data) or block-diagonal (super-group) copy in p.b.
constexpr int HRING_TAPS = 9;
struct PackSource {
    const uint16_t *w;      // element (k, c, tap) at k * sk + c * sc + tap * st
    int32_t sk, sc, st;
    int32_t dgrad;          // columns are channels and the reduction filters
    int32_t m;              // channels per group within a 64-channel super-group, 0: dense
    int32_t kg;             // filters per (super-)group
    int32_t tap_elems;      // p.taps.boff of tap 1
    int32_t *flags;         // null, or per block whether it met an inf or NaN
    uint32_t expmask;       // all exponent bits of the operand type
};
// blocks of the packing launch with a source: the flags it writes
int64_t hring_pack_blocks(int64_t ncols, int64_t cr, int64_t groups);
bool hring_supported(const TNParams &p, int span, bool grouped = false);
size_t hring_pack_bytes(int64_t ncols, int64_t cr, int64_t groups = 1);
hipError_t launch_igemm_hring(int dtype, HaloConfig cfg, TNParams &p, void *pack, bool diag32,
                              const PackSource *src, hipStream_t st);

// Forward pass for 8-channel (16-byte) channel-last pixels, 64 output
// channels, groups 1, dilation 1 and a compiled filter size / stride (the
// stem: 7x7, stride 2).  x [n][h][w][8], wt [64][r][s][8], y [n][p][q][64].
struct StemParams {
    const void *x;
    uint32_t x_bytes;
    const void *wt;
    uint32_t wt_bytes;
    void *y;
    uint32_t y_bytes;
    int32_t n, h, w, p, q;
    int32_t r, s, sh, sw, ph, pw;
    int32_t c;                  // channels per pixel: 8, or 4 (stem4_supported)
    float alpha;
};
bool stem_fwd_supported(int r, int s, int sh, int sw);
// 4-channel pixels: the same filter with an odd left padding and an even
// image width
bool stem4_supported(const StemParams &p);
// cus: workgroups to launch at most (one per CU; the kernel loops over tiles)
hipError_t launch_stem_fwd(int dtype, const StemParams &p, int cus, hipStream_t st);
// Where the operands of a backward-weight launch are taken from: the
// channel-last tensors of its parameters, or, with a source, the caller's
// tensors of any layout and channel count, gathered while they are staged.  The
// same products are summed in the same order either way.
struct WGSource {
    StridedTensor x, dy;
};
struct NoSource {};

// Backward-weight partials for the same shapes: y holds dy; splits
// workgroups each write part[split][64][r*s*c] (no loss-scale step); with
// 4-channel pixels splits is even and splits / 2 workgroups write two each.
hipError_t launch_stem_wgrad(int dtype, const StemParams &p, float *part, int splits,
                             const WGSource *src, hipStream_t st);

// Backward-weight split-K partial sums:
//   ws[split][k][j] = sum over pixels of this split of dy[pix, k] * xcol[pix, j]
// with j = (r*S + s)*Cg + c (the [K][R][S][Cg] order) and channel-last x, dy.
struct WGParams {
    const void *x;
    uint32_t x_bytes;
    const void *dy;
    uint32_t dy_bytes;
    float *ws;
    int32_t h, w, c, k;         // x height/width/channels, dy channels
    int32_t cg, kg;
    int32_t p, q, npq;
    FastDiv div_q, div_pq, div_cg, div_s;
    int32_t sh, sw, ph, pw, dh, dw;
    int32_t rscg;
    int32_t groups, splits, pix_per_split;
    int32_t group_inner;        // workgroup order: groups inside the splits
    int32_t tiles_m, tiles_n;   // filled by the launcher
};

enum WGConfig { WG_128x128 = 0, WG_64x128 = 1, WG_256x256 = 2, WG_128x128S = 3,
                WG_64x128D = 4,  // WG_64x128 for block-diagonal super-group gradients
                WG_HALO = 5 };   // wgrad_halo.hip (3x3 stride-1 "same", 64 -> 64 channels)

// Pixel ranges of pix_per_split (a multiple of 32) pixels each.
hipError_t launch_wgrad_splitk(int dtype, WGConfig cfg, WGParams &p, const WGSource *src,
                               hipStream_t st);

// Backward-weight of a 3x3 stride-1 convolution with padding 1 and groups of
// 64 input and 64 output channels (wgrad_halo.hip): blocks of rb whole image
// rows (rb * w a multiple of 16, at most 128 pixels, wgh_slots(rb, w) at
// most WGH_MAX_SLOTS), blocks_per_split consecutive blocks per workgroup,
// workgroup (split, group) writing rows group * 64 .. + 63 of
// ws[split][groups * 64][9 * 64] (fp32, columns (tap, c)).  diag32: the
// groups are super-groups of groups of at most 32 channels, whose gradient
// is block-diagonal in 32x32 blocks: only those blocks are computed and
// written (the rest of each row is left as it was).
constexpr int WGH_MAX_SLOTS = 3392;
// 16-byte LDS slots a block of rb rows of a w-wide image stages
int wgh_slots(int rb, int w);
struct WGHParams {
    const void *x;
    const void *dy;
    float *ws;
    uint32_t x_bytes, dy_bytes;
    int32_t h, w;                  // image size (input = output)
    int32_t c_stride, k_stride;    // channels per pixel of x and dy
    int32_t rb, blocks_per_img, nblocks, blocks_per_split, splits;
    int32_t groups;                // of 64 channels, side by side in x and dy pixels
    int32_t diag32;
};
hipError_t launch_wgrad_halo(int dtype, const WGHParams &p, const WGSource *src, hipStream_t st);

// dw[e'] = (accumulate ? dw[e'] : 0) + inv_scale * sum_{s < splits} ws[s][e]
// over e < count = K * R*S*Cg; e' = e for [K][R][S][Cg] output, or the
// matching [K][Cg][R][S] index when kcrs != 0.  Stores 1 into *flag when a
// final value is not finite.
hipError_t launch_wgrad_reduce(const float *ws, int32_t splits, int64_t count, void *dw,
                               int out_dtype, float inv_scale, int accumulate, int32_t *flag,
                               int kcrs, int32_t cg, int32_t rs, hipStream_t st);

// Direct (one thread per output) kernels for any valid geometry and either
// layout; element offsets are given by strides.
struct DirectParams {
    int32_t n, c, h, w, k, r, s, p, q;
    int32_t sh, sw, ph, pw, dh, dw, groups, cg, kg;
    int64_t xs[4];   // x strides for (n, c, h, w)
    int64_t ys[4];   // y / dy strides for (n, k, p, q)
    int64_t wsd[4];  // w strides for (k, c, r, s)
    float alpha;
};

hipError_t launch_direct_fwd(int dtype, const DirectParams &p, const void *x, const void *w,
                             void *y, hipStream_t st);
hipError_t launch_direct_dgrad(int dtype, const DirectParams &p, const void *dy, const void *w,
                               void *dx, hipStream_t st);
// Raw sums into ws[split][k][(r*S+s)*Cg + c], pixels split into `splits` ranges.
hipError_t launch_direct_wgrad(int dtype, const DirectParams &p, const void *x, const void *dy,
                               float *ws, int32_t splits, hipStream_t st);

// The three passes of very small convolutions, one launch each, in either
// layout (igemm_tiny.hip): pass 0 out = y from a = x, b = w; 1 out = dx from
// a = dy, b = w; 2 out = dw (0 fp16, 1 bf16, 2 fp32) from a = dy, b = x with the
// loss-scale step of launch_wgrad_reduce.
bool tiny_pays(const DirectParams &p, int pass, bool fast, bool single);
double tiny_us(const DirectParams &p, int pass);
hipError_t launch_igemm_tiny(int dtype, int pass, const DirectParams &p, const void *a,
                             const void *b, void *out, int out_code, float inv_scale,
                             int accumulate, int32_t *flag, hipStream_t st);

// Grouped convolution as super-groups of sg channels (block-diagonal
// weights).  dst[k][t][c'] = w[k][c' - base][t] inside output channel k's
// own group of m channels (base = ((k % sg) / m) * m), else 0; src is
// [K][rs][m] (kcrs = 0) or [K][m][rs] (kcrs = 1).
hipError_t launch_expand_group_weights(const void *src, void *dst, int64_t k, int32_t rs, int32_t m,
                                       int32_t sg, int kcrs, hipStream_t st);
// dw[k][t][c] (k < K, c < m; [K][m][R][S] when kcrs) = (accumulate ? dw : 0) +
// inv_scale * sum_s ws[s][k][t][base(k) + c] over partials of pcount elements
// whose taps are `pitch` elements apart: base(k) = ((k % pitch) / m) * m with
// diag (the diagonal blocks of super-group weight-gradient partials), 0
// without (partials of a convolution with padded channel counts).
hipError_t launch_wgrad_reduce_pick(const float *ws, int32_t splits, int64_t pcount, int64_t k,
                                    int32_t rs, int32_t m, int32_t pitch, bool diag, void *dw,
                                    int out_dtype, float inv_scale, int accumulate, int32_t *flag,
                                    int kcrs, hipStream_t st);

// dst[b][cc][rr] = rr < rows ? src[b][rr][cc] : 0   for rr < dst_ld, cc < cols
hipError_t launch_transpose16(const void *src, void *dst, int64_t batch, int64_t rows,
                              int64_t cols, int64_t dst_ld, hipStream_t st);
// The same from source rows src_ld >= cols elements apart.
hipError_t launch_transpose16_ld(const void *src, void *dst, int64_t batch, int64_t rows,
                                 int64_t cols, int64_t src_ld, int64_t dst_ld, hipStream_t st);
// launch_transpose16 that also stores, per workgroup b of the
// transpose16_blocks(batch, cols, dst_ld) it launches, whether its tile of
// src held an inf or NaN of the given operand dtype into flags[b].
int64_t transpose16_blocks(int64_t batch, int64_t cols, int64_t dst_ld);
// Two independent launch_transpose16 calls in one launch (two launches
// when either cannot take the 16-byte kernel).
hipError_t launch_transpose16_pair(const void *src0, void *dst0, int64_t batch0, int64_t rows0,
                                   int64_t cols0, int64_t dst_ld0, const void *src1, void *dst1,
                                   int64_t batch1, int64_t rows1, int64_t cols1, int64_t dst_ld1,
                                   hipStream_t st);
hipError_t launch_transpose16_scan(const void *src, void *dst, int64_t batch, int64_t rows,
                                   int64_t cols, int64_t dst_ld, int dtype, int32_t *flags,
                                   hipStream_t st);
// flags[b] (b < nonfinite_scan16_blocks(count)) = whether src[2048 b ..
// 2048 b + 2047] holds an inf or NaN.
int64_t nonfinite_scan16_blocks(int64_t count);
hipError_t launch_nonfinite_scan16(const void *src, int64_t count, int dtype, int32_t *flags,
                                   hipStream_t st);
// If any of flags[0, nflags) is set: recompute dx at the border pixels (rows
// [0, bt), [H - bb, H); columns [0, bl), [W - br, W)) from the definition,
// skipping the taps outside dy.  Element strides come from p.
hipError_t launch_dgrad_border(int dtype, const DirectParams &p, const void *dy, const void *w,
                               void *dx, const int32_t *flags, int32_t nflags, int32_t bt,
                               int32_t bb, int32_t bl, int32_t br, hipStream_t st);

// dst[row][ch] = ch < c ? src[row][ch] : 0   for ch < c_pad
hipError_t launch_pad_channels16(const void *src, void *dst, int64_t rows, int32_t c,
                                 int32_t c_pad, hipStream_t st);

// dst[row][ch] = src[row][ch] for ch < c, source rows of c_pad channels
hipError_t launch_unpad_channels16(const void *src, void *dst, int64_t rows, int32_t c,
                                   int32_t c_pad, hipStream_t st);
// dst[n][i][ch] = ch < c ? src[n][ch][i] : 0 for i < hw, ch < c_pad = 4 or 8
hipError_t launch_interleave16(const void *src, void *dst, int64_t n, int32_t c, int64_t hw,
                               int32_t c_pad, hipStream_t st);
// [K][C][rs] (kcrs) or [K][rs][C] weights into [k_pad][rs][c_pad], or with
// klast into [rs][c_pad][k_pad], zero-padded; flags (may be null): per block
// of the pad_weights16_blocks(), whether it holds an inf or NaN.
int64_t pad_weights16_blocks(int64_t k_pad, int64_t c_pad, int64_t rs);
hipError_t launch_pad_weights16(const void *src, void *dst, int32_t k, int32_t c, int32_t k_pad,
                                int32_t c_pad, int32_t rs, int kcrs, bool klast, int dtype,
                                int32_t *flags, hipStream_t st);

// Depthwise convolution (groups = C = K), channel-last, C % 8 == 0, square
// 3x3 / 5x5 / 7x7 filters (depthwise.hip).  Weights are [C][R][S] (the
// KRSC and KCRS layouts coincide for one channel per group).
struct DWParams {
    int32_t n, c, h, w, p, q, r, s;
    int32_t sh, sw, ph, pw, dh, dw;
    int32_t c8;              // c / 8
    int32_t cblocks;         // 64-channel blocks: (c8 + 7) / 8
    uint32_t x_bytes, dy_bytes;  // x and y / dy sizes (buffer range checks)
    int32_t splits;          // backward-weight pixel ranges
    int64_t pix_per_split;
    float alpha;
};
bool dw_supported(int r, int s);
// pass 0: forward (a = x, b = w, out = y); 1: backward-data (a = dy, b = w,
// out = dx); 2: backward-weight partials (a = x, b = dy,
// out = ws[split][c][r*S + s], fp32).
hipError_t launch_depthwise(int dtype, int pass, const DWParams &p, const void *a, const void *b,
                            void *out, hipStream_t st);

// LDS-tiled depthwise kernels (depthwise_tiled.hip): equal strides of 1 or 2,
// no dilation.
struct DWTParams {
    int32_t n, c, c8, cblocks;
    int32_t ih, iw, oh, ow;        // input image; output image (forward) or dy
    int32_t ph, pw;                // top / left padding of the input (may be < 0)
    int32_t tiles_h, tiles_w;
    int32_t th;                    // backward-weight: dy rows per tile
    int32_t tiles_per_split, splits;
    uint32_t in_bytes, dy_bytes;   // buffer range checks
    float alpha;
};
struct DWWgPlan {
    int32_t cbv, th, tiles_h, tiles_w, cblocks, splits, tiles_per_split;
};
bool dw_tiled(const DWParams &p, int pass);
int32_t dw_tiled_wgrad_splits(const DWParams &p);
hipError_t launch_depthwise_tiled(int dtype, int pass, const DWParams &p, const void *a,
                                  const void *b, void *out, hipStream_t st);

// Stride-1 depthwise on the matrix cores (depthwise_mfma.hip): forward, or the
// forward correlation with the rotated filter (flip: backward-data); the input
// and output images, padding and byte sizes are set in p.
// whether it is the faster kernel for this launch; the LDS-tiled kernel's
// workgroups x rows per thread, and rows per thread
bool depthwise_mfma_pays(int dtype, const DWTParams &p, int r, int64_t tiled_work, int tiled_rows);
hipError_t launch_depthwise_mfma(int dtype, const DWTParams &p, int r, bool flip, const void *in,
                                 const void *w, void *out, hipStream_t st);

// Backward-weight on the matrix cores (3x3 and 5x5, stride 1): the number of
// splits (at most max_splits), or 0 where the LDS-tiled kernel runs it; fills
// q's tiling when q is given.
int32_t depthwise_mfma_wgrad_plan(const DWParams &p, int32_t max_splits, DWTParams *q);
hipError_t launch_depthwise_mfma_wgrad(int dtype, int r, const DWTParams &q, const void *x,
                                       const void *dy, float *ws, hipStream_t st);

// Training-step pieces (update.hip).  The state type is the C ABI's.
hipError_t launch_loss_scaler_init(nnconv_loss_scaler *s, float scale, float factor,
                                   int32_t interval, hipStream_t st);
hipError_t launch_loss_scaler_update(nnconv_loss_scaler *s, int32_t *flag, hipStream_t st);
hipError_t launch_sgd_update(int64_t count, float *master, float *mom, void *w16, int w16_dtype,
                             const float *grad, const nnconv_loss_scaler *state,
                             const int32_t *flag, float lr, float mu, float wd, hipStream_t st);

}  // namespace nnconv

// depthwise_mfma.hip -- stride-1 depthwise convolution on the matrix cores:
// forward, and backward-data (the forward correlation of dy with the rotated
// filter); no dilation, 3x3 / 5x5 / 7x7, channel-last.
//
// On the vector ALUs a 5x5 layer needs 25 multiply-adds per output, and with
// bf16 operands each also widens a weight: 128 images of 28x28x240 took 62 us
// (fp16 39) where the tensors' bytes take 19.  v_mfma_f32_16x16x32 does 512 products per
// clock and SIMD against 16, so it pays even though only 1 of 16 is useful:
//   D[channel, pixel] += sum_k W[channel, k] * X[k, pixel],
//   k = (one of two filter columns s, one of 16 channels),
// where W is the 16x16 diagonal matrix of the filter's weights at (r, s).  X is
// read from the channel-last LDS tile as it lies (8 consecutive channels of a
// pixel are a lane's 16 bytes), D holds 4 consecutive channels of a pixel per
// lane.  An X fragment (one tile row, one pair of filter columns) serves every
// filter row, each into its own output row, so 3 fragment reads feed 15 MFMAs
// of a 5x5 layer.  Per 16x16 outputs: R * ceil(R/2) MFMAs of 16 clocks.
//
// The zeros off the diagonal must not meet an inf or NaN of another channel
// (0 * inf = NaN): the staging checks every element, and a workgroup whose
// tile holds one computes it on the vector ALUs, channel by channel.
// 128 images of 28x28x240, 5x5: bf16 61.5 -> 29.5 us, fp16 39 -> 29.5.
#include <cstring>

#include "launch.hpp"

namespace nnconv {

namespace dwm {

// Running maximum of the magnitudes of 16-bit values, two at a time; at or
// above INF one of them was inf or NaN.
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
template <class T>
constexpr uint32_t INF = T::id == Half::id ? 0x7C00u : 0x7F80u;
__device__ __forceinline__ void max_abs(u16x2 &m, u32x4 v) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
        m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, v[i] & 0x7FFF7FFFu));
}

// Mask of 8 consecutive 16-bit values that keeps the first n.
__device__ __forceinline__ u32x4 keep_first(int n) {
    u32x4 m;
#pragma unroll
    for (int d = 0; d < 4; ++d)
        m[d] = (2 * d < n ? 0xFFFFu : 0u) | (2 * d + 1 < n ? 0xFFFF0000u : 0u);
    return m;
}

// Tile: NCG groups of 16 channels x NCB blocks of 16 pixels, one wave each;
// a block is 16 columns of a row (PXW = 16), or 8 columns of two rows TR rows
// apart (PXW = 8, narrow images).  TR: output rows per strip of a wave.
template <int R, int NCG, int NCB, int PXW, int TR>
struct Tile {
    static constexpr int CPP = NCG * 2;  // 16-byte chunks per pixel
    static constexpr int TW = NCB * PXW;
    static constexpr int HALVES = 16 / PXW;
    static constexpr int TH = TR * HALVES;
    static constexpr int IW = TW - 1 + R;
    static constexpr int IH = TH - 1 + R;
    static constexpr int CHUNKS = IH * IW * CPP;
    static constexpr int NL = (CHUNKS + 255) / 256;
    static constexpr int NP = (R + 1) / 2;  // pairs of filter columns
    static constexpr int RS = R * R;
};

// Swizzle of the 16-byte chunks of a pixel in tile column c: any 16
// consecutive columns at one chunk fall in 16 distinct 16-byte bank groups.
template <int CPP>
__device__ __forceinline__ int swz(int c) {
    return CPP == 2 ? (c >> 3) & 1 : CPP == 4 ? (c >> 2) & 3 : (c >> 1) & 7;
}

}  // namespace dwm

// out[n, o, u, c] = alpha * sum_{r,s} in[n, o - ph + r, u - pw + s, c] * w'[c, r, s]
// with w' = w, or w rotated by 180 degrees (FLIP).
template <class T, int R, int NCG, int NCB, int PXW, int TR, bool FLIP>
__global__ __launch_bounds__(256) void dwm_fwd_kernel(const DWTParams P,
                                                      const uint16_t *__restrict__ in,
                                                      const uint16_t *__restrict__ w,
                                                      uint16_t *__restrict__ out) {
    using namespace dwm;
    using F = Tile<R, NCG, NCB, PXW, TR>;
    static_assert(NCG * NCB == 4, "four waves");
    constexpr int CW = NCG * 16;  // channels of the block
    __shared__ u32x4 tile[F::CHUNKS];
    __shared__ uint16_t wl[CW * F::RS];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    uint32_t b = xcd_remap(blockIdx.x, gridDim.x);
    const int cb = (int)(b % (uint32_t)P.cblocks);
    b /= (uint32_t)P.cblocks;
    const int tw = (int)(b % (uint32_t)P.tiles_w);
    b /= (uint32_t)P.tiles_w;
    const int th = (int)(b % (uint32_t)P.tiles_h);
    const int n = (int)(b / (uint32_t)P.tiles_h);
    const int oh0 = th * F::TH, ow0 = tw * F::TW;

    // The whole input tile in flight; outside the image (or past the last
    // channel vector) the range check returns zeros.  A thread keeps its
    // chunk of a pixel and walks PX pixels (in tile raster order) per load.
    constexpr int PX = 256 / F::CPP, DROW = PX / F::IW, DCOL = PX % F::IW;
    const int cvl = tid % F::CPP;
    const int row0 = (tid / F::CPP) / F::IW, col0 = (tid / F::CPP) % F::IW;
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(in, P.in_bytes);
    u32x4 ld[F::NL];
    {
        const int h0 = oh0 - P.ph, w0 = ow0 - P.pw;
        const int c2 = P.c * 2;
        int h = h0 + row0, wc = w0 + col0;
        uint32_t off = (uint32_t)((n * P.ih + h) * P.iw + wc) * (uint32_t)c2 +
                       (uint32_t)(cb * F::CPP + cvl) * 16u;
        const uint32_t step = (uint32_t)((DROW * P.iw + DCOL) * c2);
        const uint32_t wrap = (uint32_t)((P.iw - F::IW) * c2);
        // rows past the tile fail the row test
        const int h_end = min(P.ih, h0 + F::IH);
        const int w_lim = w0 + F::IW;
        const bool lane_in = cb * F::CPP + cvl < P.c8;
#pragma unroll
        for (int k = 0; k < F::NL; ++k) {
            const bool ok = lane_in && h >= 0 && h < h_end && (unsigned)wc < (unsigned)P.iw;
            ld[k] = load16(rin, ok ? off : OOB_OFFSET);
            h += DROW;
            wc += DCOL;
            off += step;
            if (wc >= w_lim) {
                wc -= F::IW;
                h += 1;
                off += wrap;
            }
        }
    }
    // weights of the block's channels, [channel][tap] as in memory
    for (int e = tid; e < CW * F::RS; e += 256) {
        const int64_t g0 = (int64_t)cb * CW * F::RS;
        const int cl = e / F::RS, t = e - cl * F::RS;
        wl[e] = cb * CW + cl < P.c ? w[g0 + (FLIP ? cl * F::RS + F::RS - 1 - t : e)] : (uint16_t)0;
    }
    u16x2 big = {};
    {
        int col = col0;
#pragma unroll
        for (int k = 0; k < F::NL; ++k) {
            max_abs(big, ld[k]);
            if (F::NL * 256 == F::CHUNKS || k * 256 + tid < F::CHUNKS)
                tile[(k * PX + tid / F::CPP) * F::CPP + (cvl ^ swz<F::CPP>(col))] = ld[k];
            col += DCOL;
            if (col >= F::IW) col -= F::IW;
        }
    }
    const bool bad = __syncthreads_or(big[0] >= INF<T> || big[1] >= INF<T>);

    if (bad) {
        // 8 channels of a column of RT rows per thread, RC rows at a time, the
        // taps in the order of the definition.  An overflow step of training
        // has such tiles everywhere: 128 images of 28x28x240, 5x5, every input
        // inf, 46 us (one output element at a time: 186; the vector kernel: 36).
        constexpr int ITEMS = F::CPP * F::TW, RT = (F::TH * ITEMS + 255) / 256, RC = RT < 4 ? RT : 4;
        static_assert(256 % ITEMS == 0, "whole columns per row group");
        const int j = tid / F::CPP % F::TW, ch = cb * CW + cvl * 8, ow = ow0 + j;
        if (ch >= P.c || ow >= P.ow) return;
        const int i1 = min(tid / ITEMS * RT + RT, F::TH);
#pragma unroll 1
        for (int i0 = tid / ITEMS * RT; i0 < i1; i0 += RC) {
            float acc[RC][8] = {};
#pragma unroll 1
            for (int t = 0; t < F::RS; ++t) {
                const int r = t / R, s = t - r * R;
                float wv[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) wv[e] = from16<T>(wl[(cvl * 8 + e) * F::RS + t]);
                const u32x4 *col = tile + (r * F::IW + j + s) * F::CPP + (cvl ^ swz<F::CPP>(j + s));
#pragma unroll
                for (int i = 0; i < RC; ++i) {
                    const u32x4 xv = col[min(i0 + i, F::TH - 1) * (F::IW * F::CPP)];
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        acc[i][e] = __builtin_fmaf(from16<T>((uint16_t)(xv[e >> 1] >> (16 * (e & 1)))),
                                                   wv[e], acc[i][e]);
                }
            }
#pragma unroll
            for (int i = 0; i < RC; ++i) {
                const int oh = oh0 + i0 + i;
                if (i0 + i >= i1 || oh >= P.oh) break;
                u32x4 v;
#pragma unroll
                for (int d = 0; d < 4; ++d)
                    v[d] = to16<T>(acc[i][2 * d] * P.alpha) | (to16<T>(acc[i][2 * d + 1] * P.alpha) << 16);
                *(u32x4 *)(out + (((int64_t)n * P.oh + oh) * P.ow + ow) * P.c + ch) = v;
            }
        }
        return;
    }

    const int g = wave % NCG, blk = wave / NCG;  // channel group, pixel block
    const int l16 = lane & 15, q = lane >> 4;
    // diagonal weight fragments: lane row = channel l16, k = 8 q + e is
    // channel 8 (q & 1) + e of filter column 2 pr + (q >> 1)
    u32x4 wf[R][F::NP];
    {
        const bool diag = (q & 1) == (l16 >> 3);
        const int dword = (l16 & 7) >> 1, sh = (l16 & 1) * 16;
        const uint16_t *wc = wl + (g * 16 + l16) * F::RS;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int pr = 0; pr < F::NP; ++pr) {
                const int s = 2 * pr + (q >> 1);
                const uint32_t v =
                    diag && s < R ? (uint32_t)wc[r * R + (s < R ? s : 0)] << sh : 0u;
#pragma unroll
                for (int d = 0; d < 4; ++d) wf[r][pr][d] = d == dword ? v : 0u;
            }
    }
    // LDS address of the lane's 16 bytes per pair of filter columns (a column
    // past the filter re-reads the last one: its weight is zero, and what it
    // reads is finite)
    const int dr = PXW == 16 ? 0 : l16 / PXW, dc = l16 % PXW;
    const int col = blk * PXW + dc;
    const u32x4 *xb[F::NP];
#pragma unroll
    for (int pr = 0; pr < F::NP; ++pr) {
        const int c = col + (2 * pr + (q >> 1) < R ? 2 * pr + (q >> 1) : R - 1);
        xb[pr] = tile + (dr * TR * F::IW + c) * F::CPP + ((g * 2 + (q & 1)) ^ swz<F::CPP>(c));
    }

    const int ch = (cb * NCG + g) * 16 + 4 * q;
    const int ow = ow0 + col;
    // output rows of this lane's strip inside the image
    const int live = ch < P.c && ow < P.ow ? P.oh - (oh0 + dr * TR) : 0;
    uint16_t *o = out + (((int64_t)n * P.oh + oh0 + dr * TR) * P.ow + ow) * P.c + ch;
    const int64_t ostep = (int64_t)P.ow * P.c;
    f32x4 acc[TR];
#pragma unroll
    for (int hh = 0; hh < TR - 1 + R; ++hh) {
        u32x4 xf[F::NP];
#pragma unroll
        for (int pr = 0; pr < F::NP; ++pr) xf[pr] = xb[pr][hh * (F::IW * F::CPP)];
        // input row hh is filter row r of output row hh - r
#pragma unroll
        for (int pr = 0; pr < F::NP; ++pr)
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (hh - r >= 0 && hh - r < TR)
                    acc[hh - r] = mfma16<T>(wf[r][pr], xf[pr],
                                            r == 0 && pr == 0 ? f32x4{} : acc[hh - r]);
        if (hh >= R - 1) {  // its last filter row
            const int p = hh - (R - 1);
            if (p < live) {
                u32x2 pk;
                pk[0] = to16<T>(acc[p][0] * P.alpha) | (to16<T>(acc[p][1] * P.alpha) << 16);
                pk[1] = to16<T>(acc[p][2] * P.alpha) | (to16<T>(acc[p][3] * P.alpha) << 16);
                *(u32x2 *)(o + p * ostep) = pk;
            }
        }
    }
}

// Backward-weight of the same layers (3x3 and 5x5, stride 1): partials
// ws[split][c][r*R + s] = sum over the split's pixels of dy * x.
//
//   D[i, j] += sum_k dy[pixel k, channel i] * x[pixel k + tap, channel j]
//
// of which the diagonal i = j is the gradient: 1 of 16 products is useful, at
// 512 a clock, and an inf or NaN cannot leave its own row and column (nor its
// own taps: sums that are not finite are taken again without the pixels past
// the output's edge).  Both
// operands are pixel-major in LDS and read with the transposing reads; k runs
// over 32 pixels, COLS columns of 32 / COLS image rows HR apart, so that one
// x fragment (an input row, a column shift s) meets the dy fragments of all R
// filter rows: R + 1 fragment reads feed R*R MFMAs.
//
// A workgroup is two pairs of waves; wave g of a pair owns 16 of the block's
// 32 channels, and the pairs take every other block of HR * 32 / COLS rows x
// COLS columns of the split, staged by buffer_load ... lds, rows and columns
// outside the image as zeros.  The pairs' sums are added in order at the end.
// 128 images of 28x28x240, 5x5: 47.7 -> 28.8 us (with the split reduction);
// 14x14x480, 5x5: 31.8 -> 20.1; 7x7x1152, 3x3: 15.3 -> 10.7.
namespace dwm {
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

template <int R, int COLS, int HR>
struct WBlock {
    static constexpr int PARTS = 32 / COLS;      // row ranges of a k-step
    static constexpr int ROWS = PARTS * HR;      // dy rows
    static constexpr int IW = COLS + R - 1;
    static constexpr int XP = (ROWS + R - 1) * IW, DP = ROWS * COLS;  // pixels of 64 bytes
    static constexpr int NX = (XP * 4 + 63) / 64, ND = (DP * 4 + 63) / 64;  // 1 KB loads
    static constexpr int BYTES = (NX + ND) * 1024;
};
}  // namespace dwm

template <class T, int R, int COLS, int HR>
__global__ __launch_bounds__(256) void dwm_wgrad_kernel(const DWTParams P,
                                                        const uint16_t *__restrict__ x,
                                                        const uint16_t *__restrict__ dy,
                                                        float *__restrict__ ws) {
    using namespace dwm;
    using W = WBlock<R, COLS, HR>;
    constexpr int RS = R * R;
    __shared__ __align__(16) char lds[2 * W::BYTES];
    static_assert(2 * W::BYTES >= 2 * RS * 16 * 4, "the second pair's sums");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pair = wave >> 1, g = wave & 1;
    const uint32_t b = xcd_remap(blockIdx.x, gridDim.x);
    const int cb = (int)(b % (uint32_t)P.cblocks);  // 32 channels
    const int split = (int)(b / (uint32_t)P.cblocks);
    const int nblocks = P.n * P.tiles_h * P.tiles_w;
    const int begin = split * P.tiles_per_split;
    const int end = min(nblocks, begin + P.tiles_per_split);

    const i32x4 rx = desc_of(x, P.in_bytes);
    const i32x4 rdy = desc_of(dy, P.dy_bytes);
    const uint32_t lx = (uint32_t)(uintptr_t)(lds_void *)&lds[0] + (uint32_t)(pair * W::BYTES);
    const uint32_t ld = lx + W::NX * 1024u;
    const int c2 = P.c * 2;
    const int cvl = lane & 3;
    const bool ch_ok = cb * 4 + cvl < P.c8;
    const uint32_t ch_ofs = (uint32_t)(cb * 4 + cvl) * 16u;

    auto stage = [&](int t) {
        const bool live = t < end;
        const int tw = t % P.tiles_w;
        const int t2 = t / P.tiles_w;
        const int th = t2 % P.tiles_h;
        const int n = t2 / P.tiles_h;
        const int p0 = th * W::ROWS, q0 = tw * COLS;
        const int h0 = p0 - P.ph, w0 = q0 - P.pw;
#pragma unroll
        for (int j0 = 0; j0 < W::NX; j0 += 2) {
            const int j = j0 + g;
            const int px = j * 16 + (lane >> 2);
            const int row = px / W::IW, col = px - row * W::IW;
            const int h = h0 + row, wc = w0 + col;
            const bool ok = live && ch_ok && px < W::XP && (unsigned)h < (unsigned)P.ih &&
                            (unsigned)wc < (unsigned)P.iw;
            if (j < W::NX)
                dma16(lx + (uint32_t)j * 1024u,
                      ok ? (uint32_t)((n * P.ih + h) * P.iw + wc) * (uint32_t)c2 + ch_ofs : OOB_OFFSET,
                      rx);
        }
#pragma unroll
        for (int j0 = 0; j0 < W::ND; j0 += 2) {
            const int j = j0 + g;
            const int px = j * 16 + (lane >> 2);
            const int row = px / COLS, col = px - row * COLS;
            const int p = p0 + row, q = q0 + col;
            const bool ok = live && ch_ok && px < W::DP && p < P.oh && q < P.ow;
            if (j < W::ND)
                dma16(ld + (uint32_t)j * 1024u,
                      ok ? (uint32_t)((n * P.oh + p) * P.ow + q) * (uint32_t)c2 + ch_ofs : OOB_OFFSET,
                      rdy);
        }
    };

    // transposing reads: lane group gq holds pixels 8 gq .. 8 gq + 7 of the
    // k-step, four per read; lane li addresses pixel li / 4, channels 4 (li % 4)
    const int li = lane & 15, gq = lane >> 4;
    const int k0 = 8 * gq + (li >> 2);
    const int rpart = k0 / COLS, rcol = k0 % COLS;
    const uint32_t xa = lx + (uint32_t)((rpart * HR * W::IW + rcol) * 64 + g * 32 + (li & 3) * 8);
    const uint32_t da = ld + (uint32_t)((rpart * HR * COLS + rcol) * 64 + g * 32 + (li & 3) * 8);
    auto frag = [&](uint32_t a) -> u32x4 {
        const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(uintptr_t)a);
        const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(uintptr_t)(a + 256));
        const u32x2 lo = __builtin_bit_cast(u32x2, v0), hi = __builtin_bit_cast(u32x2, v1);
        return u32x4{lo[0], lo[1], hi[0], hi[1]};
    };

    f32x4 acc[R][R];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int s = 0; s < R; ++s) acc[r][s] = f32x4{};

    for (int t0 = begin; t0 < end; t0 += 2) {
        if (t0 > begin) barrier_lds();  // the previous blocks have been read
        stage(t0 + pair);
        wait_vmcnt<0>();
        barrier_lds();
        u32x4 df[HR];
#pragma unroll
        for (int h = 0; h < HR + R - 1; ++h) {
            u32x4 xf[R];
#pragma unroll
            for (int s = 0; s < R; ++s) xf[s] = frag(xa + (uint32_t)((h * W::IW + s) * 64));
            if (h < HR) df[h] = frag(da + (uint32_t)(h * COLS * 64));
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (h - r >= 0 && h - r < HR)
#pragma unroll
                    for (int s = 0; s < R; ++s) acc[r][s] = mfma16<T>(df[h - r], xf[s], acc[r][s]);
        }
    }

    // the diagonal: lane (channel li as column) of group li / 4, element li % 4
    barrier_lds();
    float *other = (float *)&lds[0] + g * (RS * 16);
    const bool mine = gq == (li >> 2);
    float v[RS];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int s = 0; s < R; ++s) {
            const f32x4 a = acc[r][s];
            v[r * R + s] = (li & 2) ? ((li & 1) ? a[3] : a[2]) : ((li & 1) ? a[1] : a[0]);
        }
    if (pair == 1 && mine) {
#pragma unroll
        for (int t = 0; t < RS; ++t) other[t * 16 + li] = v[t];
    }
    barrier_lds();
    const int ch = cb * 32 + g * 16 + li;
    const bool store = pair == 0 && mine && ch < P.c;
    bool bad = false;
    if (store) {
#pragma unroll
        for (int t = 0; t < RS; ++t) {
            v[t] += other[t * 16 + li];
            bad |= !__builtin_isfinite(v[t]);
        }
    }
    float *o = ws + ((int64_t)split * P.c + ch) * RS;
    if (store) {
#pragma unroll
        for (int t = 0; t < RS; ++t) o[t] = v[t];
    }
    // The zeros staged for dy past the last output row and column have met x
    // pixels inside the image: an inf among those is no term of the tap's sum.
    // Sums that are not finite are an overflow step's as a rule, with a finite
    // x: a look at x says so.  Otherwise the sums again without those pixels, a
    // filter row at a time.  128 images of 28x28x240, 5x5: 31 us, with every dy
    // inf 39, with every x inf 131 (term by term, whatever x holds: 2940).
    if (P.oh % W::ROWS == 0 && P.ow % COLS == 0) return;
    if (!__syncthreads_or(bad)) return;
    const __amdgpu_buffer_rsrc_t rxv = make_rsrc(x, P.in_bytes);
    u16x2 big = {};
#pragma unroll 1
    for (int t = begin; t < end; ++t) {
        const int t2 = t / P.tiles_w;
        const int h0 = t2 % P.tiles_h * W::ROWS - P.ph, w0 = t % P.tiles_w * COLS - P.pw;
        const int n = t2 / P.tiles_h;
#pragma unroll
        for (int px0 = 0; px0 < W::XP; px0 += 64) {
            const int px = px0 + (tid >> 2), h = h0 + px / W::IW, wc = w0 + px % W::IW;
            const bool ok = ch_ok && px < W::XP && (unsigned)h < (unsigned)P.ih &&
                            (unsigned)wc < (unsigned)P.iw;
            max_abs(big, load16(rxv, ok ? (uint32_t)((n * P.ih + h) * P.iw + wc) * (uint32_t)c2 + ch_ofs
                                        : OOB_OFFSET));
        }
    }
    if (!__syncthreads_or(big[0] >= INF<T> || big[1] >= INF<T>)) return;
#pragma unroll 1
    for (int r = 0; r < R; ++r) {
        f32x4 sum[R];
#pragma unroll
        for (int s = 0; s < R; ++s) sum[s] = f32x4{};
#pragma unroll 1
        for (int t0 = begin; t0 < end; t0 += 2) {
            barrier_lds();
            stage(t0 + pair);
            // of the lane's 8 pixels, which lie in one row, and of its rows
            const int cols = P.ow - (t0 + pair) % P.tiles_w * COLS - 8 * gq % COLS;
            const int rows = P.oh - (t0 + pair) / P.tiles_w % P.tiles_h * W::ROWS - rpart * HR;
            wait_vmcnt<0>();
            barrier_lds();
#pragma unroll 1
            for (int h = 0; h < HR; ++h) {
                const u32x4 keep = keep_first(h < rows ? cols : 0);
                const u32x4 d = frag(da + (uint32_t)(h * COLS * 64));
#pragma unroll
                for (int s = 0; s < R; ++s)
                    sum[s] = mfma16<T>(d, frag(xa + (uint32_t)(((h + r) * W::IW + s) * 64)) & keep, sum[s]);
            }
        }
        barrier_lds();
        float f[R];
#pragma unroll
        for (int s = 0; s < R; ++s) {
            f[s] = (li & 2) ? ((li & 1) ? sum[s][3] : sum[s][2]) : ((li & 1) ? sum[s][1] : sum[s][0]);
            if (pair == 1 && mine) other[s * 16 + li] = f[s];
        }
        barrier_lds();
        if (store) {
#pragma unroll
            for (int s = 0; s < R; ++s) o[r * R + s] = f[s] + other[s * 16 + li];
        }
    }
}

namespace {

constexpr int strip_rows(int r) { return r <= 5 ? 14 : 7; }

struct DwmPlan {
    int cfg;      // as in launch_dwm_rs
    int64_t wgs;
};
DwmPlan plan(const DWTParams &q, int r) {
    const int tr = strip_rows(r);
    auto up = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
    if (q.ow <= 8) return {0, q.n * up(q.c, 64) * up(q.oh, 8)};
    if (q.ow <= 16) return {1, q.n * up(q.c, 64) * up(q.oh, tr)};
    // wider images, tiles 32 pixels wide: 32 channels x tr rows, or 16
    // channels x 2 tr rows (less halo where the image's height fills it),
    // whichever stages fewer vectors
    const int64_t tw = up(q.ow, 32);
    const int64_t a = up(q.c, 32) * up(q.oh, tr), va = a * (tr - 1 + r) * (31 + r) * 4;
    const int64_t b = up(q.c, 16) * up(q.oh, 2 * tr), vb = b * (2 * tr - 1 + r) * (31 + r) * 2;
    return vb < va ? DwmPlan{2, q.n * tw * b} : DwmPlan{3, q.n * tw * a};
}

template <class T, int R, int NCG, int NCB, int PXW, int TR, bool FLIP>
hipError_t launch_dwm_cfg(DWTParams q, const void *in, const void *w, void *out, hipStream_t st) {
    using F = dwm::Tile<R, NCG, NCB, PXW, TR>;
    q.cblocks = (q.c + NCG * 16 - 1) / (NCG * 16);
    q.tiles_w = (q.ow + F::TW - 1) / F::TW;
    q.tiles_h = (q.oh + F::TH - 1) / F::TH;
    const int64_t nb = (int64_t)q.n * q.tiles_h * q.tiles_w * q.cblocks;
    if (nb <= 0) return hipSuccess;
    if (nb > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL((dwm_fwd_kernel<T, R, NCG, NCB, PXW, TR, FLIP>), dim3((uint32_t)nb),
                       dim3(256), 0, st, q, (const uint16_t *)in, (const uint16_t *)w,
                       (uint16_t *)out);
    return hipGetLastError();
}

template <class T, int R, bool FLIP>
hipError_t launch_dwm_rs(const DWTParams &q, const void *in, const void *w, void *out,
                         hipStream_t st) {
    constexpr int TR = strip_rows(R);
    // 3x3: bf16, 9 to 16 wide only (depthwise_mfma_pays)
    if constexpr (R == 3 && T::id == Half::id) return hipErrorInvalidValue;
    else if constexpr (R == 3) return launch_dwm_cfg<T, R, 4, 1, 16, TR, FLIP>(q, in, w, out, st);
    else switch (plan(q, R).cfg) {
        case 0: return launch_dwm_cfg<T, R, 4, 1, 8, 4, FLIP>(q, in, w, out, st);
        case 1: return launch_dwm_cfg<T, R, 4, 1, 16, TR, FLIP>(q, in, w, out, st);
        case 2: return launch_dwm_cfg<T, R, 1, 4, 8, TR, FLIP>(q, in, w, out, st);
        default: return launch_dwm_cfg<T, R, 2, 2, 16, TR, FLIP>(q, in, w, out, st);
    }
}

template <class T, bool FLIP>
hipError_t launch_dwm_t(const DWTParams &q, int r, const void *in, const void *w, void *out,
                        hipStream_t st) {
    switch (r) {
        case 3: return launch_dwm_rs<T, 3, FLIP>(q, in, w, out, st);
        case 5: return launch_dwm_rs<T, 5, FLIP>(q, in, w, out, st);
        case 7: return launch_dwm_rs<T, 7, FLIP>(q, in, w, out, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace

// The faster kernel for a launch by estimates in microseconds, fitted to 8800
// random and EfficientNet-like layers (6% rms here, 7-15% the LDS-tiled kernel).
// Both pay for the tensors' MB and for their tiles, inside the image or not: the
// strips here are long, so the vector kernel keeps small grids and images that
// fill the tiles badly, and in fp16, where it needs no widening, more of them
// than in bf16.  tiled_work: its workgroups x rows per thread; tiled_rows: rows
// per thread.
// Against thresholds of one or two workgroups per CU, calls that are more than
// 5% slower than the vector kernel: 423 -> 60 (47 of 464 channels, 15x15, 7x7 fp16
// 17 us against 25; 106 of 864, 5x8, 5x5 11 against 13), geometric mean 0.903 ->
// 0.893 of its time.
// 3x3 layers in fp16 stay there (960 channels, 14x14, 128 images 25.8 us against
// 28.4), and wide and narrow images: on wide ones both are near the HBM rate,
// and the blocks of up to 64 channels touch fewer partial lines (three passes, 128
// images, vector -> matrix cores: 96 channels, 112x112, fp16 413 -> 527 us, bf16
// 453 -> 530; 144 channels, 56x56, fp16 186 -> 211, bf16 208 both); up to 8 wide a
// tile is little more than its set-up (1152 channels, 7x7, 128 images 9.4 -> 10.7).
bool depthwise_mfma_pays(int dtype, const DWTParams &q, int r, int64_t tiled_work, int tiled_rows) {
    if (r == 3 && (dtype == Half::id || q.ow <= 8 || q.ow > 16)) return false;
    // start, per MB, per workgroup row (tiled) or workgroup (by tile) on each CU
    static const double tiled[2][3][3] = {
        {{0.0, 0.0, 0.0}, {4.25, 0.100, 0.589}, {5.08, 0.109, 1.224}},
        {{3.82, 0.037, 0.437}, {3.53, 0.0, 1.211}, {4.80, 0.0, 2.183}}};
    static const double here[3][6] = {{4.86, 0.130, 0.0, 1.07, 0.0, 0.0},
                                      {5.56, 0.146, 0.44, 2.37, 1.75, 1.99},
                                      {5.05, 0.163, 2.27, 3.43, 2.50, 2.82}};
    const double mb = 2e-6 * q.n * q.c * ((double)q.ih * q.iw + (double)q.oh * q.ow);
    const double *a = tiled[dtype == Half::id ? 0 : 1][(r - 3) / 2], *b = here[(r - 3) / 2];
    const DwmPlan pl = plan(q, r);
    const double rows = (double)tiled_work / 256, wgs = (double)pl.wgs / 256;
    const double t = a[0] + a[1] * mb + a[2] * (rows > tiled_rows ? rows : tiled_rows);
    const double m = b[0] + b[1] * mb + b[2 + pl.cfg] * (wgs > 1 ? wgs : 1);
    return 1.03 * m < t;
}

hipError_t launch_depthwise_mfma(int dtype, const DWTParams &q, int r, bool flip, const void *in,
                                 const void *w, void *out, hipStream_t st) {
    if (dtype == Half::id)
        return flip ? launch_dwm_t<Half, true>(q, r, in, w, out, st)
                    : launch_dwm_t<Half, false>(q, r, in, w, out, st);
    return flip ? launch_dwm_t<BFloat, true>(q, r, in, w, out, st)
                : launch_dwm_t<BFloat, false>(q, r, in, w, out, st);
}

namespace {

// Blocks of the backward-weight kernel: 16 columns x 14 rows, or 8 x 8 for
// images up to 8 wide.
template <class T, int R, int COLS, int HR>
hipError_t launch_dwm_wgrad_cfg(DWTParams q, const void *x, const void *dy, float *ws,
                                hipStream_t st) {
    const int64_t nb = (int64_t)q.cblocks * q.splits;
    if (nb > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL((dwm_wgrad_kernel<T, R, COLS, HR>), dim3((uint32_t)nb), dim3(256), 0, st, q,
                       (const uint16_t *)x, (const uint16_t *)dy, ws);
    return hipGetLastError();
}

template <class T, int R>
hipError_t launch_dwm_wgrad_r(const DWTParams &q, const void *x, const void *dy, float *ws,
                              hipStream_t st) {
    if (q.ow <= 8) return launch_dwm_wgrad_cfg<T, R, 8, 2>(q, x, dy, ws, st);
    return launch_dwm_wgrad_cfg<T, R, 16, 7>(q, x, dy, ws, st);
}

}  // namespace

// About 1024 workgroups, no more splits than the LDS-tiled kernel would write
// (the workspace does not grow), at least two blocks each; below 96 workgroups
// that kernel's smaller tiles spread better (480 channels, 14x14, 3x3 on one
// image: both 7.0 us; 16 images 8.6 against 6.8).
int32_t depthwise_mfma_wgrad_plan(const DWParams &p, int32_t max_splits, DWTParams *q) {
    if (p.sh != 1 || p.sw != 1 || (p.r != 3 && p.r != 5)) return 0;
    if (p.r == 3 && p.q > 16) return 0;  // wide images: as for the forward pass
    const int rows = p.q <= 8 ? 8 : 14, cols = p.q <= 8 ? 8 : 16;
    const int th = (p.p + rows - 1) / rows, tw = (p.q + cols - 1) / cols;
    const int64_t blocks = (int64_t)p.n * th * tw;
    const int cblocks = (p.c + 31) / 32;
    int64_t splits = 1024 / cblocks;
    if (splits > blocks / 2) splits = blocks / 2;  // two blocks at a time
    if (splits > max_splits) splits = max_splits;
    if (splits < 1 || splits * cblocks < 96) return 0;
    // two workgroups fit a CU: a few more than that would be a second round (a
    // 5x5 layer with 513 workgroups 23.2 us, the LDS-tiled kernel 16.0)
    if (splits * cblocks > 512 && splits * cblocks < 768 && cblocks <= 512) splits = 512 / cblocks;
    const int64_t per = (blocks + splits - 1) / splits;
    splits = (blocks + per - 1) / per;
    if (q) {
        q->cblocks = cblocks;
        q->tiles_h = th;
        q->tiles_w = tw;
        q->tiles_per_split = (int32_t)per;
        q->splits = (int32_t)splits;
    }
    return (int32_t)splits;
}

hipError_t launch_depthwise_mfma_wgrad(int dtype, int r, const DWTParams &q, const void *x,
                                       const void *dy, float *ws, hipStream_t st) {
    if (dtype == Half::id)
        return r == 3 ? launch_dwm_wgrad_r<Half, 3>(q, x, dy, ws, st)
                      : launch_dwm_wgrad_r<Half, 5>(q, x, dy, ws, st);
    return r == 3 ? launch_dwm_wgrad_r<BFloat, 3>(q, x, dy, ws, st)
                  : launch_dwm_wgrad_r<BFloat, 5>(q, x, dy, ws, st);
}

}  // namespace nnconv

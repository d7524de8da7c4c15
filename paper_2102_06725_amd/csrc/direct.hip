// direct.hip -- direct convolution kernels (one thread per output element)
// for geometries the matrix-core kernels do not take: channel counts per
// group that are not multiples of 8, unaligned pointers, tensors beyond the
// 2 GiB buffer range, or more than 64 filter taps.  Same semantics as the
// fast path: fp32 accumulation, round-to-nearest-even output.  Both layouts
// are handled through element strides.  Also the 16-bit layout transforms.
#include <type_traits>

#include "launch.hpp"

namespace nnconv {

template <class T>
__device__ __forceinline__ float ld16(const void *p, int64_t i) {
    return from16<T>(((const uint16_t *)p)[i]);
}

// Exponent field of a 16-bit storage type: all ones means inf or NaN.
static uint32_t expmask16(int dtype) { return dtype == Half::id ? 0x7C00u : 0x7F80u; }

template <class T>
__global__ __launch_bounds__(256) void direct_fwd_kernel(const DirectParams P, const void *x,
                                                         const void *w, void *y) {
    const int64_t total = (int64_t)P.n * P.k * P.p * P.q;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    int64_t f = idx;
    const int q = (int)(f % P.q); f /= P.q;
    const int p = (int)(f % P.p); f /= P.p;
    const int k = (int)(f % P.k); f /= P.k;
    const int n = (int)f;
    const int g = k / P.kg;
    // Taps outside the image multiply the zero of the zero-extended input
    // rather than being skipped, so a non-finite weight gives a non-finite
    // output there too, as the definition does (and as the kernels whose
    // range-checked loads return zeros do).
    float acc = 0.f;
    for (int c = 0; c < P.cg; ++c) {
        const int ci = g * P.cg + c;
        for (int r = 0; r < P.r; ++r) {
            const int h = p * P.sh - P.ph + r * P.dh;
            const bool hin = h >= 0 && h < P.h;
            for (int s = 0; s < P.s; ++s) {
                const int wv = q * P.sw - P.pw + s * P.dw;
                const bool in = hin && wv >= 0 && wv < P.w;
                const float xv =
                    in ? ld16<T>(x, n * P.xs[0] + ci * P.xs[1] + h * P.xs[2] + wv * P.xs[3]) : 0.f;
                const float fv = ld16<T>(w, k * P.wsd[0] + c * P.wsd[1] + r * P.wsd[2] + s * P.wsd[3]);
                acc += xv * fv;
            }
        }
    }
    ((uint16_t *)y)[n * P.ys[0] + k * P.ys[1] + p * P.ys[2] + q * P.ys[3]] =
        (uint16_t)to16<T>(acc * P.alpha);
}

template <class T>
__global__ __launch_bounds__(256) void direct_dgrad_kernel(const DirectParams P, const void *dy,
                                                           const void *w, void *dx) {
    const int64_t total = (int64_t)P.n * P.c * P.h * P.w;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    int64_t f = idx;
    const int j = (int)(f % P.w); f /= P.w;
    const int i = (int)(f % P.h); f /= P.h;
    const int c = (int)(f % P.c); f /= P.c;
    const int n = (int)f;
    const int g = c / P.cg;
    const int cc = c - g * P.cg;
    float acc = 0.f;
    for (int kk = 0; kk < P.kg; ++kk) {
        const int k = g * P.kg + kk;
        for (int r = 0; r < P.r; ++r) {
            const int nump = i + P.ph - r * P.dh;
            if (nump < 0 || nump % P.sh) continue;
            const int p = nump / P.sh;
            if (p >= P.p) continue;
            for (int s = 0; s < P.s; ++s) {
                const int numq = j + P.pw - s * P.dw;
                if (numq < 0 || numq % P.sw) continue;
                const int q = numq / P.sw;
                if (q >= P.q) continue;
                const float dv = ld16<T>(dy, n * P.ys[0] + k * P.ys[1] + p * P.ys[2] + q * P.ys[3]);
                const float fv = ld16<T>(w, k * P.wsd[0] + cc * P.wsd[1] + r * P.wsd[2] + s * P.wsd[3]);
                acc += dv * fv;
            }
        }
    }
    ((uint16_t *)dx)[n * P.xs[0] + c * P.xs[1] + i * P.xs[2] + j * P.xs[3]] =
        (uint16_t)to16<T>(acc * P.alpha);
}

// ws[split][k][(r*S + s)*Cg + c] = sum over the split's pixels of dy * x
template <class T>
__global__ __launch_bounds__(256) void direct_wgrad_kernel(const DirectParams P, const void *x,
                                                           const void *dy, float *ws,
                                                           int32_t splits) {
    const int64_t rscg = (int64_t)P.r * P.s * P.cg;
    const int64_t count = (int64_t)P.k * rscg;
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int split = blockIdx.y;
    if (idx >= count) return;
    const int k = (int)(idx / rscg);
    const int64_t jj = idx - (int64_t)k * rscg;
    const int tap = (int)(jj / P.cg);
    const int c = (int)(jj - (int64_t)tap * P.cg);
    const int r = tap / P.s, s = tap - (tap / P.s) * P.s;
    const int ci = (k / P.kg) * P.cg + c;
    const int64_t npq = (int64_t)P.n * P.p * P.q;
    const int64_t per = (npq + splits - 1) / splits;
    const int64_t b = split * per;
    const int64_t e = b + per < npq ? b + per : npq;
    float acc = 0.f;
    for (int64_t pix = b; pix < e; ++pix) {
        const int n = (int)(pix / ((int64_t)P.p * P.q));
        const int rm = (int)(pix - (int64_t)n * P.p * P.q);
        const int p = rm / P.q, q = rm - (rm / P.q) * P.q;
        const int h = p * P.sh - P.ph + r * P.dh;
        const int wv = q * P.sw - P.pw + s * P.dw;
        // outside the image: the zero of the zero-extended input, multiplied
        // (a non-finite dy then makes the sum non-finite, as defined)
        const bool in = h >= 0 && h < P.h && wv >= 0 && wv < P.w;
        const float xv =
            in ? ld16<T>(x, n * P.xs[0] + ci * P.xs[1] + h * P.xs[2] + wv * P.xs[3]) : 0.f;
        const float dv = ld16<T>(dy, n * P.ys[0] + k * P.ys[1] + p * P.ys[2] + q * P.ys[3]);
        acc += dv * xv;
    }
    ws[(int64_t)split * count + idx] = acc;
}

hipError_t launch_direct_fwd(int dtype, const DirectParams &p, const void *x, const void *w,
                             void *y, hipStream_t st) {
    const int64_t total = (int64_t)p.n * p.k * p.p * p.q;
    const dim3 grid((uint32_t)((total + 255) / 256));
    if (dtype == Half::id)
        hipLaunchKernelGGL(direct_fwd_kernel<Half>, grid, dim3(256), 0, st, p, x, w, y);
    else
        hipLaunchKernelGGL(direct_fwd_kernel<BFloat>, grid, dim3(256), 0, st, p, x, w, y);
    return hipGetLastError();
}

hipError_t launch_direct_dgrad(int dtype, const DirectParams &p, const void *dy, const void *w,
                               void *dx, hipStream_t st) {
    const int64_t total = (int64_t)p.n * p.c * p.h * p.w;
    const dim3 grid((uint32_t)((total + 255) / 256));
    if (dtype == Half::id)
        hipLaunchKernelGGL(direct_dgrad_kernel<Half>, grid, dim3(256), 0, st, p, dy, w, dx);
    else
        hipLaunchKernelGGL(direct_dgrad_kernel<BFloat>, grid, dim3(256), 0, st, p, dy, w, dx);
    return hipGetLastError();
}

hipError_t launch_direct_wgrad(int dtype, const DirectParams &p, const void *x, const void *dy,
                               float *ws, int32_t splits, hipStream_t st) {
    const int64_t count = (int64_t)p.k * p.r * p.s * p.cg;
    const dim3 grid((uint32_t)((count + 255) / 256), (uint32_t)splits);
    if (dtype == Half::id)
        hipLaunchKernelGGL(direct_wgrad_kernel<Half>, grid, dim3(256), 0, st, p, x, dy, ws, splits);
    else
        hipLaunchKernelGGL(direct_wgrad_kernel<BFloat>, grid, dim3(256), 0, st, p, x, dy, ws,
                           splits);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// 16-bit transforms
// ---------------------------------------------------------------------------

// A batched transpose; source rows are src_ld elements apart (>= cols).
struct T16 {
    const uint16_t *src;
    uint16_t *dst;
    int64_t rows, cols, src_ld, dst_ld, tiles_c, tiles_r;
};

// dst[b][cc][rr] = rr < rows ? src[b][rr][cc] : 0, one 64x64 tile (index t)
// through LDS.  vr: 16-byte loads (src_ld a multiple of 8, src 16-byte
// aligned; the last chunk of a row may hold padding columns); vw: 16-byte
// stores (dst_ld a multiple of 8, dst aligned).  Without them 2-byte accesses,
// all 16 of a thread in flight at once: images with an odd number of pixels
// have one such side (256 channels x 16 images of 33x45, both sides
// element-wise and a load per loop turn before: to channel-last 12.3 -> 10.5
// us, back 18.0 -> 8.6).
//
// For 16-byte stores a thread gathers 8 consecutive rows of one column; a
// wave's gather touches rows 8 apart, which share banks for any row pitch that
// keeps chunks 16-byte aligned, so chunk c of row r is stored at chunk
// c ^ ((r >> 3) & 7).  For 2-byte stores a wave reads 64 rows of a column:
// rows are 65 elements apart.
//
// SCAN: also store into flags[t] whether any element of the tile is inf or
// NaN (all exponent bits of expmask set).
constexpr int T16_LDS = 64 * 65 + 8;  // elements, 16-byte aligned

template <bool SCAN>
__device__ __forceinline__ void transpose16_tile(const T16 &p, int64_t t, bool vr, bool vw,
                                                 uint16_t *tile, uint32_t expmask, int32_t *flags) {
    const int64_t b = t / (p.tiles_c * p.tiles_r);
    const int64_t rem = t - b * p.tiles_c * p.tiles_r;
    const int64_t tr = rem / p.tiles_c, tc = rem - (rem / p.tiles_c) * p.tiles_c;
    const int64_t r0 = tr * 64, c0 = tc * 64;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const uint16_t *s = p.src + b * p.rows * p.src_ld;
    int bad = 0;
    if (vr) {
        u32x4 v[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int id = threadIdx.x + 256 * i;
            const int64_t rr = r0 + (id >> 3), col = c0 + (id & 7) * 8;
            v[i] = u32x4{};
            if (rr < p.rows && col < p.cols) v[i] = *(const u32x4 *)(s + rr * p.src_ld + col);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int id = threadIdx.x + 256 * i;
            const int row = id >> 3, cc = id & 7;
            if (vw) {
                *(u32x4 *)(&tile[row * 64 + ((cc ^ ((row >> 3) & 7)) << 3)]) = v[i];
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    tile[row * 65 + cc * 8 + e] = (uint16_t)(v[i][e >> 1] >> (16 * (e & 1)));
            }
            if constexpr (SCAN) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    bad |= ((v[i][e] & expmask) == expmask) |
                           (((v[i][e] >> 16) & expmask) == expmask);
            }
        }
    } else {
        uint16_t v[16];
        const int64_t cc = c0 + tx;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int64_t rr = r0 + ty + 4 * i;
            v[i] = rr < p.rows && cc < p.cols ? s[rr * p.src_ld + cc] : (uint16_t)0;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int row = ty + 4 * i;
            tile[vw ? row * 64 + (((tx >> 3) ^ ((row >> 3) & 7)) << 3) + (tx & 7) : row * 65 + tx] =
                v[i];
            if constexpr (SCAN) bad |= (v[i] & expmask) == expmask;
        }
    }
    if constexpr (SCAN) {
        bad = __syncthreads_or(bad);
        if (threadIdx.x == 0) flags[t] = bad;
    } else {
        __syncthreads();
    }
    uint16_t *d = p.dst + b * p.cols * p.dst_ld;
    if (vw) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int id = threadIdx.x + 256 * i;
            const int oc = id >> 3, rc = (id & 7) * 8;
            const int64_t col = c0 + oc, rr = r0 + rc;
            if (col < p.cols && rr < p.dst_ld) {
                // rows rc .. rc + 7 share (r >> 3) = rc >> 3
                const int pc = (((oc >> 3) ^ ((rc >> 3) & 7)) << 3) + (oc & 7);
                uint32_t w[4];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    w[e] = (uint32_t)tile[(rc + 2 * e) * 64 + pc] |
                           ((uint32_t)tile[(rc + 2 * e + 1) * 64 + pc] << 16);
                *(u32x4 *)(d + col * p.dst_ld + rr) = u32x4{w[0], w[1], w[2], w[3]};
            }
        }
    } else {
        const int64_t rr = r0 + tx;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int64_t col = c0 + ty + 4 * i;
            if (col < p.cols && rr < p.dst_ld) d[col * p.dst_ld + rr] = tile[tx * 65 + ty + 4 * i];
        }
    }
}

template <bool SCAN>
__global__ __launch_bounds__(256) void transpose16_kernel(const T16 p, int vr, int vw,
                                                          uint32_t expmask, int32_t *flags) {
    __shared__ __align__(16) uint16_t tile[T16_LDS];
    transpose16_tile<SCAN>(p, blockIdx.x, vr, vw, tile, expmask, flags);
}

// Both sides 16 bytes wide.
template <bool SCAN>
__global__ __launch_bounds__(256) void transpose16_vec_kernel(const T16 p, uint32_t expmask,
                                                              int32_t *flags) {
    __shared__ __align__(16) uint16_t tile[64 * 64];
    transpose16_tile<SCAN>(p, blockIdx.x, true, true, tile, expmask, flags);
}

// Two independent transposes in one launch (workgroups [0, n0) do the first,
// the rest the second): the layout copies on the input side of a channel-first
// call, one launch instead of two.  vec: bits 0, 1 of each are vr, vw.
__global__ __launch_bounds__(256) void transpose16_pair_kernel(const T16 p0, const T16 p1,
                                                               int64_t n0, int vec0, int vec1) {
    __shared__ __align__(16) uint16_t tile[T16_LDS];
    const int64_t t = blockIdx.x;
    const bool first = t < n0;
    const int vec = first ? vec0 : vec1;
    transpose16_tile<false>(first ? p0 : p1, first ? t : t - n0, vec & 1, vec & 2, tile, 0u, nullptr);
}

// Block-diagonal super-group weights: dst[k][t][c'] (c' < sg, t < rs) is
// w[k][c' - base][t] when c' lies in output channel k's own group of m
// channels (base = ((k % sg) / m) * m), else 0.  src is [K][rs][m] (kcrs = 0)
// or [K][m][rs] (kcrs = 1).
__global__ __launch_bounds__(256) void expand_group_weights_kernel(
    const uint16_t *__restrict__ src, uint16_t *__restrict__ dst, int64_t count, int32_t rs,
    int32_t m, int32_t sg, int kcrs) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= count) return;
    const int64_t per_k = (int64_t)rs * sg;
    const int64_t k = e / per_k;
    const int64_t rem = e - k * per_k;
    const int64_t t = rem / sg;
    const int64_t cp = rem - t * sg;
    const int64_t base = ((k % sg) / m) * m;
    uint16_t v = 0;
    if (cp >= base && cp < base + m) {
        const int64_t c = cp - base;
        v = kcrs ? src[(k * m + c) * rs + t] : src[(k * rs + t) * m + c];
    }
    dst[e] = v;
}

hipError_t launch_expand_group_weights(const void *src, void *dst, int64_t k, int32_t rs, int32_t m,
                                       int32_t sg, int kcrs, hipStream_t st) {
    const int64_t count = k * rs * sg;
    if (count <= 0) return hipSuccess;
    const int64_t nb = (count + 255) / 256;
    if (nb > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL(expand_group_weights_kernel, dim3((uint32_t)nb), dim3(256), 0, st,
                       (const uint16_t *)src, (uint16_t *)dst, count, rs, m, sg, kcrs);
    return hipGetLastError();
}

int64_t transpose16_blocks(int64_t batch, int64_t cols, int64_t dst_ld) {
    return batch * ((cols + 63) / 64) * ((dst_ld + 63) / 64);
}

static T16 t16(const void *src, void *dst, int64_t rows, int64_t cols, int64_t src_ld,
               int64_t dst_ld) {
    T16 p;
    p.src = (const uint16_t *)src;
    p.dst = (uint16_t *)dst;
    p.rows = rows;
    p.cols = cols;
    p.src_ld = src_ld;
    p.dst_ld = dst_ld;
    p.tiles_c = (cols + 63) / 64;
    p.tiles_r = (dst_ld + 63) / 64;
    return p;
}

// which sides take 16-byte accesses: bit 0 loads, bit 1 stores
static int t16_vec(const T16 &p) {
    return (p.src_ld % 8 == 0 && (uintptr_t)p.src % 16 == 0 ? 1 : 0) |
           (p.dst_ld % 8 == 0 && (uintptr_t)p.dst % 16 == 0 ? 2 : 0);
}

template <bool SCAN>
static hipError_t transpose16_go(const void *src, void *dst, int64_t batch, int64_t rows,
                                 int64_t cols, int64_t src_ld, int64_t dst_ld, uint32_t expmask,
                                 int32_t *flags, hipStream_t st) {
    const int64_t tiles_c = (cols + 63) / 64, tiles_r = (dst_ld + 63) / 64;
    const int64_t nb = batch * tiles_c * tiles_r;
    if (nb <= 0) return hipSuccess;
    if (nb > 0x7FFFFFFF) return hipErrorInvalidValue;
    const T16 p = t16(src, dst, rows, cols, src_ld, dst_ld);
    const int vec = t16_vec(p);
    if (vec == 3)
        hipLaunchKernelGGL(transpose16_vec_kernel<SCAN>, dim3((uint32_t)nb), dim3(256), 0, st, p,
                           expmask, flags);
    else
        hipLaunchKernelGGL(transpose16_kernel<SCAN>, dim3((uint32_t)nb), dim3(256), 0, st, p,
                           vec & 1, vec & 2, expmask, flags);
    return hipGetLastError();
}

hipError_t launch_transpose16(const void *src, void *dst, int64_t batch, int64_t rows,
                              int64_t cols, int64_t dst_ld, hipStream_t st) {
    return transpose16_go<false>(src, dst, batch, rows, cols, cols, dst_ld, 0u, nullptr, st);
}

hipError_t launch_transpose16_ld(const void *src, void *dst, int64_t batch, int64_t rows,
                                 int64_t cols, int64_t src_ld, int64_t dst_ld, hipStream_t st) {
    return transpose16_go<false>(src, dst, batch, rows, cols, src_ld, dst_ld, 0u, nullptr, st);
}

hipError_t launch_transpose16_pair(const void *src0, void *dst0, int64_t batch0, int64_t rows0,
                                   int64_t cols0, int64_t dst_ld0, const void *src1, void *dst1,
                                   int64_t batch1, int64_t rows1, int64_t cols1, int64_t dst_ld1,
                                   hipStream_t st) {
    const int64_t n0 = batch0 * ((cols0 + 63) / 64) * ((dst_ld0 + 63) / 64);
    const int64_t n1 = batch1 * ((cols1 + 63) / 64) * ((dst_ld1 + 63) / 64);
    if (n0 <= 0 || n1 <= 0 || n0 + n1 > 0x7FFFFFFF) {
        const hipError_t e = launch_transpose16(src0, dst0, batch0, rows0, cols0, dst_ld0, st);
        if (e != hipSuccess) return e;
        return launch_transpose16(src1, dst1, batch1, rows1, cols1, dst_ld1, st);
    }
    const T16 p0 = t16(src0, dst0, rows0, cols0, cols0, dst_ld0);
    const T16 p1 = t16(src1, dst1, rows1, cols1, cols1, dst_ld1);
    hipLaunchKernelGGL(transpose16_pair_kernel, dim3((uint32_t)(n0 + n1)), dim3(256), 0, st, p0, p1,
                       n0, t16_vec(p0), t16_vec(p1));
    return hipGetLastError();
}

hipError_t launch_transpose16_scan(const void *src, void *dst, int64_t batch, int64_t rows,
                                   int64_t cols, int64_t dst_ld, int dtype, int32_t *flags,
                                   hipStream_t st) {
    return transpose16_go<true>(src, dst, batch, rows, cols, cols, dst_ld, expmask16(dtype), flags,
                                st);
}

// flags[b] = whether any of the 16-bit elements [2048 b, 2048 b + 2048) of
// src[0, count) is inf or NaN.
__global__ __launch_bounds__(256) void nonfinite_scan16_kernel(const uint16_t *__restrict__ src,
                                                               int64_t count, uint32_t expmask,
                                                               int32_t *flags) {
    int bad = 0;
    const int64_t base = (int64_t)blockIdx.x * 2048;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        const int64_t e = base + u * 256 + threadIdx.x;
        if (e < count) bad |= (src[e] & expmask) == expmask;
    }
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) flags[blockIdx.x] = bad;
}

int64_t nonfinite_scan16_blocks(int64_t count) { return (count + 2047) / 2048; }

hipError_t launch_nonfinite_scan16(const void *src, int64_t count, int dtype, int32_t *flags,
                                   hipStream_t st) {
    const int64_t nb = nonfinite_scan16_blocks(count);
    if (nb <= 0) return hipSuccess;
    if (nb > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL(nonfinite_scan16_kernel, dim3((uint32_t)nb), dim3(256), 0, st,
                       (const uint16_t *)src, count, expmask16(dtype), flags);
    return hipGetLastError();
}

// Backward-data border fix-up.  The matrix-core and depthwise kernels read
// dy zero-extended at every filter tap of a stride phase, so an inf or NaN
// weight meets those zeros (0 * inf = NaN) at dx pixels whose taps leave dy
// -- terms the definition does not have.  When any weight is non-finite
// (some flag set), this kernel recomputes every such border pixel from the
// definition: rows [0, bt) and [H - bb, H), and columns [0, bl) and
// [W - br, W) of the other rows, every channel, skipping the taps outside dy.
// With all flags clear every workgroup returns at once.
template <class T>
__global__ __launch_bounds__(256) void dgrad_border_kernel(const DirectParams P, const void *dy,
                                                           const void *w, void *dx,
                                                           const int32_t *flags, int32_t nflags,
                                                           int32_t bt, int32_t bb, int32_t bl,
                                                           int32_t br) {
    int any = 0;
    for (int i = threadIdx.x; i < nflags; i += 256) any |= flags[i];
    if (!__syncthreads_or(any)) return;
    const int64_t mid = P.h - bt - bb;
    const int64_t per_img = (int64_t)(bt + bb) * P.w + mid * (bl + br);
    const int64_t total = (int64_t)P.n * per_img * P.c;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * 256) {
        const int c = (int)(e % P.c);
        int64_t f = e / P.c;
        const int64_t pix = f % per_img;
        const int n = (int)(f / per_img);
        int i, j;
        if (pix < (int64_t)bt * P.w) {
            i = (int)(pix / P.w);
            j = (int)(pix % P.w);
        } else if (pix < (int64_t)(bt + bb) * P.w) {
            const int64_t q = pix - (int64_t)bt * P.w;
            i = P.h - bb + (int)(q / P.w);
            j = (int)(q % P.w);
        } else {
            const int64_t q = pix - (int64_t)(bt + bb) * P.w;
            i = bt + (int)(q / (bl + br));
            const int u = (int)(q % (bl + br));
            j = u < bl ? u : P.w - br + (u - bl);
        }
        const int g = c / P.cg;
        const int cc = c - g * P.cg;
        float acc = 0.f;
        for (int kk = 0; kk < P.kg; ++kk) {
            const int k = g * P.kg + kk;
            for (int r = 0; r < P.r; ++r) {
                const int nump = i + P.ph - r * P.dh;
                if (nump < 0 || nump % P.sh) continue;
                const int p = nump / P.sh;
                if (p >= P.p) continue;
                for (int s = 0; s < P.s; ++s) {
                    const int numq = j + P.pw - s * P.dw;
                    if (numq < 0 || numq % P.sw) continue;
                    const int q = numq / P.sw;
                    if (q >= P.q) continue;
                    const float dv =
                        ld16<T>(dy, n * P.ys[0] + k * P.ys[1] + p * P.ys[2] + q * P.ys[3]);
                    const float fv =
                        ld16<T>(w, k * P.wsd[0] + cc * P.wsd[1] + r * P.wsd[2] + s * P.wsd[3]);
                    acc += dv * fv;
                }
            }
        }
        ((uint16_t *)dx)[n * P.xs[0] + c * P.xs[1] + i * P.xs[2] + j * P.xs[3]] =
            (uint16_t)to16<T>(acc * P.alpha);
    }
}

hipError_t launch_dgrad_border(int dtype, const DirectParams &p, const void *dy, const void *w,
                               void *dx, const int32_t *flags, int32_t nflags, int32_t bt,
                               int32_t bb, int32_t bl, int32_t br, hipStream_t st) {
    if (bt + bb == 0 && bl + br == 0) return hipSuccess;
    if (bt < 0 || bb < 0 || bl < 0 || br < 0 || bt + bb > p.h || bl + br > p.w)
        return hipErrorInvalidValue;
    const dim3 grid(256), block(256);
    if (dtype == Half::id)
        hipLaunchKernelGGL(dgrad_border_kernel<Half>, grid, block, 0, st, p, dy, w, dx, flags,
                           nflags, bt, bb, bl, br);
    else
        hipLaunchKernelGGL(dgrad_border_kernel<BFloat>, grid, block, 0, st, p, dy, w, dx, flags,
                           nflags, bt, bb, bl, br);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void pad_channels16_kernel(const uint16_t *__restrict__ src,
                                                             uint16_t *__restrict__ dst,
                                                             int64_t total, int32_t c,
                                                             int32_t c_pad) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const int64_t row = i / c_pad;
    const int ch = (int)(i - row * c_pad);
    dst[i] = ch < c ? src[row * c + ch] : (uint16_t)0;
}

// c_pad a multiple of 8 and dst 16-byte aligned: one thread builds one
// 8-channel (16-byte) chunk of the output and stores it whole.
__global__ __launch_bounds__(256) void pad_channels16_vec_kernel(const uint16_t *__restrict__ src,
                                                                 u32x4 *__restrict__ dst,
                                                                 int64_t chunks, int32_t c,
                                                                 int32_t chunks_per_row) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= chunks) return;
    const int64_t row = i / chunks_per_row;
    const int ch0 = (int)(i - row * chunks_per_row) * 8;
    const uint16_t *s = src + row * c;
    uint32_t v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int a = ch0 + 2 * u, b = a + 1;
        const uint32_t lo = a < c ? s[a] : 0u;
        const uint32_t hi = b < c ? s[b] : 0u;
        v[u] = lo | (hi << 16);
    }
    dst[i] = u32x4{v[0], v[1], v[2], v[3]};
}

// c_pad == 4 and dst 16-byte aligned: one thread builds two 4-channel
// pixels (16 bytes; the last thread of an odd row count one, 8 bytes).
__global__ __launch_bounds__(256) void pad_channels4_vec_kernel(const uint16_t *__restrict__ src,
                                                                u32x4 *__restrict__ dst,
                                                                int64_t rows, int32_t c) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t r0 = 2 * i;
    if (r0 >= rows) return;
    uint32_t v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t row = r0 + (u >> 1);
        const int a = 2 * (u & 1), b = a + 1;
        const uint16_t *sp = src + row * c;
        const uint32_t lo = row < rows && a < c ? sp[a] : 0u;
        const uint32_t hi = row < rows && b < c ? sp[b] : 0u;
        v[u] = lo | (hi << 16);
    }
    if (r0 + 1 < rows)
        dst[i] = u32x4{v[0], v[1], v[2], v[3]};
    else
        *(u32x2 *)&dst[i] = u32x2{v[0], v[1]};
}

hipError_t launch_pad_channels16(const void *src, void *dst, int64_t rows, int32_t c,
                                 int32_t c_pad, hipStream_t st) {
    const int64_t total = rows * c_pad;
    if (total <= 0) return hipSuccess;
    if (c_pad == 4 && ((uintptr_t)dst % 16) == 0) {
        const int64_t pairs = (rows + 1) / 2;
        hipLaunchKernelGGL(pad_channels4_vec_kernel, dim3((uint32_t)((pairs + 255) / 256)), dim3(256),
                           0, st, (const uint16_t *)src, (u32x4 *)dst, rows, c);
        return hipGetLastError();
    }
    if (c_pad % 8 == 0 && ((uintptr_t)dst % 16) == 0) {
        const int64_t chunks = total / 8;
        hipLaunchKernelGGL(pad_channels16_vec_kernel, dim3((uint32_t)((chunks + 255) / 256)),
                           dim3(256), 0, st, (const uint16_t *)src, (u32x4 *)dst, chunks, c,
                           c_pad / 8);
    } else {
        hipLaunchKernelGGL(pad_channels16_kernel, dim3((uint32_t)((total + 255) / 256)), dim3(256),
                           0, st, (const uint16_t *)src, (uint16_t *)dst, total, c, c_pad);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// channel padding of convolutions whose channel counts are not multiples of
// 8 (the matrix-core kernels read 8-channel chunks)
// ---------------------------------------------------------------------------

// Channel-first images of at most 8 channels (RGB, grey) to channel-last
// pixels of CP = 4 or 8 channels: dst[n][i][ch] = ch < c ? src[n][ch][i] : 0.
// A 64x64 transpose tile would leave all but c of its 64 rows idle.  A thread
// builds two neighbouring pixels from one 4-byte load per plane (PAIR: hw
// even and src 4-byte aligned; otherwise 2-byte loads) and stores them whole.
template <int CP, bool PAIR>
__global__ __launch_bounds__(256) void interleave16_kernel(const uint16_t *__restrict__ src,
                                                           uint16_t *__restrict__ dst, int64_t n,
                                                           int32_t c, int64_t hw) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 2;
    if (i >= hw) return;
    for (int64_t b = blockIdx.y; b < n; b += gridDim.y) {
        const uint16_t *s = src + b * c * hw + i;
        uint32_t lo[CP] = {}, hi[CP] = {};
#pragma unroll
        for (int ch = 0; ch < CP; ++ch) {
            if (ch < c) {
                if constexpr (PAIR) {
                    const uint32_t v = *(const uint32_t *)(s + ch * hw);
                    lo[ch] = v & 0xFFFFu;
                    hi[ch] = v >> 16;
                } else {
                    lo[ch] = s[ch * hw];
                    hi[ch] = i + 1 < hw ? s[ch * hw + 1] : (uint16_t)0;
                }
            }
        }
        uint16_t *d = dst + (b * hw + i) * CP;
#pragma unroll
        for (int ch = 0; ch < CP; ch += 4)
            *(u32x2 *)(d + ch) = u32x2{lo[ch] | (lo[ch + 1] << 16), lo[ch + 2] | (lo[ch + 3] << 16)};
        if (i + 1 < hw) {
#pragma unroll
            for (int ch = 0; ch < CP; ch += 4)
                *(u32x2 *)(d + CP + ch) =
                    u32x2{hi[ch] | (hi[ch + 1] << 16), hi[ch + 2] | (hi[ch + 3] << 16)};
        }
    }
}

hipError_t launch_interleave16(const void *src, void *dst, int64_t n, int32_t c, int64_t hw,
                               int32_t c_pad, hipStream_t st) {
    if (n <= 0 || hw <= 0) return hipSuccess;
    if (c > c_pad || (c_pad != 4 && c_pad != 8) || (uintptr_t)dst % 16 != 0)
        return hipErrorInvalidValue;
    const int64_t nb = (hw + 511) / 512;
    if (nb > 0x7FFFFFFF) return hipErrorInvalidValue;
    const dim3 grid((uint32_t)nb, (uint32_t)(n < 65535 ? n : 65535));
    const bool pair = hw % 2 == 0 && (uintptr_t)src % 4 == 0;
    const uint16_t *sp = (const uint16_t *)src;
    uint16_t *dp = (uint16_t *)dst;
    if (c_pad == 4 && pair)
        hipLaunchKernelGGL((interleave16_kernel<4, true>), grid, dim3(256), 0, st, sp, dp, n, c, hw);
    else if (c_pad == 4)
        hipLaunchKernelGGL((interleave16_kernel<4, false>), grid, dim3(256), 0, st, sp, dp, n, c, hw);
    else if (pair)
        hipLaunchKernelGGL((interleave16_kernel<8, true>), grid, dim3(256), 0, st, sp, dp, n, c, hw);
    else
        hipLaunchKernelGGL((interleave16_kernel<8, false>), grid, dim3(256), 0, st, sp, dp, n, c, hw);
    return hipGetLastError();
}

// Weights with both channel counts padded: dst is [k_pad][rs][c_pad]
// (KLAST = false, the forward operand) or [rs][c_pad][k_pad] (true, the
// backward-data operand), zero where k >= K or c >= C; element (k, c, tap)
// of src is at k * sk + c * sc + tap * st.  flags (may be null): whether any
// of the block's PW_ELEMS elements is inf or NaN.  At most 2^30 elements.
constexpr int PW_ELEMS = 512;
template <bool KLAST>
__global__ __launch_bounds__(256) void pad_weights16_kernel(
    const uint16_t *__restrict__ src, uint16_t *__restrict__ dst, int32_t kn, int32_t cn,
    FastDiv k_pad, FastDiv c_pad, FastDiv rs, uint32_t sk, uint32_t sc, uint32_t stap,
    uint32_t expmask, int32_t *flags) {
    const uint32_t count = k_pad.d * c_pad.d * rs.d;
    uint16_t v[PW_ELEMS / 256];
#pragma unroll
    for (int u = 0; u < PW_ELEMS / 256; ++u) {
        const uint32_t e = blockIdx.x * PW_ELEMS + u * 256 + threadIdx.x;
        uint32_t k, c, t;
        if constexpr (KLAST) {
            const uint32_t f = fdiv(e, k_pad);
            k = e - f * k_pad.d;
            t = fdiv(f, c_pad);
            c = f - t * c_pad.d;
        } else {
            const uint32_t f = fdiv(e, c_pad);
            c = e - f * c_pad.d;
            k = fdiv(f, rs);
            t = f - k * rs.d;
        }
        v[u] = e < count && k < (uint32_t)kn && c < (uint32_t)cn ? src[k * sk + c * sc + t * stap]
                                                                 : (uint16_t)0;
    }
    int bad = 0;
#pragma unroll
    for (int u = 0; u < PW_ELEMS / 256; ++u) {
        const uint32_t e = blockIdx.x * PW_ELEMS + u * 256 + threadIdx.x;
        if (e < count) dst[e] = v[u];
        bad |= (v[u] & expmask) == expmask;
    }
    if (flags) {
        bad = __syncthreads_or(bad);
        if (threadIdx.x == 0) flags[blockIdx.x] = bad;
    }
}

int64_t pad_weights16_blocks(int64_t k_pad, int64_t c_pad, int64_t rs) {
    return (k_pad * c_pad * rs + PW_ELEMS - 1) / PW_ELEMS;
}

hipError_t launch_pad_weights16(const void *src, void *dst, int32_t k, int32_t c, int32_t k_pad,
                                int32_t c_pad, int32_t rs, int kcrs, bool klast, int dtype,
                                int32_t *flags, hipStream_t st) {
    const int64_t nb = pad_weights16_blocks(k_pad, c_pad, rs);
    if (nb <= 0) return hipSuccess;
    if ((int64_t)k_pad * c_pad * rs > (int64_t(1) << 30)) return hipErrorInvalidValue;
    const uint32_t sk = (uint32_t)(c * rs), sc = kcrs ? rs : 1, stap = kcrs ? 1 : c;
    const uint32_t em = expmask16(dtype);
    const FastDiv dk = make_fastdiv((uint32_t)k_pad), dc = make_fastdiv((uint32_t)c_pad);
    const FastDiv dr = make_fastdiv((uint32_t)rs);
    if (klast)
        hipLaunchKernelGGL(pad_weights16_kernel<true>, dim3((uint32_t)nb), dim3(256), 0, st,
                           (const uint16_t *)src, (uint16_t *)dst, k, c, dk, dc, dr, sk, sc, stap, em,
                           flags);
    else
        hipLaunchKernelGGL(pad_weights16_kernel<false>, dim3((uint32_t)nb), dim3(256), 0, st,
                           (const uint16_t *)src, (uint16_t *)dst, k, c, dk, dc, dr, sk, sc, stap, em,
                           flags);
    return hipGetLastError();
}

// dst[rows][c] = src[rows][c_pad] without the padding channels.  A thread
// stores 8 consecutive elements of the flat result (16 bytes when dst is
// aligned for it), whatever rows they fall in.
__global__ __launch_bounds__(256) void unpad_channels16_kernel(const uint16_t *__restrict__ src,
                                                               uint16_t *__restrict__ dst,
                                                               int64_t total, FastDiv div_c,
                                                               int32_t c, int32_t c_pad, int vec) {
    const int64_t e0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
    if (e0 >= total) return;
    const uint32_t row = fdiv((uint32_t)e0, div_c);
    int32_t ch = (int32_t)((uint32_t)e0 - row * (uint32_t)c);
    int64_t at = (int64_t)row * c_pad + ch;
    uint16_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        v[u] = e0 + u < total ? src[at] : (uint16_t)0;
        ++at;
        if (++ch == c) {
            ch = 0;
            at += c_pad - c;
        }
    }
    if (vec && e0 + 8 <= total) {
        uint32_t w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) w[u] = (uint32_t)v[2 * u] | ((uint32_t)v[2 * u + 1] << 16);
        *(u32x4 *)(dst + e0) = u32x4{w[0], w[1], w[2], w[3]};
    } else {
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (e0 + u < total) dst[e0 + u] = v[u];
    }
}

// rows * c below 2^31 (the padded tensor is within the 2 GiB buffer range).
hipError_t launch_unpad_channels16(const void *src, void *dst, int64_t rows, int32_t c,
                                   int32_t c_pad, hipStream_t st) {
    const int64_t total = rows * c;
    if (total <= 0) return hipSuccess;
    if (c > c_pad || total > 0x7FFFFFFF) return hipErrorInvalidValue;
    const int64_t nb = (total + 2047) / 2048;
    hipLaunchKernelGGL(unpad_channels16_kernel, dim3((uint32_t)nb), dim3(256), 0, st,
                       (const uint16_t *)src, (uint16_t *)dst, total, make_fastdiv((uint32_t)c), c,
                       c_pad, (int)((uintptr_t)dst % 16 == 0));
    return hipGetLastError();
}

}  // namespace nnconv

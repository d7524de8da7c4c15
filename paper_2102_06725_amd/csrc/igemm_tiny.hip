// igemm_tiny.hip -- the three passes of very small convolutions in one launch
// each, straight from the caller's tensors in either layout.
//
// A layer of a few MFLOP is all launches: in channel-first layout its passes
// were 11 (two input copies, weight re-layout, GEMM, border check, output
// copy, ...), 2-6 us each, on a device that could do the arithmetic in
// nanoseconds.  Here a workgroup of 8 waves owns a 16x16 output tile and
// splits its reduction, 32 elements a step; every lane gathers its 8 elements
// of each matrix-core operand with 2-byte loads through the tensors' strides,
// so nothing is copied, transposed or padded first.  The gathers cost some 100
// instructions a step, which is why larger layers don't come here (tiny_pays).
//   forward        rows = pixels (n, p, q), columns = filters k,
//                  reduction = (r, s, c), 8 channels of one tap per chunk
//   backward-data  rows = pixels (n, i, j), columns = channels c,
//                  reduction = (r, s, k); a tile that met an inf or NaN weight
//                  is recomputed from the definition's own terms, because the
//                  zeros of taps outside dy must not meet it
//   backward-weight  rows = filters k, columns = (r, s, c), reduction =
//                  pixels, 8 neighbours of one output row per chunk; ends with
//                  the loss-scale step, no partials
// 3x3 16 -> 16 on 2 images of 16x16, channel-first: forward 10.4 -> 4.5 us,
// backward-data 14.4 -> 4.6, backward-weight 11.5 -> 9.5 (device time; 11
// launches -> 3).
#include <type_traits>

#include "launch.hpp"

namespace nnconv {

namespace tiny {

constexpr int NW = 8;

// 8 elements at p, p + stride, ...; zero past the first `n`
__device__ __forceinline__ u32x4 gather8(const uint16_t *p, int64_t stride, int n) {
    uint32_t v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = e < n ? p[e * stride] : (uint16_t)0;
    return u32x4{v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16)};
}

template <class T>
__device__ __forceinline__ bool has_nonfinite(u32x4 v) {
    constexpr uint32_t M = T::id == Half::id ? 0x7C00u : 0x7F80u;
    bool bad = false;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        bad |= (v[i] & M) == M || ((v[i] >> 16) & M) == M;
    return bad;
}

}  // namespace tiny

// PASS 0: out = y from a = x, b = w.  PASS 1: out = dx from a = dy, b = w.
// PASS 2: out = dw (type OUT: 0 fp16, 1 bf16, 2 fp32) from a = dy, b = x.
// One group.  Indices fit 32 bits (tiny_pays).
template <class T, int PASS, int OUT>
__global__ __launch_bounds__(tiny::NW * 64) void igemm_tiny_kernel(
    const DirectParams P, const uint16_t *__restrict__ a, const uint16_t *__restrict__ b, void *out,
    int tiles_n, FastDiv d0, FastDiv d1, FastDiv d2, FastDiv d3, float inv_scale, int accumulate,
    int32_t *flag) {
    using namespace tiny;
    __shared__ float part[NW][16][20];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tm = blockIdx.x / tiles_n, tn = blockIdx.x - tm * tiles_n;
    const int l16 = lane & 15, q4 = lane >> 4;
    const int row = tm * 16 + l16, col = tn * 16 + l16;

    // Chunks of the reduction.  PASS 0/1: (tap, 8 channels), d0 = chunks per
    // tap, d1 = S.  PASS 2: (n, p, 8 columns), d0 = chunks per row, d1 = P.
    const int per = (int)d0.d;
    const int chunks = PASS == 2 ? P.n * P.p * per : P.r * P.s * per;
    const int nrows = PASS == 0 ? P.n * P.p * P.q : PASS == 1 ? P.n * P.h * P.w : P.k;
    const int ncols = PASS == 0 ? P.k : PASS == 1 ? P.c : P.r * P.s * P.c;
    const bool row_ok = row < nrows, col_ok = col < ncols;

    // what the lane's row and column fix.  d2, d3: PASS 0 Q and P, PASS 1 W
    // and H (row -> pixel), PASS 2 C and S (column -> tap, channel)
    int ri = 0, rj = 0, cr = 0, cs = 0;
    int64_t a0 = 0, b0 = 0;
    if constexpr (PASS != 2) {
        const int m = row_ok ? row : 0;
        const int q1 = (int)fdiv((uint32_t)m, d2);
        const int jj = m - q1 * (int)d2.d;
        const int n = (int)fdiv((uint32_t)q1, d3);
        const int ii = q1 - n * (int)d3.d;
        if constexpr (PASS == 0) {
            ri = ii * P.sh - P.ph;
            rj = jj * P.sw - P.pw;
            a0 = n * P.xs[0];
            b0 = col * P.wsd[0];
        } else {
            ri = ii + P.ph;
            rj = jj + P.pw;
            a0 = n * P.ys[0];
            b0 = col * P.wsd[1];
        }
    } else {
        const int c1 = col_ok ? col : 0;
        const int tap = (int)fdiv((uint32_t)c1, d2);
        const int c = c1 - tap * (int)d2.d;
        const int r = (int)fdiv((uint32_t)tap, d3);
        cr = r * P.dh - P.ph;
        cs = (tap - r * (int)d3.d) * P.dw - P.pw;
        a0 = row * P.ys[1];
        b0 = c * P.xs[1];
    }

    f32x4 acc = {};
    bool bad = false;
    // chunk 4 * step + q4 of the lane, steps wave, wave + NW, ...
    for (int ch = wave * 4 + q4; ch - q4 < chunks; ch += NW * 4) {
        u32x4 va = {}, vb = {};
        if (ch < chunks) {
            const int t = (int)fdiv((uint32_t)ch, d0);
            const int o = (ch - t * per) * 8;  // first channel, or column
            const int u = (int)fdiv((uint32_t)t, d1);
            const int v = t - u * (int)d1.d;
            if constexpr (PASS == 0) {  // tap (u, v), channels o ..
                const int h = ri + u * P.dh, w = rj + v * P.dw;
                const int n = P.c - o;
                if (row_ok && (unsigned)h < (unsigned)P.h && (unsigned)w < (unsigned)P.w)
                    va = gather8(a + a0 + o * P.xs[1] + h * P.xs[2] + w * P.xs[3], P.xs[1], n);
                if (col_ok)
                    vb = gather8(b + b0 + o * P.wsd[1] + u * P.wsd[2] + v * P.wsd[3], P.wsd[1], n);
            } else if constexpr (PASS == 1) {  // tap (u, v), filters o ..
                const int nh = ri - u * P.dh, nw = rj - v * P.dw;
                const int p = nh / P.sh, q = nw / P.sw;
                const int n = P.k - o;
                if (row_ok && nh >= 0 && nw >= 0 && p * P.sh == nh && q * P.sw == nw && p < P.p &&
                    q < P.q)
                    va = gather8(a + a0 + o * P.ys[1] + p * P.ys[2] + q * P.ys[3], P.ys[1], n);
                if (col_ok) {
                    vb = gather8(b + b0 + o * P.wsd[0] + u * P.wsd[2] + v * P.wsd[3], P.wsd[0], n);
                    bad |= has_nonfinite<T>(vb);
                }
            } else {  // image u, row v, columns o ..
                const int n = P.q - o;
                if (row_ok) va = gather8(a + a0 + u * P.ys[0] + v * P.ys[2] + o * P.ys[3], P.ys[3], n);
                const int h = v * P.sh + cr;
                if (col_ok && (unsigned)h < (unsigned)P.h) {
                    const uint16_t *s = b + b0 + u * P.xs[0] + h * P.xs[2];
                    uint32_t x[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int w = (o + e) * P.sw + cs;
                        x[e] = e < n && (unsigned)w < (unsigned)P.w ? s[w * P.xs[3]] : (uint16_t)0;
                    }
                    vb = u32x4{x[0] | (x[1] << 16), x[2] | (x[3] << 16), x[4] | (x[5] << 16),
                               x[6] | (x[7] << 16)};
                }
            }
        }
        // PASS 0/1: D rows = columns of the tile (channels), D columns = pixels
        acc = PASS == 2 ? mfma16<T>(va, vb, acc) : mfma16<T>(vb, va, acc);
    }

    // part[wave][i][j]: PASS 0/1 pixel i, channel j; PASS 2 filter j, column i
    *(f32x4 *)&part[wave][l16][4 * q4] = acc;
    if constexpr (PASS == 1)
        bad = __syncthreads_or(bad);
    else
        __syncthreads();
    if (tid >= 256) return;
    // neighbouring threads store neighbouring channels (channel-last) or
    // pixels (channel-first)
    const bool cfast = PASS == 2 ? P.wsd[1] == 1 : P.ys[1] == 1;
    const int i = PASS == 2 || !cfast ? tid & 15 : tid >> 4, j = PASS == 2 || !cfast ? tid >> 4 : tid & 15;
    float v = part[0][i][j];
#pragma unroll
    for (int w = 1; w < NW; ++w) v += part[w][i][j];
    if constexpr (PASS != 2) {
        const int m = tm * 16 + i, c = tn * 16 + j;
        if (m >= nrows || c >= ncols) return;
        const int q1 = (int)fdiv((uint32_t)m, d2);
        const int jj = m - q1 * (int)d2.d;
        const int n = (int)fdiv((uint32_t)q1, d3);
        const int ii = q1 - n * (int)d3.d;
        const int64_t *os = PASS == 0 ? P.ys : P.xs;
        if (PASS == 1 && bad) {
            v = 0.f;
            for (int k = 0; k < P.k; ++k)
                for (int r = 0; r < P.r; ++r) {
                    const int nh = ii + P.ph - r * P.dh;
                    if (nh < 0 || nh % P.sh || nh / P.sh >= P.p) continue;
                    for (int s = 0; s < P.s; ++s) {
                        const int nw = jj + P.pw - s * P.dw;
                        if (nw < 0 || nw % P.sw || nw / P.sw >= P.q) continue;
                        v += from16<T>(a[n * P.ys[0] + k * P.ys[1] + nh / P.sh * P.ys[2] +
                                         nw / P.sw * P.ys[3]]) *
                             from16<T>(b[k * P.wsd[0] + c * P.wsd[1] + r * P.wsd[2] + s * P.wsd[3]]);
                    }
                }
        }
        ((uint16_t *)out)[n * os[0] + c * os[1] + ii * os[2] + jj * os[3]] =
            (uint16_t)to16<T>(v * P.alpha);
    } else {
        const int k = tm * 16 + j, c1 = tn * 16 + i;
        if (k >= nrows || c1 >= ncols) return;
        const int tap = (int)fdiv((uint32_t)c1, d2);
        const int c = c1 - tap * (int)d2.d;
        const int r = (int)fdiv((uint32_t)tap, d3);
        const int64_t o = k * P.wsd[0] + c * P.wsd[1] + r * P.wsd[2] + (tap - r * (int)d3.d) * P.wsd[3];
        v *= inv_scale;
        bool over;
        if constexpr (OUT == 2) {
            float *p = (float *)out + o;
            if (accumulate) v = *p + v;
            *p = v;
            over = !__builtin_isfinite(v);
        } else {
            using D = typename std::conditional<OUT == 0, Half, BFloat>::type;
            uint16_t *p = (uint16_t *)out + o;
            if (accumulate) v = from16<D>(*p) + v;
            const uint32_t bits = to16<D>(v) & 0xFFFFu;
            *p = (uint16_t)bits;
            over = !__builtin_isfinite(from16<D>(bits));
        }
        if (over && flag) *flag = 1;
    }
}

namespace {

struct TinyGrid {
    int64_t rows, cols, chunks, wgs, steps;
};

TinyGrid grid_of(const DirectParams &p, int pass) {
    TinyGrid g;
    const int64_t taps = (int64_t)p.r * p.s;
    g.rows = pass == 0 ? (int64_t)p.n * p.p * p.q : pass == 1 ? (int64_t)p.n * p.h * p.w : p.k;
    g.cols = pass == 0 ? p.k : pass == 1 ? p.c : taps * p.c;
    g.chunks = pass == 2 ? (int64_t)p.n * p.p * ((p.q + 7) / 8)
                         : taps * (((pass == 0 ? p.c : p.k) + 7) / 8);
    g.wgs = (g.rows + 15) / 16 * ((g.cols + 15) / 16);
    g.steps = (g.chunks + 4 * tiny::NW - 1) / (4 * tiny::NW);
    return g;
}

template <class T, int PASS, int OUT>
hipError_t go(const DirectParams &p, const void *a, const void *b, void *out, float inv_scale,
              int accumulate, int32_t *flag, hipStream_t st) {
    const TinyGrid g = grid_of(p, PASS);
    const int per = PASS == 2 ? (p.q + 7) / 8 : ((PASS == 0 ? p.c : p.k) + 7) / 8;
    const FastDiv d0 = make_fastdiv((uint32_t)per);
    const FastDiv d1 = make_fastdiv((uint32_t)(PASS == 2 ? p.p : p.s));
    const FastDiv d2 = make_fastdiv((uint32_t)(PASS == 0 ? p.q : PASS == 1 ? p.w : p.c));
    const FastDiv d3 = make_fastdiv((uint32_t)(PASS == 0 ? p.p : PASS == 1 ? p.h : p.s));
    hipLaunchKernelGGL((igemm_tiny_kernel<T, PASS, OUT>), dim3((uint32_t)g.wgs), dim3(tiny::NW * 64), 0,
                       st, p, (const uint16_t *)a, (const uint16_t *)b, out,
                       (int)((g.cols + 15) / 16), d0, d1, d2, d3, inv_scale, accumulate, flag);
    return hipGetLastError();
}

template <class T>
hipError_t go_pass(int pass, const DirectParams &p, const void *a, const void *b, void *out,
                   int out_code, float inv_scale, int accumulate, int32_t *flag, hipStream_t st) {
    if (pass == 0) return go<T, 0, T::id>(p, a, b, out, 1.f, 0, nullptr, st);
    if (pass == 1) return go<T, 1, T::id>(p, a, b, out, 1.f, 0, nullptr, st);
    if (out_code == 2) return go<T, 2, 2>(p, a, b, out, inv_scale, accumulate, flag, st);
    return go<T, 2, T::id>(p, a, b, out, inv_scale, accumulate, flag, st);
}

}  // namespace

// A step costs about 2 us whatever the layer, and from 512 workgroups (two
// rounds of four per CU's worth of waves) on they queue; against that stand the
// launches of the other path.  fast: that path needs no padded channels.  single:
// it is one launch of a matrix-core kernel for the forward pass (4.7 us), three
// for backward-data (8.8), two for backward-weight (7.8): worth 0, 3 and 2 steps;
// with the copies of channel-first layout or padded channels 10.5, 13 and 11 us:
// worth 4, 4, 3.
// Backward-weight of channel-first filters of several taps scatters its stores,
// which the split reduction's copy does not: 900 workgroups 12.9 us against 14.3
// there, 1152 16.4 against 14.0, 1250 20.0 against 13.9.
bool tiny_pays(const DirectParams &p, int pass, bool fast, bool single) {
    const TinyGrid g = grid_of(p, pass);
    if (pass == 2 && fast && p.wsd[1] > 1 && g.wgs > 1024) return false;
    const int limit = single ? (pass == 0 ? 0 : pass == 1 ? 3 : 2) : (pass == 2 ? 3 : 4);
    return g.steps * (g.wgs > 512 ? g.wgs : 512) <= (int64_t)limit * 512;
}

// Estimated time of a forward or backward-data pass here, in microseconds
// (fitted to 8000 random layers, 9% rms).
double tiny_us(const DirectParams &p, int pass) {
    const TinyGrid g = grid_of(p, pass);
    const double s = (double)g.steps, w = (double)g.wgs / 512;
    const double u = w < 1 ? w : 1, v = w > 1 ? w - 1 : 0;
    if (pass == 0) return 2.81 + s * (1.23 + 0.57 * u) + v * (0.53 + 0.65 * s);
    return 3.20 + s * (1.24 + 0.77 * u) + v * (0.35 + 1.21 * s);
}

hipError_t launch_igemm_tiny(int dtype, int pass, const DirectParams &p, const void *a,
                             const void *b, void *out, int out_code, float inv_scale,
                             int accumulate, int32_t *flag, hipStream_t st) {
    if (dtype == Half::id)
        return go_pass<Half>(pass, p, a, b, out, out_code, inv_scale, accumulate, flag, st);
    return go_pass<BFloat>(pass, p, a, b, out, out_code, inv_scale, accumulate, flag, st);
}

}  // namespace nnconv

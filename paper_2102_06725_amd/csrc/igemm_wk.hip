// igemm_wk.hip -- implicit GEMM for small grids (forward pass and every
// stride phase of backward-data): the waves of a workgroup split the
// reduction of one output tile among themselves.
//
// The large-tile kernel (igemm_c64.hip) gives each workgroup a 128-row tile
// and its whole reduction.  At small batches that leaves most CUs idle and
// every launch waits on a few long chains of load -> barrier -> multiply: a
// 3x3 layer of 512 channels over 8 images of 7x7 is 16 tiles of 4608-long
// reductions.  Here a tile is 32 or 64 pixels by 32 or 64 channels, and wave w
// of NW takes the 32-element k-steps w, w + NW, ... of it:
//   - each wave stages its own steps with buffer_load ... lds into its own
//     LDS ring, DEPTH - 1 steps ahead, so the loop has no barrier: a wave
//     waits for its own loads only.  A load instruction takes 4 lanes per row
//     (64 consecutive bytes); loading fragments straight into registers
//     touches 16 rows with 16 consecutive lanes and ran at a quarter of the
//     rate (16 bytes per clock and CU);
//   - v_mfma_f32_16x16x32 on the 64-byte rows;
//   - the NW partial tiles meet in LDS and are summed in wave order, so
//     results are reproducible.
// What bounds it is the bytes each CU draws from L2: a step moves
// (BM + BN) * 64 of them.
// 3x3 512 -> 512 on 8 images of 7x7: 57.8 -> 10.7 us (8 workgroups before, 208
// now); on one image 256 -> 256, 14x14: 29.8 -> 7.6; 1x1 2048 -> 512, 7x7,
// 8 images: 24.0 -> 6.4.
#include "launch.hpp"

namespace nnconv {

// BM pixels x BN channels per tile, NW waves, LDS ring of DEPTH steps per
// wave.  PAD: some (row, tap) pairs fall outside the A image.  MIX: cr is not
// a multiple of 32, so the four 8-channel chunks of a step may belong to
// different taps, decoded per lane.
template <class T, int BM, int BN, int NW, int DEPTH, bool PAD, bool MIX>
__global__ __launch_bounds__(NW * 64) void igemm_wk_kernel(const TNParams P) {
    constexpr int FM = BM / 16, FN = BN / 16;  // 16x16 blocks; also loads per step
    constexpr int LOADS = FM + FN;
    constexpr int STEP = (BM + BN) * 64;       // LDS bytes of a step
    constexpr int LDP = BN + 4;  // floats per partial row: 16 rows fall on distinct banks
    constexpr int RING_BYTES = NW * DEPTH * STEP, PART_BYTES = NW * BM * LDP * 4;
    __shared__ u32x4 lds[(RING_BYTES > PART_BYTES ? RING_BYTES : PART_BYTES) / 16];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    int phi = 0;
    for (int i = 1; i < P.nphase; ++i)
        if ((int)blockIdx.x >= P.ph[i].block_start) phi = i;
    const TNPhase &F = P.ph[phi];
    const int phase_blocks =
        (phi + 1 < P.nphase ? P.ph[phi + 1].block_start : (int)gridDim.x) - F.block_start;
    // row tiles fastest: the tiles of one column block, which share its
    // weights, run on one XCD
    const int local = (int)xcd_remap(blockIdx.x - F.block_start, phase_blocks);
    int g, rem;
    split_group(local, F.tiles_m * P.tiles_n, P.groups, P.group_inner, g, rem);
    const int tn = rem / F.tiles_m;
    const int tm = rem - tn * F.tiles_m;
    const int m0 = tm * BM, n0 = tn * BN;
    const int tap0 = F.tap_start, ntaps = F.tap_count;

    // block-diagonal weights (groups of 64 channels, 32-column tiles): only
    // the half of the channels that the tile's columns meet is read
    const bool diag = BN == 32 && P.diag32;
    const int cr = diag ? 32 : P.cr;
    const int half_ofs = diag ? (n0 & 32) : 0;

    const i32x4 ra = desc_of(P.a, P.a_bytes);
    const i32x4 rb = desc_of(P.b, P.b_bytes);

    // Staging role: load f fills rows f*16 + lane/4 of A (or B), physical
    // chunk lane%4, i.e. logical chunk (lane%4) ^ ((row >> 2) & 3): the 16
    // rows of a fragment read then fall in 16 distinct 16-byte bank groups.
    const int lrow = lane >> 2;
    const int lchunk = (lane & 3) ^ ((lrow >> 2) & 3);
    const uint32_t chunk = MIX ? 0u : (uint32_t)lchunk * 16u;
    uint32_t a_voff[FM];
    int a_h[FM], a_w[FM];
#pragma unroll
    for (int f = 0; f < FM; ++f) {
        const int m = m0 + f * 16 + lrow;
        if (m < F.M) {
            const int q1 = (int)fdiv((uint32_t)m, F.div_mj);
            const int jj = m - q1 * F.mj;
            const int n = (int)fdiv((uint32_t)q1, F.div_mi);
            const int ii = q1 - n * F.mi;
            a_h[f] = ii * P.ai_mul + P.ai_add;
            a_w[f] = jj * P.aj_mul + P.aj_add;
            a_voff[f] =
                (uint32_t)(((n * P.a_h + a_h[f]) * P.a_w + a_w[f]) * P.a_c + g * P.a_cg_ofs +
                           half_ofs) * 2u + chunk;
        } else {
            a_h[f] = -(1 << 24);
            a_w[f] = 0;
            a_voff[f] = OOB_OFFSET;
        }
    }
    uint32_t b_voff[FN];
#pragma unroll
    for (int f = 0; f < FN; ++f) {
        const int col = n0 + f * 16 + lrow;
        b_voff[f] = col < P.ncols ? (uint32_t)(g * P.b_g_ofs + col * P.b_ld + half_ofs) * 2u + chunk
                                  : OOB_OFFSET;
    }

    // per-tap shifts, tap t held by lane t (read back with v_readlane)
    const int tl = tap0 + (lane < ntaps ? lane : 0);
    const int v_dh = P.taps.dh[tl], v_dw = P.taps.dw[tl];
    const uint32_t v_ashift = (uint32_t)(v_dh * P.a_w + v_dw) * (uint32_t)P.a_c * 2u;
    const uint32_t v_boff = (uint32_t)P.taps.boff[tl] * 2u;

    // this wave's k-steps: wave, wave + NW, ... of the ntaps * cr / 32
    const int chunks = ntaps * (P.cr >> 3);
    const int steps = MIX ? (chunks + 3) >> 2 : ntaps * (cr >> 5);
    const int mine = steps > wave ? (steps - wave + NW - 1) / NW : 0;
    const int adv_t = (NW * 32) / cr, adv_c = (NW * 32) % cr;
    int ld_t = (wave * 32) / cr, ld_c = (wave * 32) % cr, ld_i = 0;
    const uint32_t ring = (uint32_t)(uintptr_t)(lds_void *)&lds[0] + (uint32_t)(wave * DEPTH * STEP);

    // loads of this wave's next step into ring slot s; a step past the end
    // reads zeros, which keeps the wait counts uniform
    auto load = [&](int s) {
        bool live;
        uint32_t ash, bsh;
        int dh = 0, dw = 0;
        if constexpr (MIX) {
            const int gv = (wave + ld_i * NW) * 4 + lchunk;
            live = ld_i < mine && gv < chunks;
            const int t = live ? (int)fdiv((uint32_t)gv, P.div_crv) : 0;
            const uint32_t cofs = (uint32_t)(gv - t * (P.cr >> 3)) * 16u;
            ash = (uint32_t)__shfl((int)v_ashift, t) + cofs;
            bsh = (uint32_t)__shfl((int)v_boff, t) + cofs;
            dh = __shfl(v_dh, t);
            dw = __shfl(v_dw, t);
        } else {
            live = ld_i < mine;
            const int t = live ? ld_t : 0;
            const uint32_t cofs = (uint32_t)ld_c * 2u;
            ash = (uint32_t)__builtin_amdgcn_readlane((int)v_ashift, t) + cofs;
            bsh = (uint32_t)__builtin_amdgcn_readlane((int)v_boff, t) + cofs;
            if constexpr (PAD) {
                dh = __builtin_amdgcn_readlane(v_dh, t);
                dw = __builtin_amdgcn_readlane(v_dw, t);
            }
        }
        const uint32_t base = ring + (uint32_t)(s * STEP);
#pragma unroll
        for (int f = 0; f < FM; ++f) {
            bool ok = live;
            if constexpr (PAD)
                ok = ok && (unsigned)(a_h[f] + dh) < (unsigned)P.a_h &&
                     (unsigned)(a_w[f] + dw) < (unsigned)P.a_w;
            else
                ok = ok && a_voff[f] != OOB_OFFSET;
            dma16(base + (uint32_t)f * 1024u, ok ? a_voff[f] + ash : OOB_OFFSET, ra);
        }
#pragma unroll
        for (int f = 0; f < FN; ++f)
            dma16(base + (uint32_t)(FM + f) * 1024u,
                  live && b_voff[f] != OOB_OFFSET ? b_voff[f] + bsh : OOB_OFFSET, rb);
        ++ld_i;
        ld_t += adv_t;
        ld_c += adv_c;
        if (ld_c >= cr) {
            ld_c -= cr;
            ++ld_t;
        }
    };

    f32x4 acc[FN][FM];
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int i = 0; i < FM; ++i) acc[j][i] = f32x4{};

    const int l16 = lane & 15;
    // 16-byte slot of the lane's fragment within a 16-row block
    const int fslot = l16 * 4 + ((lane >> 4) ^ ((l16 >> 2) & 3));
    if (mine > 0) {
#pragma unroll
        for (int s = 0; s < DEPTH - 1; ++s) load(s);
        const u32x4 *my = &lds[wave * (DEPTH * STEP / 16)];
        for (int it = 0; it < mine; it += DEPTH) {
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                // this step has landed once at most DEPTH - 2 later ones are
                // pending; the fragments of the previous step, whose slot is
                // loaded next, have been read
                wait_vmcnt<(DEPTH - 2) * LOADS>();
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                load((u + DEPTH - 1) % DEPTH);
                const u32x4 *st = my + u * (STEP / 16) + fslot;
                u32x4 fa[FM], fb[FN];
#pragma unroll
                for (int i = 0; i < FM; ++i) fa[i] = st[i * 64];
#pragma unroll
                for (int j = 0; j < FN; ++j) fb[j] = st[(FM + j) * 64];
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int i = 0; i < FM; ++i) acc[j][i] = mfma16<T>(fb[j], fa[i], acc[j][i]);
            }
        }
        // steps past the end may still be landing in the ring that the
        // partial tiles take over
        wait_vmcnt<0>();
    }
    __syncthreads();
    float *part = (float *)&lds[0];

    // lane holds pixel l16 of each 16-pixel block and channels
    // 4 * (lane / 16) + {0..3} of each 16-channel block
    {
        float *mp = part + wave * (BM * LDP);
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
                *(f32x4 *)(mp + (i * 16 + l16) * LDP + j * 16 + 4 * (lane >> 4)) = acc[j][i];
    }
    __syncthreads();
    uint16_t *out = (uint16_t *)P.out;
    constexpr int QPR = BN / 4;  // 4-channel quads per tile row
#pragma unroll
    for (int e0 = 0; e0 < BM * QPR; e0 += NW * 64) {
        const int e = e0 + tid;
        if (BM * QPR % (NW * 64) != 0 && e >= BM * QPR) break;
        const int r = e / QPR, ch = n0 + (e % QPR) * 4;
        const int m = m0 + r;
        if (m >= F.M || ch >= P.ncols) continue;
        const float *src = part + r * LDP + (e % QPR) * 4;
        f32x4 v = *(const f32x4 *)src;
#pragma unroll
        for (int w = 1; w < NW; ++w) v += *(const f32x4 *)(src + w * (BM * LDP));
        const int q1 = (int)fdiv((uint32_t)m, F.div_mj);
        const int jj = m - q1 * F.mj;
        const int n = (int)fdiv((uint32_t)q1, F.div_mi);
        const int ii = q1 - n * F.mi;
        const int oh = ii * P.oi_mul + F.oi_add;
        const int ow = jj * P.oj_mul + F.oj_add;
        const int64_t o =
            ((int64_t)(n * P.o_h + oh) * P.o_w + ow) * P.o_c + (int64_t)g * P.o_cg_ofs + ch;
        u32x2 pk;
        pk[0] = to16<T>(v[0] * P.alpha) | (to16<T>(v[1] * P.alpha) << 16);
        pk[1] = to16<T>(v[2] * P.alpha) | (to16<T>(v[3] * P.alpha) << 16);
        *(u32x2 *)(out + o) = pk;
    }
}

template <class T, int BM, int BN, int NW, int DEPTH>
static hipError_t launch_wk_cfg(TNParams &p, bool pad, hipStream_t st) {
    p.tiles_n = (p.ncols + BN - 1) / BN;
    int64_t nb = 0;
    for (int i = 0; i < p.nphase; ++i) {
        p.ph[i].tiles_m = (p.ph[i].M + BM - 1) / BM;
        p.ph[i].block_start = (int32_t)nb;
        nb += (int64_t)p.ph[i].tiles_m * p.tiles_n * p.groups;
    }
    if (nb <= 0) return hipSuccess;
    if (nb > 0x7FFFFFFF) return hipErrorInvalidValue;
    if (p.diag32 && (BN != 32 || p.cr != 64)) return hipErrorInvalidValue;
    const dim3 grid((uint32_t)nb), block(NW * 64);
    if (p.cr % 32 != 0)
        hipLaunchKernelGGL((igemm_wk_kernel<T, BM, BN, NW, DEPTH, true, true>), grid, block, 0, st, p);
    else if (pad)
        hipLaunchKernelGGL((igemm_wk_kernel<T, BM, BN, NW, DEPTH, true, false>), grid, block, 0, st, p);
    else
        hipLaunchKernelGGL((igemm_wk_kernel<T, BM, BN, NW, DEPTH, false, false>), grid, block, 0, st, p);
    return hipGetLastError();
}

template <class T>
static hipError_t launch_wk_t(WKConfig cfg, TNParams &p, bool pad, hipStream_t st) {
    switch (cfg) {
        case WK_32x32_4W: return launch_wk_cfg<T, 32, 32, 4, 4>(p, pad, st);
        case WK_32x32_8W: return launch_wk_cfg<T, 32, 32, 8, 4>(p, pad, st);
        case WK_64x64_4W: return launch_wk_cfg<T, 64, 64, 4, 2>(p, pad, st);
        case WK_64x64_8W:
        default: return launch_wk_cfg<T, 64, 64, 8, 2>(p, pad, st);
    }
}

hipError_t launch_igemm_wk(int dtype, WKConfig cfg, TNParams &p, bool pad, hipStream_t st) {
    if (dtype == Half::id) return launch_wk_t<Half>(cfg, p, pad, st);
    return launch_wk_t<BFloat>(cfg, p, pad, st);
}

}  // namespace nnconv

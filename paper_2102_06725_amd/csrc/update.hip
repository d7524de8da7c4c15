// update.hip -- the training-step pieces after the backward passes, kept on
// the device so a step needs no host synchronisation:
//   - dynamic loss scaling (Sec. 3.3, Listing 6) as a one-thread state
//     machine over a device-resident state and the overflow flag that the
//     backward-weight reduction sets;
//   - the fp32 master-weight update (momentum SGD with L2 weight decay),
//     which divides the loss-scaled gradient by the current scale, skips
//     itself when the flag reports an inf or NaN, and refreshes the 16-bit
//     working copy of the weights.
#include "launch.hpp"

static_assert(sizeof(nnconv_loss_scaler) == 24, "scaler state is part of the C ABI");

namespace nnconv {

__global__ __launch_bounds__(64) void loss_scaler_init_kernel(nnconv_loss_scaler *s, float scale,
                                                              float factor, int32_t interval) {
    if (threadIdx.x != 0) return;
    s->scale = scale;
    s->factor = factor;
    s->interval = interval;
    s->counter = 0;
    s->skipped = 0;
    s->reserved = 0;
}

// One step: overflow -> scale /= factor, counter = 0 (update skipped);
// otherwise grow the scale once the counter has passed the interval, then
// count the step.  The flag is cleared for the next step.
__global__ __launch_bounds__(64) void loss_scaler_update_kernel(nnconv_loss_scaler *s,
                                                                int32_t *flag) {
    if (threadIdx.x != 0) return;
    if (*flag != 0) {
        s->scale = s->scale / s->factor;
        s->counter = 0;
        s->skipped = s->skipped + 1;
    } else {
        if (s->counter > s->interval) {
            s->scale = s->scale * s->factor;
            s->counter = 0;
        }
        s->counter = s->counter + 1;
    }
    *flag = 0;
}

// g = grad / scale + wd * w;  v = mu * v + g;  w -= lr * v
__device__ __forceinline__ void sgd_one(float &w, float &v, float g, float inv_scale, float lr,
                                        float mu, float wd) {
    const float gg = g * inv_scale + wd * w;
    v = mu * v + gg;
    w = w - lr * v;
    // The 16-bit copy must be the rounding of the stored fp32 master; keep
    // the compiler from fusing the last multiply-add into the conversion
    // (a mixed-precision fma that rounds once, straight to 16 bits).
    asm volatile("" : "+v"(w));
}

// OUT: 0 writes an f16 copy of the new master, 1 a bf16 copy, -1 none.
constexpr int SGD_VECS = 2;
// VEC: 16-byte loads and stores, SGD_VECS vectors per thread.  Bound by HBM: 22
// bytes per parameter, all but the 16-bit copy (the next forward's weights)
// not touched again before the next step, so they stream past the caches.
// The data loads are issued before the flag and the scale are waited for.
// 23.45 M parameters, update and loss scaler in turn: 98.6 us with ordinary
// accesses, one vector per thread and the loads behind the flag (5.2 TB/s); 95.7
// with two vectors ahead of it, 91.9 with streaming loads too, 78.4 (6.6 TB/s)
// with streaming fp32 stores as well (83.3 when the 16-bit copy streams too).
// What they win depends on what the last-level cache holds; ordinary -> this, us, by
// parameters:
//                          3 M           12 M          23.45 M       60 M
//   back to back           9.2 -> 10.7   38.5 -> 42.4  74.2 -> 78.9  247 -> 199
//   after 1 GiB of writes  19.4 -> 15.0  61.1 -> 48.1  111 -> 90     259 -> 235
//   gradients just written 15.8 -> 14.0  46.8 -> 43.1  85.0 -> 78.7  252 -> 196
//   after 128 MB           12.1 -> 14.6  40.8 -> 43.9  82.6 -> 78.2  252 -> 196
// Neither is faster in every state; between two updates of one array a training
// step writes its gradients and more than the cache holds.
template <int OUT, bool VEC>
__global__ __launch_bounds__(256) void sgd_update_kernel(int64_t count, float *__restrict__ master,
                                                         float *__restrict__ mom,
                                                         uint16_t *__restrict__ w16,
                                                         const float *__restrict__ grad,
                                                         const nnconv_loss_scaler *state,
                                                         const int32_t *flag, float lr, float mu,
                                                         float wd) {
    using T = typename std::conditional<OUT == 1, BFloat, Half>::type;
    if constexpr (VEC) {
        const int64_t base = ((int64_t)blockIdx.x * (256 * SGD_VECS) + threadIdx.x) * 4;
        f32x4 w[SGD_VECS], v[SGD_VECS], g[SGD_VECS];
#pragma unroll
        for (int k = 0; k < SGD_VECS; ++k) {
            const int64_t i4 = base + k * 1024;
            if (i4 < count) {
                w[k] = __builtin_nontemporal_load((const f32x4 *)(master + i4));
                v[k] = __builtin_nontemporal_load((const f32x4 *)(mom + i4));
                g[k] = __builtin_nontemporal_load((const f32x4 *)(grad + i4));
            }
        }
        if (flag && *flag != 0) return;  // inf/NaN in this step's gradients: skip
        const float inv_scale = state ? 1.0f / state->scale : 1.0f;
#pragma unroll
        for (int k = 0; k < SGD_VECS; ++k) {
            const int64_t i4 = base + k * 1024;
            if (i4 >= count) return;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float wu = w[k][u], vu = v[k][u];
                sgd_one(wu, vu, g[k][u], inv_scale, lr, mu, wd);
                w[k][u] = wu;
                v[k][u] = vu;
            }
            __builtin_nontemporal_store(w[k], (f32x4 *)(master + i4));
            __builtin_nontemporal_store(v[k], (f32x4 *)(mom + i4));
            if constexpr (OUT >= 0) {
                const uint32_t b0 = to16<T>(w[k][0]) & 0xFFFFu, b1 = to16<T>(w[k][1]) & 0xFFFFu;
                const uint32_t b2 = to16<T>(w[k][2]) & 0xFFFFu, b3 = to16<T>(w[k][3]) & 0xFFFFu;
                *(u32x2 *)(w16 + i4) = u32x2{b0 | (b1 << 16), b2 | (b3 << 16)};
            }
        }
    } else {
        if (flag && *flag != 0) return;
        const float inv_scale = state ? 1.0f / state->scale : 1.0f;
        const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
        if (i >= count) return;
        float w = master[i], v = mom[i];
        sgd_one(w, v, grad[i], inv_scale, lr, mu, wd);
        master[i] = w;
        mom[i] = v;
        if constexpr (OUT >= 0) w16[i] = (uint16_t)to16<T>(w);
    }
}

hipError_t launch_loss_scaler_init(nnconv_loss_scaler *s, float scale, float factor,
                                   int32_t interval, hipStream_t st) {
    hipLaunchKernelGGL(loss_scaler_init_kernel, dim3(1), dim3(64), 0, st, s, scale, factor,
                       interval);
    return hipGetLastError();
}

hipError_t launch_loss_scaler_update(nnconv_loss_scaler *s, int32_t *flag, hipStream_t st) {
    hipLaunchKernelGGL(loss_scaler_update_kernel, dim3(1), dim3(64), 0, st, s, flag);
    return hipGetLastError();
}

template <int OUT>
static void launch_sgd_out(int64_t count, float *master, float *mom, uint16_t *w16,
                           const float *grad, const nnconv_loss_scaler *state, const int32_t *flag,
                           float lr, float mu, float wd, hipStream_t st) {
    const bool vec = count % 4 == 0 && (uintptr_t)master % 16 == 0 && (uintptr_t)mom % 16 == 0 &&
                     (uintptr_t)grad % 16 == 0 && (OUT < 0 || (uintptr_t)w16 % 8 == 0);
    if (vec) {
        const int64_t nb = (count / 4 + 256 * SGD_VECS - 1) / (256 * SGD_VECS);
        hipLaunchKernelGGL((sgd_update_kernel<OUT, true>), dim3((uint32_t)nb), dim3(256), 0, st,
                           count, master, mom, w16, grad, state, flag, lr, mu, wd);
    } else {
        const int64_t nb = (count + 255) / 256;
        hipLaunchKernelGGL((sgd_update_kernel<OUT, false>), dim3((uint32_t)nb), dim3(256), 0, st,
                           count, master, mom, w16, grad, state, flag, lr, mu, wd);
    }
}

hipError_t launch_sgd_update(int64_t count, float *master, float *mom, void *w16, int w16_dtype,
                             const float *grad, const nnconv_loss_scaler *state, const int32_t *flag,
                             float lr, float mu, float wd, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    if ((count + 255) / 256 > 0x7FFFFFFF) return hipErrorInvalidValue;
    uint16_t *o = (uint16_t *)w16;
    if (!o)
        launch_sgd_out<-1>(count, master, mom, o, grad, state, flag, lr, mu, wd, st);
    else if (w16_dtype == BFloat::id)
        launch_sgd_out<1>(count, master, mom, o, grad, state, flag, lr, mu, wd, st);
    else
        launch_sgd_out<0>(count, master, mom, o, grad, state, flag, lr, mu, wd, st);
    return hipGetLastError();
}

}  // namespace nnconv

// ECG misfit (Sec. 2.4 Eq. (inverse_ecg), rectangle rule in time) and the Adam
// update used to fit the model parameters (Sec. 2.4).
#include <math.h>

#include <algorithm>

#include "gbp_internal.h"

namespace {

// Misfit and its gradient of instance blockIdx.x.  The sum is one block's, in a fixed
// order (deterministic), eight strides of loads at a time; from kLossSplit entries on
// its other blocks write the gradient.  One CU's loads are the bound:
// 62,000 entries 8.8 us (one stride at a time, one block for both: 22.8 us).
constexpr int kLossSplit = 8192;

__global__ void __launch_bounds__(1024)
    k_loss(const float* __restrict__ e_all, const float* __restrict__ t_all, int n,
           float* __restrict__ loss, float* __restrict__ grad_all) {
    __shared__ float sh[1024];
    const size_t base = (size_t)blockIdx.x * n;
    const float* e = e_all + base;
    const float* t = t_all + base;
    const float inv = 1.f / (float)n;
    if (blockIdx.y > 0) {
        for (size_t i = (blockIdx.y - 1) * 1024u + threadIdx.x; i < (size_t)n; i += (gridDim.y - 1) * 1024u)
            grad_all[base + i] = 2.f * (e[i] - t[i]) * inv;
        return;
    }
    float* grad = grad_all && gridDim.y == 1 ? grad_all + base : nullptr;
    float acc = 0.f;
    for (size_t i0 = threadIdx.x; i0 < (size_t)n; i0 += 8 * 1024) {
        float a[8], b[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const size_t i = i0 + u * 1024, at = i < (size_t)n ? i : 0;   // no branch: all loads in flight
            a[u] = e[at];
            b[u] = t[at];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const size_t i = i0 + u * 1024;
            const float d = i < (size_t)n ? a[u] - b[u] : 0.f;
            acc += d * d;
            if (grad && i < (size_t)n) grad[i] = 2.f * d * inv;
        }
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss[blockIdx.x] = sh[0] * inv;
}

// Blocks of an instance; one if the gradient overwrites what the sum reads.
int loss_blocks(const float* e, const float* t, const float* grad, int n_inst, int n) {
    const size_t all = (size_t)n_inst * n;
    if (!grad || n < kLossSplit || (grad < e + all && e < grad + all) || (grad < t + all && t < grad + all)) return 1;
    return 1 + std::min(n / 4096 + 1, 128);
}

// Adam with the step number in device memory (bias corrections computed here).
__global__ void k_adam_dev(float* __restrict__ p, const float* __restrict__ g,
                           float* __restrict__ m, float* __restrict__ v, int n, float lr, float b1,
                           float b2, float eps, const int* __restrict__ step, float lo, float hi,
                           int clamp) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float k = (float)max(*step, 1);
    const float c1 = 1.f / (1.f - powf(b1, k));
    const float c2 = 1.f / (1.f - powf(b2, k));
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    float x = p[i] - lr * (mi * c1) / (sqrtf(vi * c2) + eps);
    if (clamp) x = fminf(fmaxf(x, lo), hi);
    p[i] = x;
}

__global__ void k_counter_add(int* c, int d) {
    if (threadIdx.x == 0) *c += d;
}

__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, int n, float lr, float b1, float b2, float eps,
                       float c1, float c2, float lo, float hi, int clamp) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    float x = p[i] - lr * (mi * c1) / (sqrtf(vi * c2) + eps);
    if (clamp) x = fminf(fmaxf(x, lo), hi);
    p[i] = x;
}

}  // namespace

extern "C" int gbp_ecg_loss(const float* ecg, const float* target, int n, float* loss,
                            float* dL_decg, void* stream) {
    if (!ecg || !target || !loss || n <= 0) {
        gbp_set_error("ecg_loss: bad arguments");
        return GBP_ERR_ARG;
    }
    k_loss<<<dim3(1, loss_blocks(ecg, target, dL_decg, 1, n)), 1024, 0, (hipStream_t)stream>>>(ecg, target, n, loss, dL_decg);
    GBP_LAUNCH_CHECK();
    return GBP_OK;
}

extern "C" int gbp_adam_step(float* param, const float* grad, float* m, float* v, int n, float lr,
                             float beta1, float beta2, float eps, int step, float lo, float hi,
                             void* stream) {
    if (!param || !grad || !m || !v || n < 0 || step < 1) {
        gbp_set_error("adam_step: bad arguments");
        return GBP_ERR_ARG;
    }
    if (n == 0) return GBP_OK;
    const float c1 = (float)(1.0 / (1.0 - pow((double)beta1, step)));
    const float c2 = (float)(1.0 / (1.0 - pow((double)beta2, step)));
    k_adam<<<gbp_blocks(n, 256), 256, 0, (hipStream_t)stream>>>(param, grad, m, v, n, lr, beta1,
                                                                beta2, eps, c1, c2, lo, hi,
                                                                lo < hi ? 1 : 0);
    GBP_LAUNCH_CHECK();
    return GBP_OK;
}

extern "C" int gbp_ecg_loss_batched(const float* ecg, const float* target, int n_inst, int n_per,
                                    float* loss, float* dL_decg, void* stream) {
    if (!ecg || !target || !loss || n_inst < 1 || n_per < 1) {
        gbp_set_error("ecg_loss_batched: bad arguments");
        return GBP_ERR_ARG;
    }
    k_loss<<<dim3(n_inst, loss_blocks(ecg, target, dL_decg, n_inst, n_per)), 1024, 0, (hipStream_t)stream>>>(
        ecg, target, n_per, loss, dL_decg);
    GBP_LAUNCH_CHECK();
    return GBP_OK;
}

extern "C" int gbp_adam_step_dev(float* param, const float* grad, float* m, float* v, int n,
                                 float lr, float beta1, float beta2, float eps, const int* step,
                                 float lo, float hi, void* stream) {
    if (!param || !grad || !m || !v || !step || n < 0) {
        gbp_set_error("adam_step_dev: bad arguments");
        return GBP_ERR_ARG;
    }
    if (n == 0) return GBP_OK;
    k_adam_dev<<<gbp_blocks(n, 256), 256, 0, (hipStream_t)stream>>>(param, grad, m, v, n, lr, beta1,
                                                                    beta2, eps, step, lo, hi,
                                                                    lo < hi ? 1 : 0);
    GBP_LAUNCH_CHECK();
    return GBP_OK;
}

extern "C" int gbp_counter_add(int* counter, int delta, void* stream) {
    if (!counter) {
        gbp_set_error("counter is NULL");
        return GBP_ERR_ARG;
    }
    k_counter_add<<<1, 64, 0, (hipStream_t)stream>>>(counter, delta);
    GBP_LAUNCH_CHECK();
    return GBP_OK;
}

// Internal interface of the warm-start network kernels (64 channels).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

namespace sgtv {
namespace wsn {

// out = relu(conv(X) + bias)
hipError_t conv_relu(const __bf16 *X, const __bf16 *Wk, const float *bias, int B, int H, __bf16 *out, hipStream_t st);
// z = conv(X) + bias (FP32, or nullptr); sp (or nullptr): softplus(z); 16-byte aligned
hipError_t conv_softplus(const __bf16 *X, const __bf16 *Wk, const float *bias, int B, int H, float *z, float *sp,
                         hipStream_t st);
// out = conv(X) masked by mask > 0
hipError_t conv_masked(const __bf16 *X, const __bf16 *Wk, int B, int H, const __bf16 *mask, __bf16 *out,
                       hipStream_t st);
// blocks of the weight gradient of B images of H rows
int wgrad_blocks(int B, int H);
// weight and bias gradient of one layer into grad (C*9*C weights, then C biases);
// wpart: wgrad_blocks(B, H) * (C*9*C + C) floats of scratch
hipError_t conv_wgrad(const __bf16 *X, const __bf16 *DZ, int B, int H, float *wpart, float *grad, hipStream_t st);
// FP32 arrays below are 16-byte aligned, n and img multiples of 8
hipError_t to_bf16(const float *x, __bf16 *y, int64_t n, hipStream_t st);
// per-image FP64 partial sums (n_blocks per image, image-major)
hipError_t image_partials(const float *x, int64_t img, int n_images, int n_blocks, double *partials,
                          hipStream_t st);
// y = bf16(x / m_b), m_b = sums[b] / img (1 where not positive), b = i / img
hipError_t scale_to_bf16(const float *x, const double *sums, int64_t img, int n_images, __bf16 *y, hipStream_t st);
// x0 = c_out * s * (ratio ? f : m_b), raised to at least floor * c_out * m_b when floor > 0
// (x0 may be f)
hipError_t start_image(const float *f, const float *s, const double *sums, int64_t img, int n_images, float c_out,
                       int ratio, float floor, float *x0, hipStream_t st);
// dz = bf16(2 (softplus(z) - target) / n * sigmoid(z)), FP64 squared-error partials
hipError_t mse_grad(const float *target, const float *z, int64_t n, __bf16 *dz, double *partials,
                    int n_blocks, hipStream_t st);
// acc[0] += l[0] / cnt, acc[1] += 1 (FP64, one thread)
hipError_t loss_accumulate(const double *l, double cnt, double *acc, hipStream_t st);
hipError_t adam(float *p, const float *g, float *m, float *v, int64_t n, float lr, float b1,
                float b2, float omb1, float omb2, float eps, float c1, float c2, hipStream_t st);
hipError_t weights_bf16(const float *w, __bf16 *wf, __bf16 *wb, hipStream_t st);

}  // namespace wsn
}  // namespace sgtv

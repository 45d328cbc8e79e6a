// mlp.h -- the schedule-predicting network (shared by host and kernels).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "internal.h"

namespace hicr {

constexpr int kMlpIn = 32, kMlpHidden = 64, kMlpOut = 12;
constexpr int kMlpParams = kMlpHidden * kMlpIn + kMlpHidden + kMlpHidden * kMlpHidden +
                           kMlpHidden + kMlpOut * kMlpHidden + kMlpOut;  // 7,052
static_assert(kMlpParams == 7052, "parameter count");

// Activations and gradients of one mini-batch of B samples (device).
struct MlpBufs {
  float *h1, *h2;       // activations
  float *dz, *d2, *d1;  // gradients w.r.t. the logits and the two layers' pre-activations
  float *loss;          // per-sample loss
};
constexpr size_t kMlpBufFloats = 4 * kMlpHidden + kMlpOut + 1;  // per sample

// logits z[B][12]
hipError_t mlp_forward(const float *params, const float *X, uint32_t B, float *z, hipStream_t s);
// gradient of the mean loss (and the mean loss, if loss_mean)
hipError_t mlp_grad(const MlpBufs &m, const float *params, const float *X, const int32_t *y,
                    uint32_t B, float *grad, float *loss_mean, hipStream_t s);
// the t-th Adam step on that gradient (mo, ve: its moments)
hipError_t mlp_step(const MlpBufs &m, float *params, float *mo, float *ve, const float *X,
                    const int32_t *y, uint32_t B, float lr, int t, float *loss_mean,
                    hipStream_t s);

// Host mirror of the histogram feature: bin floor(log2 s) capped at 31,
// size 0 in bin 0; feature log2(1 + count).
void batch_features(const uint64_t *sizes, uint64_t n, size_t stride_bytes, float *out32);

}  // namespace hicr

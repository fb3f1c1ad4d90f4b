// Cost-model network kernels (mlp.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace qtn {

constexpr int kMlpIn = 16, kMlpHidden = 64, kMlpOut = 4;
constexpr int kMlpParams = kMlpIn * kMlpHidden + kMlpHidden + kMlpHidden * kMlpHidden +
                           kMlpHidden + kMlpHidden * kMlpOut + kMlpOut;

// Device buffers carved from one workspace for a batch of n samples.
struct MlpBuffers {
  float *params, *grad, *m1, *m2;  // parameters, gradient, Adam moments
  float *x, *t, *m;                // inputs [n][16], targets and mask [n][4]
  float *y;                        // outputs [n][4]
  float *part;                     // partial gradients, one per block of a pass
  float *loss;                     // kMlpLosses entries
  size_t bytes;
};

constexpr int kMlpLosses = 64;

// Layout for n samples starting at ws (ws == nullptr: sizes only); params to
// m are one contiguous range.
MlpBuffers mlp_buffers(void *ws, int64_t n);

hipError_t mlp_forward(const MlpBuffers &b, int n, hipStream_t s);
// Forward, loss (masked mean squared error) and the full gradient.
hipError_t mlp_loss_grad(const MlpBuffers &b, int n, hipStream_t s);
// One epoch of training: the gradient, then an Adam step (as mlp_adam) with
// it; the loss before the step goes to *loss.
hipError_t mlp_train_step(const MlpBuffers &b, int n, int step, float lr, float *loss,
                          hipStream_t s);
// One Adam step with b.grad (beta1 0.9, beta2 0.999, eps 1e-8) at step >= 1.
hipError_t mlp_adam(const MlpBuffers &b, int step, float lr, hipStream_t s);

}  // namespace qtn

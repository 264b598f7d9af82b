// The proposer's network: sizes, parameter layout and launchers (see mlp.hip).
#pragma once

#include "common.h"

namespace bbl {

constexpr int kMlpIn = 28, kMlpHid = 128, kMlpOut = 10;
constexpr int kMlpSkip = 18;      // first P_D amplitude among the inputs (residual form)
constexpr int kMlpParams = 38026;

// out[r][0..10) for all rows of the bf16 features F
void mlp_forward(const float *params, const uint16_t *F, int64_t rows, float *out, hipStream_t s);

// He-uniform hidden layers, zero output layer and biases
void mlp_init(float *params, uint64_t key, hipStream_t s);

// Gradient and loss of the mean squared error over `rows` rows, in a scratch
// of mlp_grad_bytes(rows); loss may be null.
size_t mlp_grad_bytes(int64_t rows);
void mlp_grad(const float *params, const uint16_t *F, const float *T, int64_t rows, void *ws,
              float *grad, float *loss, hipStream_t s);

void mlp_adam(float *p, float *m, float *v, const float *g, int64_t count, int step, float lr,
              float b1, float b2, float eps, hipStream_t s);

// One Adam step (0.9, 0.999, 1e-8) on `batch` rows sampled from `total`.
size_t mlp_train_bytes(int64_t batch);
void mlp_train_step(float *params, float *m, float *v, int step, float lr, const uint16_t *F,
                    const float *T, int64_t total, int64_t batch, uint64_t key, void *ws,
                    float *loss, hipStream_t s);

}  // namespace bbl

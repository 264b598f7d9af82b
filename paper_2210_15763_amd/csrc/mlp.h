// The proposer's network: sizes, parameter layout and launchers (see mlp.hip).
#pragma once

#include "common.h"

namespace bbl {

constexpr int kMlpIn = 28, kMlpHid = 128, kMlpOut = 10;
constexpr int kMlpSkip = 18;      // first P_D amplitude among the inputs (residual form)
constexpr int kMlpParams = 38026;

// out[r][0..10) for all rows of the bf16 features F
void mlp_forward(const float *params, const uint16_t *F, int64_t rows, float *out, hipStream_t s);

}  // namespace bbl

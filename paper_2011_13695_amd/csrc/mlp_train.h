// The fused forward/backward pass of the training step (mlp_train.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace mdgmi {

struct TrainPass {
    const float* x;        // features [n][in0], or null: formed from y and snr_db
    const float* y;        // [n][in0 - 1]
    const float* snr_db;   // [n]
    const float* target;   // [n][out] target LLRs
    int64_t n;
    int in0, out;
    const __bf16* w[4];    // weights: layer 0 in the order of fused_offset, others of train_w_offset (mlp_layout.h)
    const __bf16* wt[4];   // transposed, in the order of train_wt_offset
    const float* b[4];
    __bf16* ht[4];         // inputs of every layer, [in][n]
    __bf16* dt[4];         // gradients at every layer's output, [out][n]
    double* lpart;         // loss sums of the blocks [train_pass_blocks(n)]
};

int train_pass_blocks(int64_t n);
hipError_t launch_train_pass(const TrainPass& a, hipStream_t st);

}  // namespace mdgmi

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
    // inputs of every layer and gradients at every layer's output, as operands
    // of v_mfma_f32_32x32x16_bf16 with the samples as the contraction: [16-sample
    // block][32-feature tile][lane][8], lane 32 h + r holding samples 8 h .. 8 h + 7
    // of the tile's feature r; features past the layer's and samples past n
    // are there (the former zero, the latter with zero gradients)
    __bf16* ht[4];
    __bf16* dt[4];
    float* dsum[4];        // sums of dt over eight samples at a time [2 blocks][width rounded up to 32]
    double* lpart;         // loss sums of the blocks [train_pass_blocks(n)]
};

struct TrainDwLayer {
    const __bf16 *dt, *ht;
    float* part;           // [slice][out][in]
    int out, in, ot, it;   // widths, and their 32-feature tiles
};

struct TrainDw {
    TrainDwLayer layer[4];
    int first[5];          // first 64 x 64 tile of each layer, and their total
    int64_t blocks;        // 16-sample blocks
    int64_t steps;         // of them per slice
};

int train_pass_blocks(int64_t n);
hipError_t launch_train_dw(const TrainDw& s, int slices, hipStream_t st);
hipError_t launch_train_pass(const TrainPass& a, hipStream_t st);

}  // namespace mdgmi

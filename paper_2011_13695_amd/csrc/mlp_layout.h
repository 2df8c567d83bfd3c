// Weight layout of the fused MLP inference kernel, shared by the kernel
// that builds it whole and the Adam step that updates it in place.
//
// Layer l's weights W [out][in] become [out tile][K-block][lane][8] bf16
// (32-row output tiles, 16-input K-blocks, 64 lanes of 8 values): lane
// holds row 32 t + (lane & 31) and, in lane half h = lane >> 5, eight of
// the block's sixteen inputs. Layer 0 takes inputs 8h .. 8h + 7 in order;
// later layers take {4h .. 4h + 3, 8 + 4h .. 8 + 4h + 3}, the order in
// which the previous layer's MFMA output lands in a lane's registers, so
// that activations go from accumulator to operand without a shuffle.
// Each layer is scaled by a power of two: 1/4 for layer 0 (the hidden
// accumulators hold x / 4), 4 for the output layer (it reads GELU / 4).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace mdgmi {
namespace fused {

// input (within its 16-input block) of slot i of lane half h, layers >= 1
__host__ __device__ inline int perm_in(int h, int i) { return i < 4 ? 4 * h + i : 8 + 4 * h + (i - 4); }

__host__ __device__ inline float layer_scale(int l) { return l == 0 ? 0.25f : l == 3 ? 4.0f : 1.0f; }

// bf16 element offset of W[o][k] of layer l (in inputs) in the layout
__host__ __device__ inline int64_t fused_offset(int l, int o, int k, int in) {
    const int n_kb = (in + 15) / 16, kb = k / 16, r = k % 16;
    int h, slot;
    if (l == 0) {
        h = r / 8;
        slot = r % 8;
    } else if (r < 8) {  // perm_in(h, slot) = 4 h + slot
        h = r / 4;
        slot = r % 4;
    } else {             // perm_in(h, slot) = 8 + 4 h + slot - 4
        h = (r - 8) / 4;
        slot = 4 + (r - 8) % 4;
    }
    const int lane = 32 * h + o % 32;
    return (((int64_t)(o / 32) * n_kb + kb) * 64 + lane) * 8 + slot;
}

// Weights as the training pass reads them (mlp_train.hip): a matrix [rows][K]
// as A operands of v_mfma_f32_16x16x32_bf16, [16-row tile][K / 32 step][lane][8],
// lane 16 g + r holding row r's k = 8 g .. 8 g + 7 of the step: natural order, so
// that the products accumulate as on the layer-by-layer path, bit for bit.
__host__ __device__ inline int64_t operand_offset(int row, int k, int steps) {
    return (((int64_t)(row / 16) * steps + k / 32) * 64 + k % 32 / 8 * 16 + row % 16) * 8 + k % 8;
}

// For the fused shape: W_l of layers 1..3 (rows = outputs, 8 steps), and W_l^T of
// layers 1..3 (rows = inputs; 8 steps, the output layer's at most 32 outputs
// one step, zero past the last). Layer 0's W^T has no use there (row-major).
constexpr int kTrainW3Elems = 32 * 256, kTrainWt3Elems = 256 * 32;
__host__ __device__ inline int64_t train_w_offset(int o, int k) { return operand_offset(o, k, 8); }
__host__ __device__ inline int64_t train_wt_offset(int l, int o, int k, int out) {
    return l == 0 ? (int64_t)k * out + o : operand_offset(k, o, l == 3 ? 1 : 8);
}

}  // namespace fused
}  // namespace mdgmi

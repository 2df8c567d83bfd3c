// Forward and backward pass of the MLP demapper's training step for networks
// [in <= 16, 256, 256, 256, out <= 32], one launch.
//
// A block takes 16 samples through all layers and back: activations and
// back-propagated gradients go from layer to layer through LDS (bf16, the
// rounding points of the layer-by-layer path), the pre-activations that GELU'
// needs stay in the registers of the lanes that formed them, and only the
// transposed copies [features][n] that the weight gradients contract over are
// written out. Each layer is H^T = W H_prev^T (backward: D_prev^T = W^T D^T) on
// v_mfma_f32_16x16x32_bf16, weights as the A operand straight from L2 (a lane's
// operand is 16 consecutive bytes of a row), samples as the columns: wave w of
// eight owns features 32 w .. 32 w + 31, two 16-row tiles, in every hidden
// layer, forward and backward, so that Z meets its gradient in place. The 64
// registers of a layer's weights are loaded one layer ahead.
//
// Sixteen samples per block because a step is small: 4096 samples are 256
// blocks, one per CU. What bounds it is the weights' way from L2 (520 KB per
// block, 64 bytes per cycle and CU at best: 8 k of its ~30 k cycles) and the chain of
// nine dependent stages, not the 2.2 GFLOP. 4096 samples of 9-256-256-256-11: 17
// us, and 34 us for the whole step of three launches (115 us and 20 launches
// layer by layer).
#include "device_common.h"
#include "f64_math.h"
#include "mlp_gemm.h"
#include "mlp_train.h"

namespace mdgmi {

namespace {

using mlp::bf16x8;
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kS = 16;          // samples per block
constexpr int kH = 256;         // hidden width
constexpr int kP = kH + 8;      // LDS pitch of an activation row (bf16)
constexpr int kPs = 40;         // ... of the narrow ones (features, output gradients)

union Q8 {
    bf16x8 v;
    uint4 u;
    __bf16 h[8];
};
union Q4 {
    uint2 u;
    __bf16 h[4];
};

// A operands of this wave's two row tiles of a 256 x 256 layer (mlp_layout.h):
// 1 KiB per load and wave.
__device__ __forceinline__ void load_w(const __bf16* __restrict__ W, int wave, int lane, bf16x8 (&w)[2][8]) {
#pragma unroll
    for (int t = 0; t < 2; t++)
#pragma unroll
        for (int k = 0; k < 8; k++) w[t][k] = *(const bf16x8*)(W + (uint32_t)((((2 * wave + t) * 8 + k) * 64 + lane) * 8));
}

// The matching B operand of step k from an activation row.
__device__ __forceinline__ bf16x8 load_b(const __bf16* __restrict__ src, int col, int g, int k) {
    return *(const bf16x8*)(src + col * kP + 32 * k + 8 * g);
}

__device__ __forceinline__ void mfma_layer(const bf16x8 (&w)[2][8], const __bf16* __restrict__ src, int col, int g,
                                           f32x4 (&acc)[2]) {
#pragma unroll
    for (int k = 0; k < 8; k++) {
        const bf16x8 b = load_b(src, col, g, k);
#pragma unroll
        for (int t = 0; t < 2; t++) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[t][k], b, acc[t], 0, 0, 0);
    }
}

// A lane's four consecutive features of its sample.
__device__ __forceinline__ void put4(__bf16* dst, int col, int f, const float* v) {
    Q4 q;
#pragma unroll
    for (int r = 0; r < 4; r++) q.h[r] = (__bf16)v[r];
    *(uint2*)(dst + col * kP + f) = q.u;
}

// The block's tile [16 samples][32 tiles features] in src (pitch p) as operands
// of the weight-gradient products (TrainPass), 1 KiB per feature tile: thread
// (f, h) stores samples 8 h .. 8 h + 7 of feature f. Samples past n are part of
// it: their gradients are zero.
// Returns their sum, in order.
__device__ __forceinline__ float store_t(const __bf16* __restrict__ src, int p, int f, int h, __bf16* __restrict__ dst,
                                         int tiles) {
    Q8 q;
#pragma unroll
    for (int j = 0; j < 8; j++) q.h[j] = src[(8 * h + j) * p + f];
    *(uint4*)(dst + (((int64_t)blockIdx.x * tiles + f / 32) * 64 + 32 * h + f % 32) * 8) = q.u;
    float s = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; j++) s += (float)q.h[j];
    return s;
}

__global__ __launch_bounds__(512) void k_train_pass(TrainPass a) {
    __shared__ __attribute__((aligned(16))) __bf16 sx[kS * kPs], sd[kS * kPs], sA[kS * kP], sB[kS * kP];
    __shared__ float sz[kS * 33];
    __shared__ uint4 sw4[1024];  // the output layer's weights
    __shared__ double red[8];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, g = lane >> 4, f0 = 32 * wave;
    const int64_t n = a.n, s0 = (int64_t)blockIdx.x * kS;
    const int in0 = a.in0, out = a.out;
    const int tf = threadIdx.x & (kH - 1), th = threadIdx.x >> 8;  // store_t's feature and half
    double loss = 0.0;
    bf16x8 wA[2][8], wB[2][8];
    load_w(a.w[1], wave, lane, wA);
    // ---- features (K padded to 32 with zeros): one per thread
    {
        const int s = threadIdx.x >> 5, f = threadIdx.x & 31;
        const int64_t i = s0 + s;
        float v = 0.0f;
        if (i < n && f < in0) {
            if (a.x)
                v = a.x[i * in0 + f];
            else if (f < in0 - 1)
                v = a.y[i * (in0 - 1) + f];
            else  // in FP64 like the host-side scalar feature
                v = (float)(((double)a.snr_db[i] - 9.5) / 4.5);
        }
        sx[s * kPs + f] = (__bf16)v;
    }
    // this thread's element of the loss: sample and output
    const int ls = threadIdx.x >> 5, lk = threadIdx.x & 31;
    const int64_t li = s0 + ls;
    const bool lok = li < n && lk < out;
    const float target = lok ? a.target[li * out + lk] : 0.0f;
#pragma unroll
    for (int q = 0; q < 2; q++) sw4[512 * q + threadIdx.x] = ((const uint4*)a.w[3])[512 * q + threadIdx.x];
    f32x4 z1[2], z2[2], z3[2], acc[2];
    bf16x8 w1[2], w4[2];
#pragma unroll
    for (int t = 0; t < 2; t++) {
        // layer 1 (its copy is scaled by 1/4, and so are bias and result here:
        // exact powers of two) has 16 inputs, lane groups 0 and 1
        Q8 q;
        q.u = make_uint4(0u, 0u, 0u, 0u);
        if (g < 2) q.u = *(const uint4*)(a.w[0] + (uint32_t)((wave * 64 + 32 * g + 16 * t + col) * 8));
        w1[t] = q.v;
        w4[t] = *(const bf16x8*)(a.wt[3] + (uint32_t)(((2 * wave + t) * 64 + lane) * 8));
        z1[t] = 0.25f * *(const f32x4*)(a.b[0] + f0 + 16 * t + 4 * g);
        z2[t] = *(const f32x4*)(a.b[1] + f0 + 16 * t + 4 * g);
        z3[t] = *(const f32x4*)(a.b[2] + f0 + 16 * t + 4 * g);
    }
    auto gelu_out = [&](const f32x4 (&z)[2], __bf16* dst) {
#pragma unroll
        for (int t = 0; t < 2; t++) {
            float v[4];
#pragma unroll
            for (int r = 0; r < 4; r++) v[r] = mlp::gelu_f(z[t][r]);
            put4(dst, col, f0 + 16 * t + 4 * g, v);
        }
    };
    auto grad_out = [&](const f32x4 (&z)[2], __bf16* dst) {
#pragma unroll
        for (int t = 0; t < 2; t++) {
            float v[4];
#pragma unroll
            for (int r = 0; r < 4; r++) v[r] = acc[t][r] * mlp::gelu_grad_f(z[t][r]);
            put4(dst, col, f0 + 16 * t + 4 * g, v);
        }
    };
    __syncthreads();
    // ---- layer 1
    if (threadIdx.x < 64) (void)store_t(sx, kPs, threadIdx.x & 31, threadIdx.x >> 5, a.ht[0], 1);
    {
        const bf16x8 b = *(const bf16x8*)(sx + col * kPs + 8 * g);
#pragma unroll
        for (int t = 0; t < 2; t++) z1[t] = 4.0f * __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1[t], b, z1[t], 0, 0, 0);
    }
    load_w(a.w[2], wave, lane, wB);
    gelu_out(z1, sA);
    __syncthreads();
    // ---- layer 2
    mfma_layer(wA, sA, col, g, z2);
    (void)store_t(sA, kP, tf, th, a.ht[1], 8);
    load_w(a.wt[2], wave, lane, wA);
    gelu_out(z2, sB);
    __syncthreads();
    // ---- layer 3
    mfma_layer(wB, sB, col, g, z3);
    (void)store_t(sB, kP, tf, th, a.ht[2], 8);
    load_w(a.wt[1], wave, lane, wB);
    gelu_out(z3, sA);
    __syncthreads();
    // ---- layer 4: logits, 16 rows per wave
    (void)store_t(sA, kP, tf, th, a.ht[3], 8);
    if (16 * wave < out) {
        f32x4 z4;
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int o = 16 * wave + 4 * g + r;
            z4[r] = o < out ? a.b[3][o] : 0.0f;
        }
#pragma unroll
        for (int k = 0; k < 8; k++) {
            Q8 q;
            q.u = sw4[(wave * 8 + k) * 64 + lane];
            z4 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(q.v, load_b(sA, col, g, k), z4, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; r++) sz[col * 33 + 16 * wave + 4 * g + r] = z4[r];
    }
    __syncthreads();
    // ---- loss and its gradient: (sigmoid(z) - sigmoid(lambda)) / n
    const float zl = sz[ls * 33 + lk];
    const float pl = 1.0f / (1.0f + expf(-target));
    {
        const float q = 1.0f / (1.0f + expf(-zl));
        const __bf16 d = lok ? (__bf16)((q - pl) / (float)n) : (__bf16)0.0f;
        sd[ls * kPs + lk] = d;
    }
    __syncthreads();
    // ---- gradients of the hidden layers, last to first
    if (threadIdx.x < 64)
        a.dsum[3][2 * (int64_t)blockIdx.x * 32 + threadIdx.x] =
            store_t(sd, kPs, threadIdx.x & 31, threadIdx.x >> 5, a.dt[3], 1);
    {
        const bf16x8 b = *(const bf16x8*)(sd + col * kPs + 8 * g);
#pragma unroll
        for (int t = 0; t < 2; t++)
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w4[t], b, (f32x4){0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
    }
    grad_out(z3, sB);
    if (lok) {
        const double sp = (zl > 0.0f ? (double)zl : 0.0) +
                          f64::ln1p_pos(f64::exp_neg((double)fabsf(zl), f64::exp_scale_unit()));
        loss = sp - (double)pl * (double)zl;
        if (!(zl == zl)) loss = NAN;
    }
    __syncthreads();
    acc[0] = acc[1] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
    mfma_layer(wA, sB, col, g, acc);
    a.dsum[2][(2 * (int64_t)blockIdx.x + th) * kH + tf] = store_t(sB, kP, tf, th, a.dt[2], 8);
    grad_out(z2, sA);
    __syncthreads();
    acc[0] = acc[1] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
    mfma_layer(wB, sA, col, g, acc);
    a.dsum[1][(2 * (int64_t)blockIdx.x + th) * kH + tf] = store_t(sA, kP, tf, th, a.dt[1], 8);
    grad_out(z1, sB);
    __syncthreads();
    a.dsum[0][(2 * (int64_t)blockIdx.x + th) * kH + tf] = store_t(sB, kP, tf, th, a.dt[0], 8);
    // loss partial: a fixed tree per wave, then the waves in order
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) loss += __shfl_down(loss, off, 64);
    if (lane == 0) red[wave] = loss;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < 8; w++) s += red[w];
        a.lpart[blockIdx.x] = s;
    }
}

// Weight gradients of all layers, one wave per 64 x 64 tile of a layer's dW
// [out][in] and slice of samples: dW = sum_s D[s][o] H[s][i] on
// v_mfma_f32_32x32x16_bf16, both operands as the pass stored them, 1 KiB
// contiguous per load, straight into registers (four of them per four MFMAs,
// eight steps ahead: what the pass wrote comes from memory, not from this
// die's L2, and a slice of 16 steps is two such trips). The general GEMM on row-major copies, through LDS, took
// 10.4 us for these 640 tiles of 4096 samples; this 9.5 us, and the pass that
// no longer scatters 32-byte pieces into rows 17.4 instead of 23.6 us.
__global__ __launch_bounds__(64) void k_train_dw(TrainDw s) {
    int l = 0;
    while ((int)blockIdx.y >= s.first[l + 1]) l++;
    const TrainDwLayer L = s.layer[l];
    const int t = blockIdx.y - s.first[l], nx = (L.it + 1) / 2, by = t / nx, bx = t % nx;
    const int lane = threadIdx.x;
    const int64_t k0 = (int64_t)blockIdx.x * s.steps, left = s.blocks - k0;
    const int nk = (int)(left < s.steps ? left : s.steps);  // >= 1
    // a layer's only tile stands in for the second one (not stored)
    const int o1 = 2 * by + 1 < L.ot ? 2 * by + 1 : 2 * by, i1 = 2 * bx + 1 < L.it ? 2 * bx + 1 : 2 * bx;
    const __bf16* pa0 = L.dt + ((k0 * L.ot + 2 * by) * 64 + lane) * 8;
    const __bf16* pa1 = L.dt + ((k0 * L.ot + o1) * 64 + lane) * 8;
    const __bf16* pb0 = L.ht + ((k0 * L.it + 2 * bx) * 64 + lane) * 8;
    const __bf16* pb1 = L.ht + ((k0 * L.it + i1) * 64 + lane) * 8;
    const int sa = L.ot * 512, sb = L.it * 512;
    constexpr int kAhead = 8;
    bf16x8 a[kAhead][2], b[kAhead][2];
    auto fetch = [&](int u, int k) {  // past the slice: its last step again, unused
        const int64_t q = k < nk ? k : nk - 1;
        a[u][0] = *(const bf16x8*)(pa0 + q * sa);
        a[u][1] = *(const bf16x8*)(pa1 + q * sa);
        b[u][0] = *(const bf16x8*)(pb0 + q * sb);
        b[u][1] = *(const bf16x8*)(pb1 + q * sb);
    };
    mlp::f32x16 acc[2][2] = {};
    auto product = [&](int u) {
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
            for (int j = 0; j < 2; j++)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[u][i], b[u][j], acc[i][j], 0, 0, 0);
    };
#pragma unroll
    for (int u = 0; u < kAhead; u++) fetch(u, u);
    int k = 0;
    for (; k + kAhead < nk; k += kAhead) {
#pragma unroll
        for (int u = 0; u < kAhead; u++) {
            product(u);
            fetch(u, k + kAhead + u);
        }
    }
#pragma unroll
    for (int u = 0; u < kAhead; u++)
        if (k + u < nk) product(u);  // uniform
    // lane holds rows 8 (r >> 2) + 4 (lane >> 5) + (r & 3) of column lane & 31
    float* C = L.part + (int64_t)blockIdx.x * L.out * L.in;
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) {
            if ((i == 1 && o1 == 2 * by) || (j == 1 && i1 == 2 * bx)) continue;
            const int c = 32 * (2 * bx + j) + (lane & 31);
            if (c >= L.in) continue;
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const int o = 32 * (2 * by + i) + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                if (o < L.out) C[o * L.in + c] = acc[i][j][r];
            }
        }
}

}  // namespace

int train_pass_blocks(int64_t n) { return (int)((n + kS - 1) / kS); }

hipError_t launch_train_dw(const TrainDw& s, int slices, hipStream_t st) {
    hipLaunchKernelGGL(k_train_dw, dim3((unsigned)slices, (unsigned)s.first[4]), dim3(64), 0, st, s);
    return hipGetLastError();
}

hipError_t launch_train_pass(const TrainPass& a, hipStream_t st) {
    hipLaunchKernelGGL(k_train_pass, dim3((unsigned)train_pass_blocks(a.n)), dim3(512), 0, st, a);
    return hipGetLastError();
}

}  // namespace mdgmi

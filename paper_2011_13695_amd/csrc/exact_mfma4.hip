// Per-SNR kernels of the per-sample 4x4-block MFMA demapper for small
// constellations (the arithmetic is in small_core.h).
#include <algorithm>
#include <atomic>

#include "small_core.h"

namespace mdgmi {

namespace {

using namespace small;

// largest formats served: at these sizes the shape still beat 32 x 32 tiles
// (4-D M = 512: 0.339 against 0.355 ms; 8-D M = 256: 0.232 against 0.264 ms
// for 2^22 samples)
constexpr int kSmallMaxM = 512, kSmallMaxM8 = 256;

// Least waves per SIMD to compile for: the formats of 256 register rows stand within
// ten registers of the 128 that four waves leave (4-D M = 256 hard decisions of
// 3 x 10^6 samples: 166 us with three, 159 with four).
constexpr int small_waves(int dim, int ng) { return dim * ng == 256 && dim < 8 ? 4 : 1; }

// Each block makes the format's A operands itself, in LDS (at most 16 KiB): a slot
// or two a thread, once, as the launch is one resident round of blocks. A kernel
// of its own for the images cost a launch per call: 16-QAM calls of 1000 samples
// 17.5 us, LLRs of them 13.6 us (a good part of either on the host); without it
// 13.7 and 10.1 us.
template <int DIM, int NG, int MODE>
__global__ __launch_bounds__(kSmallThreads, small_waves(DIM, NG)) void k_small(const float* __restrict__ y,
                                                         const uint32_t* __restrict__ tx,
                                                         const double* __restrict__ X64, const float* __restrict__ X32,
                                                         const uint32_t* __restrict__ labels, int64_t n, SnrArgs sa,
                                                         float max_n2, float* __restrict__ llr,
                                                         double* __restrict__ part) {
    constexpr int NK = Nk4<DIM>::value;
    constexpr int M = 4 * NG;
    // the wave index is uniform: keep the batch loop on the scalar unit
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q_snr = blockIdx.y;
    const float s = sa.s32[q_snr];
    const int64_t snr = sa.snr0 + q_snr;
    __shared__ uint2 img[M * NK];
    for (int j = threadIdx.x; j < M; j += kSmallThreads) image_slot<DIM>(X64, sa.s64[q_snr], j, img + j * NK);
    __syncthreads();
    const float* ys = y + snr * n * DIM;
    const uint32_t* txs = mode_is_llr(MODE) ? nullptr : tx + snr * n;
    half4 a[Sets<NG>::value][NK];
    load_image<DIM, NG>(img, M, a);
    CostAcc acc;
    HdAcc hd;
    const float guard = mode_is_llr(MODE) ? llr_guard(s, max_n2) : 0.0f;
    const int waves = kSmallThreads / 64;
    const int64_t nbat = (n + 63) / 64;
    // wave-uniform loop over batches of 64 consecutive samples
    const int64_t step = (int64_t)gridDim.x * waves;
    int64_t b = (int64_t)blockIdx.x * waves + wave;
    SampleIn<DIM> in = load_sample<DIM, MODE>(ys, txs, b * 64 + lane, n);
    for (; b < nbat; b += step) {
        const SampleIn<DIM> next = load_sample<DIM, MODE>(ys, txs, (b + step) * 64 + lane, n);
        small_sample<DIM, NG, MODE>(a, img, in, b * 64 + lane, n, s, X32, labels, llr, acc, hd, guard);
        in = next;
    }
    double* dst = part + ((int64_t)q_snr * gridDim.x + blockIdx.x) * (MODE == kModeHd ? kNPartHd : kNPart);
    if (MODE == kModeGmi || MODE == kModeMlGmi) block_reduce_store(acc, dst);
    if (MODE == kModeHd) block_reduce_store_hd(acc, hd, dst);
}

template <int DIM, int NG>
hipError_t launch_small_t(const mdgmi_format* f, const float* y, const uint32_t* tx, int64_t n, const SnrArgs& sa,
                          int mode, float* llr, double* part, int blocks, hipStream_t st) {
    const dim3 grid(blocks, sa.n_snr), block(kSmallThreads);
#define MDGMI_SMALL(MD)                                                                                      \
    hipLaunchKernelGGL((k_small<DIM, NG, MD>), grid, block, 0, st, y, tx, f->d_X64, f->d_X32,               \
                       MD == kModeHd ? f->d_labels_hd : f->d_labels, n, sa, (float)f->max_norm2, llr, part); \
    break;
    switch (mode) {
        case kModeLlr:
            MDGMI_SMALL(kModeLlr)
        case kModeHd:
            MDGMI_SMALL(kModeHd)
        case kModeMlLlr:
            MDGMI_SMALL(kModeMlLlr)
        case kModeMlGmi:
            MDGMI_SMALL(kModeMlGmi)
        default:
            MDGMI_SMALL(kModeGmi)
    }
#undef MDGMI_SMALL
    return hipGetLastError();
}

template <int DIM>
hipError_t launch_small_d(const mdgmi_format* f, const float* y, const uint32_t* tx, int64_t n, const SnrArgs& sa,
                          int mode, float* llr, double* part, int blocks, hipStream_t st) {
    switch (f->M) {
        case 4:
            return launch_small_t<DIM, 1>(f, y, tx, n, sa, mode, llr, part, blocks, st);
        case 8:
            return launch_small_t<DIM, 2>(f, y, tx, n, sa, mode, llr, part, blocks, st);
        case 16:
            return launch_small_t<DIM, 4>(f, y, tx, n, sa, mode, llr, part, blocks, st);
        case 32:
            return launch_small_t<DIM, 8>(f, y, tx, n, sa, mode, llr, part, blocks, st);
        case 64:
            return launch_small_t<DIM, 16>(f, y, tx, n, sa, mode, llr, part, blocks, st);
        case 128:
            return launch_small_t<DIM, 32>(f, y, tx, n, sa, mode, llr, part, blocks, st);
        case 256:
            return launch_small_t<DIM, 64>(f, y, tx, n, sa, mode, llr, part, blocks, st);
        default:
            if constexpr (DIM < 8) {
                if (f->M == 512) return launch_small_t<DIM, 128>(f, y, tx, n, sa, mode, llr, part, blocks, st);
            }
            return hipErrorInvalidValue;
    }
}

template <int DIM, int NG>
const void* small_kernel_t(int mode) {
    switch (mode) {
        case kModeLlr: return (const void*)k_small<DIM, NG, kModeLlr>;
        case kModeHd: return (const void*)k_small<DIM, NG, kModeHd>;
        case kModeMlLlr: return (const void*)k_small<DIM, NG, kModeMlLlr>;
        case kModeMlGmi: return (const void*)k_small<DIM, NG, kModeMlGmi>;
        default: return (const void*)k_small<DIM, NG, kModeGmi>;
    }
}

template <int DIM>
const void* small_kernel_d(int M, int mode) {
    switch (M) {
        case 4: return small_kernel_t<DIM, 1>(mode);
        case 8: return small_kernel_t<DIM, 2>(mode);
        case 16: return small_kernel_t<DIM, 4>(mode);
        case 32: return small_kernel_t<DIM, 8>(mode);
        case 64: return small_kernel_t<DIM, 16>(mode);
        case 128: return small_kernel_t<DIM, 32>(mode);
        case 256: return small_kernel_t<DIM, 64>(mode);
        default:
            if constexpr (DIM < 8) return small_kernel_t<DIM, 128>(mode);
            return nullptr;
    }
}

}  // namespace

bool small_shape_fits(const mdgmi_format* f) {
    const int M = f->M;
    return M >= 4 && (M & (M - 1)) == 0 && (f->dim < 8 ? M <= kSmallMaxM : M <= kSmallMaxM8) &&
           (f->dim == 1 || f->dim == 2 || f->dim == 4 || f->dim == 8);
}

// Blocks of (dim, M, mode)'s kernel that a CU holds, from its registers; asked
// of the runtime once. 0 if the format is not served.
static int small_blocks_per_cu(int dim, int M, int mode) {
    static std::atomic<int> cache[4][8][5];
    int lm = 0;
    while ((4 << lm) < M) lm++;
    const int ld = dim == 1 ? 0 : dim == 2 ? 1 : dim == 4 ? 2 : 3;
    if (lm > 7 || mode < 0 || mode > 4) return 0;
    std::atomic<int>& c = cache[ld][lm][mode];
    int v = c.load(std::memory_order_relaxed);
    if (v == 0) {
        const void* k = nullptr;
        switch (dim) {
            case 1: k = small_kernel_d<1>(M, mode); break;
            case 2: k = small_kernel_d<2>(M, mode); break;
            case 4: k = small_kernel_d<4>(M, mode); break;
            default: k = small_kernel_d<8>(M, mode); break;
        }
        if (!k || hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, k, kSmallThreads, 0) != hipSuccess || v < 1) v = 4;
        v = std::min(v, 8);
        c.store(v, std::memory_order_relaxed);
    }
    return v;
}

// One resident round of blocks over the launch's SNR points, as many per CU as
// the kernel's registers allow (3 to 8). Four per CU for every format left the
// light ones waiting on their loads and dependent operations: 64-QAM LLRs of
// 2^22 samples 58 us with four, 55 so (52.9 since the images are made here); 16-QAM
// hard decisions, 41 points of 131071 samples, 60 us with four in launches of 32
// and 9 points, 42.5 so in one launch (39.2 since, with max_u). Calls of very many
// points keep four, and with it the partial sums they had room for.
int64_t small_blocks(const mdgmi_format* f, int n_snr, int mode) {
    const int per_cu = small_blocks_per_cu(f->dim, f->M, mode);
    return (int64_t)device_cu_count() * (n_snr <= 8 * kMaxSnrPerLaunch ? per_cu : std::min(per_cu, 4));
}

int64_t small_want(int64_t n) { return (n + kSmallThreads - 1) / kSmallThreads; }

LaunchCfg small_cfg(const mdgmi_format* f, int64_t n, int n_snr, int mode) {
    const int64_t want = small_want(n);
    int64_t per = std::max<int64_t>(1, small_blocks(f, n_snr, mode) / snr_per_launch(n_snr, kMaxSnrSmall));
    per = std::min<int64_t>(per, std::max<int64_t>(1, want));
    LaunchCfg c;
    c.threads = kSmallThreads;
    c.blocks_per_snr = (int)per;
    return c;
}

hipError_t launch_small(const mdgmi_format* f, const float* y, const uint32_t* tx, int64_t n, const SnrArgs& sa,
                        int mode, float* llr, double* part, LaunchCfg cfg, hipStream_t st) {
    if (!small_shape_fits(f)) return hipErrorInvalidValue;
    const int b = cfg.blocks_per_snr;
    switch (f->dim) {
        case 1:
            return launch_small_d<1>(f, y, tx, n, sa, mode, llr, part, b, st);
        case 2:
            return launch_small_d<2>(f, y, tx, n, sa, mode, llr, part, b, st);
        case 4:
            return launch_small_d<4>(f, y, tx, n, sa, mode, llr, part, b, st);
        default:
            return launch_small_d<8>(f, y, tx, n, sa, mode, llr, part, b, st);
    }
}

}  // namespace mdgmi

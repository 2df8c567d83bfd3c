// FP32 exact demapper with the distance term on the matrix cores: per-SNR
// kernels over one format (see mfma_core.h for the arithmetic and layouts).
#include <algorithm>
#include <cmath>

#include "mfma_kernels.h"

namespace mdgmi {

namespace {

using namespace mfma;

struct MfmaVariant {
    int ncol, waves;
    bool lds;
};

int g_variant_override = -1;  // set through mdgmi_set_tuning for sweeps

constexpr int kNumVariants = 8;  // 32 x 32 shapes; kSmallVariant follows them
const MfmaVariant kVariants[kNumVariants] = {{1, 4, true},  {2, 4, true},  {1, 8, true},  {2, 8, true},
                                             {1, 16, true}, {1, 12, true}, {1, 16, false}, {1, 8, false}};

int blocks_of(int dim, int split) {
    if (split == kSplitBF16) return (6 * dim + 6 + 15) / 16;
    return dim == 8 ? 2 : 1;
}

size_t image_bytes_per_snr(const mdgmi_format* f, int split = kSplitF16) {
    int ntiles = (f->M + 31) / 32;
    return (size_t)ntiles * blocks_of(f->dim, split) * 64 * sizeof(uint4);
}

bool bf16_wide(const mdgmi_format* f, int split) {
    return split == kSplitBF16 && f->dim > 1 && image_bytes_per_snr(f, split) > 128 * 1024;
}


// 32 x 32 launch shape for a launch of `total` samples over its SNR points.
int pick_variant(const mdgmi_format* f, int64_t total) {
    if (g_variant_override >= 0 && g_variant_override < kNumVariants) return g_variant_override;
    const int t = tuned_mfma_variant(f->dim, f->M, total);
    if (t >= 0 && t < kNumVariants) return t;
    // untuned: a large image leaves room for one block per CU, so 16 waves
    // per block fill the CU; small images run several 8-wave blocks per CU
    return image_bytes_per_snr(f) > 32 * 1024 ? 4 : 2;
}

// The per-sample 4x4 shape serves small fp16-split formats unless a 32 x 32
// variant is asked for (override or tuning table).
bool use_small(const mdgmi_format* f, int split, int64_t total) {
    if (split != kSplitF16 || !small_shape_fits(f)) return false;
    int v = g_variant_override;
    if (v < 0 || v >= kMfmaVariants) v = tuned_mfma_variant(f->dim, f->M, total);
    return v < 0 || v >= kMfmaVariants || v == kSmallVariant;
}

const MfmaVariant& shape_of(int var) {
    static const MfmaVariant wide{2, 8, false};
    return var < 0 ? wide : kVariants[var];
}

// Waves of 32 x 32 shape v that a CU holds, by the registers of its kernels (as
// the compiler reports them): two-column shapes 153 to 256, those of sixteen
// waves are held to 128, the others up to 122 for GMI of 1 to 4 dimensions and up
// to 170 otherwise.
int shape_waves(const mdgmi_format* f, const MfmaVariant& v, int mode) {
    if (v.ncol == 2) return 8;
    if (v.waves == 16 || (mode == kModeGmi && f->dim <= 4 && v.lds)) return 16;
    return 12;
}

// Blocks over all CUs of 32 x 32 shape var: per CU as the LDS image (160 KiB) and
// the waves (cu_waves) allow.
int64_t shape_blocks(const mdgmi_format* f, int split, int var, int cu_waves) {
    const MfmaVariant& v = shape_of(var);
    const size_t img = image_bytes_per_snr(f, split);
    const bool lds = v.lds && img <= 128 * 1024;
    const int by_lds = lds ? std::max(1, (int)((160 * 1024) / (img + 2048))) : 8;
    const int by_waves = std::max(1, cu_waves / v.waves);
    return (int64_t)device_cu_count() * std::min(by_lds, by_waves);
}

// Launch configuration of 32 x 32 shape var (-1: the bf16 split's
// two-column L2 shape).
LaunchCfg shape_cfg(const mdgmi_format* f, int64_t n, int n_snr, int mode, int split, int var) {
    const MfmaVariant& v = shape_of(var);
    const int64_t cols = 32 * v.ncol;
    const int64_t tiles = (n + cols - 1) / cols;
    const int snr_in_launch = snr_per_launch(n_snr);
    // blocks whose waves all have a tile, up to sixteen waves per CU
    const int64_t full = std::min((tiles + v.waves - 1) / v.waves, shape_blocks(f, split, var, 16) / snr_in_launch);
    // a launch of few samples takes a block per column tile as far as they fit
    // beside each other: the tiles go to the blocks in turn, a wave or two of each
    // has work, and a SIMD with one busy wave is through its tile in a third of the
    // time. By the launch's points, not the call's: 8-D M = 2048, 40 points of 700
    // samples (two launches of 440 tiles) 98 us with sixteen tiles per block, 56 us
    // so. Blocks that do not fit would be a second round of part blocks: 8-D M = 2048
    // in the bf16 split (two columns, 256 registers), 313 column tiles, LLRs 57 us, and
    // 10 ms with samples on the per-class path; so 34 us and 5.1 ms (eight tiles
    // per block: 49 us and 5.3 ms).
    const int64_t beside = shape_blocks(f, split, var, shape_waves(f, v, mode)) / snr_in_launch;
    // Blocks whose waves all have work may run behind each other: they take the
    // points in order, so that fewer images share an L2 (the same format, 16
    // points of 10^6 samples: 5.6 ms, 6.2 in one round).
    const int64_t per = std::max<int64_t>(1, std::max(full, std::min(beside, tiles)));
    LaunchCfg c;
    c.threads = v.waves * 64;
    c.blocks_per_snr = (int)per;
    c.variant = var;
    return c;
}

}  // namespace

bool mfma_supported(const mdgmi_format* f, double max_s, int split) {
    // fp16 range of the split factors: 2 s |x| and s ||x||^2 must stay well
    // inside 65504 (the per-sample term K is checked in the kernel's range
    // through the far-point path). bf16 has the FP32 exponent range.
    if (split == kSplitBF16) return std::isfinite(max_s) && std::isfinite(f->max_norm2);
    return 2.0 * max_s * f->max_abs < 30000.0 && max_s * f->max_norm2 < 30000.0;
}

size_t mfma_image_bytes(const mdgmi_format* f, int n_snr, int split) {
    // (the 4x4 shape needs none, but the choice follows tuning: either may run)
    return (size_t)n_snr * image_bytes_per_snr(f, split);
}

// Blocks of a launch of the kernel that splits a tile's points: two per CU, one
// where a block is sixteen waves (M = 4096: all a CU holds at 128 registers).
static int64_t split_blocks(const mdgmi_format* f) {
    return (int64_t)device_cu_count() * (f->M > 2048 ? 1 : 2);
}

// Column tiles of a launch (over its SNR points) up to which the points are
// split: two per CU. 8-D M = 2048, two points of 1500 samples (94 column tiles): the
// call 24 us with a wave per tile, 19 us split (48 us with sixteen tiles per block).
// LLRs only with a block for each tile: one wave of a block ends its tile, and
// samples that take the per-class path there (2.5 ms at M = 2048) wait for each
// other: M = 2048, 28 dB, 257 to 512 tiles, two per block 5.0 ms, with a wave per
// tile or two blocks per CU 2.5 ms.
static bool split_points(const mdgmi_format* f, int mode, int64_t n, int n_snr) {
    const int64_t most = mode_is_llr(mode) ? split_blocks(f) : (int64_t)device_cu_count() * 2;
    return !mode_is_ml(mode) && (f->M + 31) / 32 >= 16 && (n + 31) / 32 * snr_per_launch(n_snr) <= most;
}

LaunchCfg mfma_cfg(const mdgmi_format* f, int64_t n, int n_snr, int mode, int split) {
    const int64_t total = n * (int64_t)n_snr;
    if (use_small(f, split, total)) {
        LaunchCfg c = small_cfg(f, n, n_snr, mode);
        c.variant = kSmallVariant;
        return c;
    }
    if (bf16_wide(f, split)) return shape_cfg(f, n, n_snr, mode, split, -1);
    // hard decisions, max-log metrics, 1-D formats and the bf16 split run the
    // 1-column, 16-wave shape only (LDS image if it fits)
    const bool fixed = mode == kModeHd || mode_is_ml(mode) || f->dim == 1 || split == kSplitBF16;
    const int var = fixed ? (image_bytes_per_snr(f, split) <= 128 * 1024 ? 4 : 6) : pick_variant(f, total);
    LaunchCfg c = shape_cfg(f, n, n_snr, mode, split, var);
    const bool forced = g_variant_override >= 0 && g_variant_override < kNumVariants;
    c.split_points = split == kSplitF16 && !forced && split_points(f, mode, n, n_snr);
    if (c.split_points)
        c.blocks_per_snr = (int)std::max<int64_t>(1, std::min((n + 31) / 32, split_blocks(f) / snr_per_launch(n_snr)));
    return c;
}

// A call over k points takes k times max(1, min(T / L, w)) blocks: T the blocks of
// a launch, L the points of one (at least k over the launches), w the column
// tiles or batches of a point. For k up to n_snr that is at most max(n_snr,
// min(launches T, n_snr w)), which grows with n_snr and n. (Counting k by k for
// every shape took 20 us of host time at 16 points and 44 us at 64, beside
// 14 us for the launches.)
int64_t mfma_blocks_bound(const mdgmi_format* f, int64_t n, int n_snr, int mode, int split) {
    auto bound = [&](int limit, int64_t blocks, int64_t want) {
        return std::max<int64_t>(n_snr, std::min((n_snr + limit - 1) / limit * blocks, n_snr * want));
    };
    int64_t b = 0;
    for (int v = -1; v < kNumVariants; v++)
        b = std::max(b, bound(kMaxSnrPerLaunch, shape_blocks(f, split, v, 16), (n + 31) / 32));
    if (split == kSplitF16) b = std::max(b, bound(kMaxSnrPerLaunch, split_blocks(f), (n + 31) / 32));
    if (split == kSplitF16 && small_shape_fits(f))
        b = std::max(b, bound(kMaxSnrSmall, small_blocks(f, 1, mode), small_want(n)));
    return b;
}

template <int S>
hipError_t image_and_run(const mdgmi_format* f, const float* y, const uint32_t* tx, int64_t n, const SnrArgs& sa,
                         int mode, float* llr, double* part, uint4* img, int ntiles, LaunchCfg cfg, hipStream_t st) {
    const bool tuned_shape = S == kSplitF16 && !(mode == kModeHd || mode_is_ml(mode) || f->dim == 1);
    MfmaShape shape{MfmaShape::kFixed, 0, image_bytes_per_snr(f, S) <= 128 * 1024};
    if (S == kSplitBF16 && bf16_wide(f, S)) {
        shape = {MfmaShape::kWide, 0, false};
    } else if (tuned_shape) {
        // the shape mfma_cfg chose for this launch (its block count matches)
        const int var = cfg.variant;
        if (var < 0 || var >= kNumVariants) return hipErrorInvalidValue;
        shape = {MfmaShape::kVariant, var, kVariants[var].lds && image_bytes_per_snr(f) <= 128 * 1024};
    }
    switch (f->dim) {
        case 1:
            return mfma_run<1, S>(f, y, tx, n, sa, mode, llr, part, img, ntiles, cfg, shape, st);
        case 2:
            return mfma_run<2, S>(f, y, tx, n, sa, mode, llr, part, img, ntiles, cfg, shape, st);
        case 4:
            return mfma_run<4, S>(f, y, tx, n, sa, mode, llr, part, img, ntiles, cfg, shape, st);
        case 8:
            return mfma_run<8, S>(f, y, tx, n, sa, mode, llr, part, img, ntiles, cfg, shape, st);
        default:
            return hipErrorInvalidValue;
    }
}

bool prefers_small(const mdgmi_format* f) { return use_small(f, kSplitF16, INT64_MAX); }

hipError_t launch_mfma(const mdgmi_format* f, const float* y, const uint32_t* tx, int64_t n,
                       const SnrArgs& sa, int mode, float* llr, double* part, void* image,
                       LaunchCfg cfg, hipStream_t st, int split) {
    const int ntiles = (f->M + 31) / 32;
    uint4* img = (uint4*)image;
    if (cfg.variant == kSmallVariant) return launch_small(f, y, tx, n, sa, mode, llr, part, cfg, st);
    if (split == kSplitBF16)
        return image_and_run<kSplitBF16>(f, y, tx, n, sa, mode, llr, part, img, ntiles, cfg, st);
    return image_and_run<kSplitF16>(f, y, tx, n, sa, mode, llr, part, img, ntiles, cfg, st);
}

}  // namespace mdgmi

extern "C" int mdgmi_set_tuning(int mfma_variant) {
    mdgmi::g_variant_override = mfma_variant;
    return 0;
}

extern "C" int mdgmi_get_tuning(void) { return mdgmi::g_variant_override; }

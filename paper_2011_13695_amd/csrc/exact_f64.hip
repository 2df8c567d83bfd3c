// FP64 exact demapper: one lane per sample, one exponential per (sample,
// point).
//
// e_j = exp(-||y - x_j||^2 / (2 sigma2)) is taken without a reference: it is at
// most 1, and every sum that is read stays far above the smallest double
// unless a class lies more than 2^-800 below (about 550 nats), where its
// relative precision could suffer. Such samples, and non-finite ones, are
// evaluated again with every class relative to its own nearest point
// (per_class_sample). The points are walked in label order through uniform
// (scalar) loads, 2^CHB = 16 at a time: the low label bits index a running
// bank, the chunk's total goes to the classes of the higher bits, so a pair
// costs its exponential and two additions whatever the number of bits.
//
// The bound is FP64 vector issue (4 cycles per instruction and wave; 59% busy
// under counters, the rest waits on dependent FP64 operations): 17
// instructions for the exponential and 2 dim + 2 others per pair, beside a
// per-sample end of two logarithms and four divisions. 16-QAM, 11 x 1e5
// samples: 34 us (before: m + 1 exponentials per pair, a logarithm or two per
// class sum and the library's functions, 241 us).
#include <algorithm>

#include "device_common.h"
#include "f64_math.h"

namespace mdgmi {

namespace {

using namespace f64;

constexpr int kF64Threads = 256;

template <int DIM>
__device__ __forceinline__ double dist2(const double* yv, const double* __restrict__ X, int j) {
    double d = 0.0;
#pragma unroll
    for (int q = 0; q < DIM; q++) {
        double e = yv[q] - X[j * DIM + q];
        d = fma(e, e, d);
    }
    return d;
}

// Class sums S0[k] / S1[k] of the CHB low label bits from a bank of 2^CHB
// running sums (consumed).
template <int CHB>
__device__ __forceinline__ void bank_sums(double* v, double* S0, double* S1) {
#pragma unroll
    for (int k = 0; k < CHB; k++) {
        const int w = 1 << (CHB - k);
        double a = v[0], b = v[1];
#pragma unroll
        for (int r = 2; r < w; r += 2) {
            a += v[r];
            b += v[r + 1];
        }
        S0[k] = a;
        S1[k] = b;
#pragma unroll
        for (int r = 0; r < w / 2; r++) v[r] = v[2 * r] + v[2 * r + 1];
    }
}

// Two passes with a reference per class: the class minima of the distance,
// then the sums of e^{(dmin - d) / (2 sigma2)}. Any distance of y or of a class,
// and non-finite y (NaN results). Four label bits at a time: the class minima
// and sums of all twelve would take the registers of the usual walk twice
// over. lw: label word of the sent row (GMI and hard decisions).
template <int DIM, int MODE>
__device__ __forceinline__ void per_class_sample(const double* __restrict__ yp, const double* __restrict__ X, int M,
                                                 int m, double inv2s2, const ExpScale& es, uint32_t lw,
                                                 double* llr, double& cg, double& cm, double& be, double& se) {
    const uint32_t slot = lw & kLabelMask;
    double yv[DIM];
#pragma unroll
    for (int q = 0; q < DIM; q++) yv[q] = yp[q];
    double dmin = INFINITY;
    int nb = 0;
    cg = 0.0;
#pragma unroll 1
    for (int k0 = 0; k0 < m; k0 += 4) {
        double cmin0[4], cmin1[4], S0[4], S1[4];
#pragma unroll
        for (int k = 0; k < 4; k++) {
            cmin0[k] = cmin1[k] = INFINITY;
            S0[k] = S1[k] = 0.0;
        }
        // j is uniform: the bit tests are uniform branches (bits past m - 1
        // are 0 in every j and their results unused)
#pragma unroll 1
        for (int j = 0; j < M; j++) {
            const double d = dist2<DIM>(yv, X, j);
            dmin = fmin(dmin, d);
#pragma unroll
            for (int k = 0; k < 4; k++) {
                if ((j >> (k0 + k)) & 1)
                    cmin1[k] = fmin(cmin1[k], d);
                else
                    cmin0[k] = fmin(cmin0[k], d);
            }
        }
        double tot = 0.0;
#pragma unroll 1
        for (int j = 0; j < M; j++) {
            const double d = dist2<DIM>(yv, X, j);
            if (k0 == 0 && !mode_is_llr(MODE)) tot += exp_neg(d - dmin, es);
#pragma unroll
            for (int k = 0; k < 4; k++) {
                if (k0 + k < m) {
                    const bool b = (j >> (k0 + k)) & 1;
                    const double e = exp_neg(d - (b ? cmin1[k] : cmin0[k]), es);
                    if (b)
                        S1[k] += e;
                    else
                        S0[k] += e;
                }
            }
        }
        if (k0 == 0 && !mode_is_llr(MODE)) {
            const double di = dist2<DIM>(yv, X, (int)slot);
            cm = (di - dmin) * inv2s2 + ln_pos(tot);
            if (MODE == kModeHd) se = !(dmin * inv2s2 < di * inv2s2) ? 0.0 : 1.0;
        }
        // ln sum_{class} e^{-t} = ln S - cmin
#pragma unroll
        for (int k = 0; k < 4; k++) {
            if (k0 + k < m) {
                const double l1 = ln_pos(S1[k]) - cmin1[k] * inv2s2, l0 = ln_pos(S0[k]) - cmin0[k] * inv2s2;
                const double lam = l1 - l0;
                if (mode_is_llr(MODE)) {
                    llr[k0 + k] = lam;
                } else {
                    // u = ln S_(not sent) - ln S_(sent) ; cost = softplus(u)
                    const int bk = (int)((slot >> (k0 + k)) & 1u);
                    const double u = bk ? -lam : lam;
                    // |u| times 2 sigma2 is a distance: e^-|u| by exp_neg
                    // (which drops NaN: the first term carries it)
                    cg += (u < 0.0 ? 0.0 : u) + ln1p_pos(exp_neg(fabs(u) / inv2s2, es));
                    nb += (lam == lam) ? ((lam > 0.0 ? 1 : 0) != bk) : 1;
                }
            }
        }
    }
    if (mode_is_llr(MODE)) return;
    if (MODE == kModeHd) be = (double)nb;
}

// Max-log metrics of one sample: lambda_k = min over class 0 of t - min over class 1 of t.
template <int DIM, int MODE>
__device__ __forceinline__ void maxlog_sample(const double* yv, const double* __restrict__ X, int M, int m,
                                              double inv2s2, uint32_t slot, double* llr, double& cg) {
    double cmin0[MDGMI_MAX_BITS], cmin1[MDGMI_MAX_BITS];
#pragma unroll
    for (int k = 0; k < MDGMI_MAX_BITS; k++) cmin0[k] = cmin1[k] = INFINITY;
    for (int j = 0; j < M; j++) {
        const double t = dist2<DIM>(yv, X, j) * inv2s2;
#pragma unroll
        for (int k = 0; k < MDGMI_MAX_BITS; k++) {
            if (k < m) {
                if ((j >> k) & 1)
                    cmin1[k] = fmin(cmin1[k], t);
                else
                    cmin0[k] = fmin(cmin0[k], t);
            }
        }
    }
    cg = 0.0;
#pragma unroll
    for (int k = 0; k < MDGMI_MAX_BITS; k++) {
        if (k < m) {
            const double lam = cmin0[k] - cmin1[k];
            if (MODE == kModeMlLlr) {
                llr[k] = lam;
            } else {
                const double u = ((slot >> k) & 1) ? -lam : lam;
                cg += fmax(u, 0.0) + log1p(exp(-fabs(u)));
            }
        }
    }
}

// Samples for the per-class evaluation are only marked in the walk and taken
// after each run of 32, outside its loop: called inside, it took the walk's
// registers from 152 to 202 (2-D, M = 16: two instead of three waves per SIMD).
template <int DIM, int CHB, int MAXHI, int MODE>
__global__ __launch_bounds__(kF64Threads, 2) void k_exact_f64(const double* __restrict__ y,
                                                              const uint32_t* __restrict__ tx,
                                                              const double* __restrict__ X,
                                                              const uint32_t* __restrict__ labels, int64_t n,
                                                              int M, int m, SnrArgs sa, double* __restrict__ llr,
                                                              double* __restrict__ part) {
    constexpr int CH = 1 << CHB, MB = CHB + MAXHI;  // label bits: up to MB
    const int q_snr = blockIdx.y;
    const double inv2s2 = sa.inv2s2[q_snr];
    const ExpScale es = exp_scale(inv2s2);
    const int64_t snr = sa.snr0 + q_snr;
    const double* ys = y + snr * n * DIM;
    constexpr bool LLR = MODE == kModeLlr;
    const uint32_t* txs = mode_is_llr(MODE) ? nullptr : tx + snr * n;
    CostAcc acc;
    HdAcc hd;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    // label word of the sent row; a row outside [0, M) gives a NaN cost
    // instead of a stray read
    auto sent = [&](int64_t i, bool& row_ok) {
        if (mode_is_llr(MODE)) return 0u;
        const uint32_t row = txs[i];
        row_ok = row < (uint32_t)M;
        return labels[row_ok ? row : 0u];
    };
    auto count = [&](double cg, double cm, double be, double se, uint32_t lw, bool row_ok) {
        if (!row_ok) cg = cm = NAN;
        acc.add(cg * kLog2e, cm * kLog2e);
        if (MODE == kModeHd) {
            // bitwise MAP decisions (sign of the LLR) and the nearest point
            // (some other point strictly nearer than the sent one, or its
            // coordinates shared with a lower label: ties go to the lowest
            // label)
            const bool finite = cg == cg && cm == cm;
            hd.be += finite ? be : (double)m;
            hd.se += finite && (lw & kTwinBit) == 0u ? se : 1.0;
        }
    };
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    while (i < n) {
        const int64_t i0 = i;
        uint32_t redo = 0u;  // samples i0 + t stride for the per-class evaluation
#pragma unroll 1
        for (int t = 0; t < 32 && i < n; t++, i += stride) {
            double yv[DIM];
#pragma unroll
            for (int q = 0; q < DIM; q++) yv[q] = ys[i * DIM + q];
            bool row_ok = true;
            const uint32_t lw = sent(i, row_ok), slot = lw & kLabelMask;
            if constexpr (mode_is_ml(MODE)) {
                double cg = 0.0;
                maxlog_sample<DIM, MODE>(yv, X, M, m, inv2s2, slot, MODE == kModeMlLlr ? llr + i * m : nullptr, cg);
                if (MODE == kModeMlGmi) acc.add((row_ok ? cg : NAN) * kLog2e, 0.0);
            } else {
                double bank[CH], S0[MB], S1[MB], dmin = INFINITY;
#pragma unroll
                for (int r = 0; r < CH; r++) bank[r] = 0.0;
#pragma unroll
                for (int l = CHB; l < MB; l++) S0[l] = S1[l] = 0.0;
                const int nchunk = MAXHI == 0 ? 1 : M >> CHB;
                for (int c = 0; c < nchunk; c++) {
                    double e[CH];
#pragma unroll
                    for (int r = 0; r < CH; r++) {
                        const double d = dist2<DIM>(yv, X, c * CH + r);
                        if (MODE == kModeHd) dmin = fmin(dmin, d);
                        e[r] = exp_neg(d, es);
                        bank[r] += e[r];
                    }
                    if constexpr (MAXHI > 0) {
#pragma unroll
                        for (int w = 1; w < CH; w <<= 1) {
#pragma unroll
                            for (int r = 0; r < CH; r += 2 * w) e[r] += e[r + w];
                        }
#pragma unroll
                        for (int l = 0; l < MAXHI; l++) {  // c is uniform
                            if (l < m - CHB) {
                                if ((c >> l) & 1)
                                    S1[CHB + l] += e[0];
                                else
                                    S0[CHB + l] += e[0];
                            }
                        }
                    }
                }
                bank_sums<CHB>(bank, S0, S1);
                const double tot = bank[0];
                if (LLR) {
                    double smin = tot;
#pragma unroll
                    for (int k = 0; k < MB; k++)
                        if (k < m) smin = fmin(smin, fmin(S0[k], S1[k]));
                    if (smin >= 0x1p-800) {
#pragma unroll
                        for (int k = 0; k < MB; k++)
                            if (k < m) llr[i * m + k] = ln_pos(fast_div(S1[k], S0[k]));
                    } else {
                        redo |= 1u << t;
                    }
                } else {
                    // GMI cost sum_k ln(1 + S_other / S_sent) = ln(1 / prod_k s_k) with
                    // s_k = S_sent,k / T, o_k = S_other,k / T = 1 - s_k: as
                    // ln(1 + num / den), den = prod s_k, num = 1 - den =
                    // sum_k o_k prod_{j<k} s_j (positive terms only, so that small
                    // costs keep their digits)
                    const double di = dist2<DIM>(yv, X, (int)slot);
                    const double ei = exp_neg(di, es), rT = fast_div(1.0, tot);
                    double num = 0.0, den = 1.0, be = 0.0;
#pragma unroll
                    for (int k = 0; k < MB; k++) {
                        if (k < m) {
                            const bool bk = (slot >> k) & 1;
                            const double s = bk ? S1[k] : S0[k], o = bk ? S0[k] : S1[k];
                            num = fma(den, o * rT, num);
                            den *= s * rT;
                            if (MODE == kModeHd) be += (S1[k] > S0[k]) != bk ? 1.0 : 0.0;
                        }
                    }
                    if (ei >= 0x1p-400 && den >= 0x1p-900) {
                        const double cg = ln1p_pos(fast_div(num, den));
                        const double cm = ln_pos(fast_div(tot, ei));  // the sent point is in the total: >= 0
                        count(cg, cm, be, dmin * inv2s2 < di * inv2s2 ? 1.0 : 0.0, lw, row_ok);
                    } else {
                        redo |= 1u << t;
                    }
                }
            }
        }
        while (redo != 0u) {
            const int t = __ffs((int)redo) - 1;
            redo &= redo - 1u;
            const int64_t k = i0 + t * stride;
            bool row_ok = true;
            const uint32_t lw = sent(k, row_ok);
            double cg = 0.0, cm = 0.0, be = 0.0, se = 0.0;
            per_class_sample<DIM, MODE>(ys + k * DIM, X, M, m, inv2s2, es, lw, LLR ? llr + k * m : nullptr, cg,
                                        cm, be, se);
            if (!LLR) count(cg, cm, be, se, lw, row_ok);
        }
    }
    double* dst = part + ((int64_t)q_snr * gridDim.x + blockIdx.x) * (MODE == kModeHd ? kNPartHd : kNPart);
    if (MODE == kModeGmi || MODE == kModeMlGmi) block_reduce_store(acc, dst);
    if (MODE == kModeHd) block_reduce_store_hd(acc, hd, dst);
}

template <int DIM, int CHB, int MAXHI>
hipError_t launch_f64_t(const mdgmi_format* f, const double* y, const uint32_t* tx, int64_t n, const SnrArgs& sa,
                        int mode, double* llr, double* part, LaunchCfg cfg, hipStream_t st) {
    dim3 grid(cfg.blocks_per_snr, sa.n_snr), block(cfg.threads);
    // part points at the first block row of this launch's first SNR.
#define MDGMI_F64_MODE(MD)                                                                                  \
    case MD:                                                                                                \
        hipLaunchKernelGGL((k_exact_f64<DIM, CHB, MAXHI, MD>), grid, block, 0, st, y, tx, f->d_X64,                \
                           MD == kModeHd ? f->d_labels_hd : f->d_labels, n, f->M, f->m, sa, llr, part);     \
        break;
    switch (mode) {
        MDGMI_F64_MODE(kModeLlr)
        MDGMI_F64_MODE(kModeHd)
        MDGMI_F64_MODE(kModeMlLlr)
        MDGMI_F64_MODE(kModeMlGmi)
        default:
            MDGMI_F64_MODE(kModeGmi)
    }
#undef MDGMI_F64_MODE
    return hipGetLastError();
}

template <int DIM>
hipError_t launch_f64_d(const mdgmi_format* f, const double* y, const uint32_t* tx, int64_t n, const SnrArgs& sa,
                        int mode, double* llr, double* part, LaunchCfg cfg, hipStream_t st) {
    switch (f->m) {  // chunks of 16 points, or the whole format where it is smaller
        case 1:
            return launch_f64_t<DIM, 1, 0>(f, y, tx, n, sa, mode, llr, part, cfg, st);
        case 2:
            return launch_f64_t<DIM, 2, 0>(f, y, tx, n, sa, mode, llr, part, cfg, st);
        case 3:
            return launch_f64_t<DIM, 3, 0>(f, y, tx, n, sa, mode, llr, part, cfg, st);
        case 4:
            return launch_f64_t<DIM, 4, 0>(f, y, tx, n, sa, mode, llr, part, cfg, st);
        default:
            return launch_f64_t<DIM, 4, MDGMI_MAX_BITS - 4>(f, y, tx, n, sa, mode, llr, part, cfg, st);
    }
}

}  // namespace

// 256-thread blocks per CU over the SNR points of the launch: twelve where
// LLRs are written (whole rounds at the two, three or four resident blocks per
// CU that the instantiations' registers allow), six where a block ends in the
// FP64 reduction, whose ~250 instructions count beside a few samples (two or
// three resident). Each block takes the same number of strides.
LaunchCfg f64_cfg(const mdgmi_format* f, int64_t n, int n_snr, int mode) {
    (void)f;
    const int64_t want = (n + kF64Threads - 1) / kF64Threads;
    const int snr_in_launch = snr_per_launch(n_snr);
    const int64_t cap = std::max<int64_t>(1, (int64_t)device_cu_count() * (mode_is_llr(mode) ? 12 : 6) / snr_in_launch);
    const int64_t strides = (want + cap - 1) / cap;
    LaunchCfg c;
    c.threads = kF64Threads;
    c.blocks_per_snr = (int)((want + strides - 1) / strides);
    return c;
}

// blocks_per_snr is at most min(want, 6 per CU) where partial sums are kept
int64_t f64_blocks_bound(int64_t n) {
    return std::min<int64_t>((n + kF64Threads - 1) / kF64Threads, (int64_t)device_cu_count() * 8);
}

hipError_t launch_f64(const mdgmi_format* f, const double* y, const uint32_t* tx, int64_t n,
                      const SnrArgs& sa, int mode, double* llr, double* part, LaunchCfg cfg,
                      hipStream_t st) {
    switch (f->dim) {
        case 1:
            return launch_f64_d<1>(f, y, tx, n, sa, mode, llr, part, cfg, st);
        case 2:
            return launch_f64_d<2>(f, y, tx, n, sa, mode, llr, part, cfg, st);
        case 4:
            return launch_f64_d<4>(f, y, tx, n, sa, mode, llr, part, cfg, st);
        case 8:
            return launch_f64_d<8>(f, y, tx, n, sa, mode, llr, part, cfg, st);
        default:
            return hipErrorInvalidValue;
    }
}

}  // namespace mdgmi

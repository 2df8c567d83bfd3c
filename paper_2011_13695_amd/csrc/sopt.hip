// s-optimised GMI and per-bit GMI of given LLRs (any demapper: exact,
// max-log, learned).
//
// For LLRs lambda_ik and sent bits b_k(i), with v_ik = (2 b_k(i) - 1) lambda_ik,
//     GMI(s) = m - (1/n) sum_i sum_k log2(1 + exp(-s v_ik)),   s >= 0,
// is the GMI of a bit-metric decoder that uses the LLRs scaled by s; the
// s-optimised GMI is its maximum over s. Each term log(1 + e^{-s v}) is
// convex in s, so GMI(s) is concave and the maximum is where the derivative
// of the total cost
//     C'(s)  = -sum v sigma(-s v),     C''(s) = sum v^2 sigma(s v) sigma(-s v)
// vanishes. The search runs on the device: each pass evaluates the cost and
// both derivatives at the current s (FP64 sums, fixed reduction order); then a
// Newton step is taken, kept inside the bracket [lo, hi] of the sign changes of
// C' (bisection, or doubling while no upper end is known), until it has
// converged. The first kSoptAhead passes are launches of their own (k_sopt_pass),
// each of which takes the step from the sums of the one before in its prologue;
// whatever passes are left are one launch (k_sopt_rest), after one that settles
// the state they start from: eight launches a call. Once the search has ended the
// remaining ones return at once.
//
// What bounds it: a pass over 1000003 x 11 FP32 LLRs takes 12 us (48 MB, 4.0
// TB/s: the copy rate), the step in its prologue and the launch about 5 us; five
// passes, and three launches after the end, 110 us a call. (The library's expf,
// log1pf and divisions per LLR and one 4-byte load each made a pass 69 us, and the
// 60 pairs of launches past the last needed pass 4 us each: 509 us.)
#include <algorithm>

#include "device_common.h"
#include "f64_math.h"

namespace mdgmi {

namespace {

constexpr int kSoptThreads = 256;
constexpr int kSoptPart = 6;      // sum C, sum C^2, sum C', sum C'', sum v, non-finite
constexpr int kSoptPasses = 64;
// Gaussian LLRs of unequal bits scaled by 0.5 to 1.4 take 5-7 passes in FP32, 6-8 in
// FP64 (matched ones 3-4): a seventh one, in k_sopt_rest, takes a 4-bit FP64 call of
// 100001 samples from 55 to 73 us
constexpr int kSoptAhead = 6;
constexpr int kSearchThreads = 512;
// state of the search: s, lo, hi, passes done, best GMI so far, ended, the s
// reported so far. Two slots, written in turn; then the words that order the
// passes of k_sopt_rest: the next ticket, the shares done, the passes published.
constexpr int kStS = 0, kStLo = 1, kStHi = 2, kStIter = 3, kStBest = 4, kStOver = 5, kStRowS = 6, kStLen = 7;
constexpr int kStSync = 2 * kStLen, kStateLen = 16;
constexpr int kSyncTicket = 0, kSyncDone = 1, kSyncPass = 2, kSyncLen = 3;
static_assert(kStSync * sizeof(double) + kSyncLen * sizeof(uint32_t) <= kStateLen * sizeof(double), "state layout");
constexpr uint32_t kSoptOver = 0xffffffffu;  // passes published, once the search has ended

// Values that blocks of k_sopt_rest hand to each other (partial sums, state, the
// result row) go through agent-scope atomic stores and loads, which bypass the
// caches of the eight dies; a writer waits for its stores (drain) before it
// counts itself done. Agent-scope fences instead write back and invalidate
// whole L2s, once per block and pass: 150 us a pass where the work is 15.
__device__ __forceinline__ void put(double* p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double get(const double* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void drain() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// One LLR (v: its sign turned so that positive favours the sent bit) at scale
// s, z = s v, e = e^-|z|, in the precision of the LLRs. The cost log(1 + e^-z) =
// max(-z, 0) + log(1 + e): the first part is summed in mx, the second goes into
// P, prod (1 + e) - 1, as P + e (1 + P), whose positive terms keep the digits of
// small e; one log1p per sample follows. d1 and d2 are the s-derivatives. NaN
// and infinities: |z| is capped where e is 0, which also drops NaN; mx and the
// derivatives carry it.
__device__ __forceinline__ void term(float v, float s, float& mx, float& P, float& d1, float& d2) {
    const float z = s * v, az = fminf(fabsf(z), 200.0f);
    // e^-az as 2^h (1 + l ln 2), h the rounded product with log2(e), l its error
    const float c = -1.44269502f, cl = -1.92596303e-8f;
    const float h = az * c, l = fmaf(az, cl, fmaf(az, c, -h));
    float e = ex2(h);
    e = fmaf(e, l * 0.693147182f, e);
    const float q = 1.0f + e;
    float p = __builtin_amdgcn_rcpf(q);
    p = fmaf(p, fmaf(-q, p, 1.0f), p);
    mx += z > 0.0f ? 0.0f : -z;
    P += fmaf(e, P, e);
    const float w = v * p;              // v sigma(-z) = w e or w
    d1 -= w * (z >= 0.0f ? e : 1.0f);
    d2 = fmaf(w * w, e, d2);
}

__device__ __forceinline__ void term(double v, double s, double& mx, double& P, double& d1, double& d2) {
    const double z = s * v, az = fabs(z);
    // exp_neg stays at 2^-1000 from |z| = 693 on; the derivatives have to reach 0, or
    // a search among LLRs without an error would go on for all its passes
    const double e0 = f64::exp_neg(az, f64::exp_scale_unit()), e = az > 693.0 ? 0.0 : e0;
    const double p = f64::fast_div(1.0, 1.0 + e);
    mx += z > 0.0 ? 0.0 : -z;
    P += fma(e, P, e);
    const double w = v * p;
    d1 -= w * (z >= 0.0 ? e : 1.0);
    d2 = fma(w * w, e, d2);
}

__device__ __forceinline__ float log1p_of(float P) { return log1pf(P); }
__device__ __forceinline__ double log1p_of(double P) { return f64::ln1p_pos(P); }

// tol: relative step (and bracket) size taken as converged; it follows the
// precision of the LLRs, whose rounding bounds how small a Newton step the
// derivative sums can resolve. flat: the rounding of the cost of one bit.
// One thread: the state after the pass whose sums are tot, from the state
// before it; with `row` the result row is updated too.
__device__ void sopt_update(const double* tot, const double* now, int64_t n, int m, double tol, double flat,
                            double* next, double* __restrict__ out, bool row) {
    const double N = (double)n, s = now[kStS];
    auto put_row = [&](int k, double v) {
        if (row) put(out + k, v);
    };
    for (int k = 0; k < kStLen; k++) next[k] = now[k];
    next[kStOver] = 1.0;
    const double gmi = m - tot[0] / N;
    const double var = n > 1 ? (tot[1] - tot[0] * tot[0] / N) / (N - 1.0) : 0.0;
    const double se = sqrt(fmax(var, 0.0) / N);
    const int it = (int)now[kStIter];
    if (it == 0) {  // s = 1
        put_row(MDGMI_S_GMI1, gmi);
        put_row(MDGMI_S_SE1, se);
        put_row(MDGMI_S_N, N);
        put_row(MDGMI_S_NONFINITE, tot[5]);
        if (tot[5] > 0.0) {  // non-finite LLRs or sent rows out of range: estimates stay NaN
            put_row(MDGMI_S_ITERS, 1.0);
            return;
        }
        if (!(tot[4] > 0.0)) {
            // C'(0) = -sum v / 2 >= 0: the cost only grows with s, the
            // maximum is GMI(0) = 0 at s = 0
            put_row(MDGMI_S_S, 0.0);
            put_row(MDGMI_S_GMI, 0.0);
            put_row(MDGMI_S_SE, 0.0);
            put_row(MDGMI_S_NGMI, 0.0);
            put_row(MDGMI_S_ITERS, 1.0);
            return;
        }
    }
    // keep the best point evaluated. Around the optimum the costs' rounding
    // decides which of two neighbouring points looks better (a step of relative
    // size d changes the GMI by at most d^2 / 3 a bit), while the derivative still
    // tells them apart: s follows it there, the GMI reported stays the largest.
    const bool better = gmi > now[kStBest];
    if (better) {
        next[kStBest] = gmi;
        put_row(MDGMI_S_GMI, gmi);
        put_row(MDGMI_S_SE, se);
        put_row(MDGMI_S_NGMI, gmi / m);
    }
    if (better || (gmi > now[kStBest] - flat * m && fabs(s - now[kStRowS]) <= 16.0 * sqrt(flat) * s)) {
        next[kStRowS] = s;
        put_row(MDGMI_S_S, s);
    }
    put_row(MDGMI_S_ITERS, it + 1);
    next[kStIter] = it + 1;
    const double d1 = tot[2], d2 = tot[3];
    if (d1 == 0.0) return;
    double lo = now[kStLo], hi = now[kStHi];
    if (d1 > 0.0)
        hi = s;
    else
        lo = s;
    const double step = d2 > 0.0 ? d1 / d2 : NAN;
    // converged: the Newton step is below the tolerance (tested before the
    // bracket, which a step of rounding size can touch)
    if (fabs(step) <= tol * s) return;
    double sn = s - step;
    if (!(sn > lo && sn < hi)) sn = hi < INFINITY ? 0.5 * (lo + hi) : 2.0 * s;
    next[kStLo] = lo;
    next[kStHi] = hi;
    next[kStS] = sn;
    next[kStOver] = (hi < INFINITY && hi - lo <= tol * hi) || it + 1 == kSoptPasses ? 1.0 : 0.0;
}

// The sums of one share (a strided set of samples) at scale s, over the block,
// into tot.
template <typename T, int BITS>
__device__ __forceinline__ void sopt_share(const T* __restrict__ llr, const uint32_t* __restrict__ tx,
                                           const uint32_t* __restrict__ labels, int M, int64_t n, int share,
                                           int shares, T s, double* tot) {
    double sc = 0.0, sc2 = 0.0, sd1 = 0.0, sd2 = 0.0, sv = 0.0, bad = 0.0;
    const int64_t stride = (int64_t)shares * kSearchThreads;
    for (int64_t i = (int64_t)share * kSearchThreads + threadIdx.x; i < n; i += stride) {
        T lam[BITS];
#pragma unroll
        for (int k = 0; k < BITS; k++) lam[k] = llr[i * BITS + k];
        const uint32_t row = tx[i];
        const bool row_ok = row < (uint32_t)M;
        const uint32_t slot = labels[row_ok ? row : 0u];
        T mx = 0, P = 0, d1 = 0, d2 = 0, vs = 0;
#pragma unroll
        for (int k = 0; k < BITS; k++) {
            const T v = ((slot >> k) & 1u) ? lam[k] : -lam[k];
            term(v, s, mx, P, d1, d2);
            vs += v;
        }
        double cb = (double)(mx + log1p_of(P)) * kLog2e;  // bits
        if (!row_ok) cb = NAN;
        sc += cb;
        sc2 += cb * cb;
        sd1 += (double)d1 * kLog2e;
        sd2 += (double)d2 * kLog2e;
        sv += (double)vs;
        bad += __builtin_isfinite(cb) ? 0.0 : 1.0;
    }
    double v[kSoptPart] = {sc, sc2, sd1, sd2, sv, bad};
    block_reduce_vals<kSoptPart>(v, tot);
}

// Sums of all shares, in a fixed order, into tot (thread 0's to read).
template <class Get>
__device__ __forceinline__ void sopt_total(const double* __restrict__ part, int shares, double* tot, Get get_part) {
    double v[kSoptPart] = {};
    for (int b = threadIdx.x; b < shares; b += kSearchThreads) {
#pragma unroll
        for (int k = 0; k < kSoptPart; k++) v[k] += get_part(part + (size_t)b * kSoptPart + k);
    }
    block_reduce_vals<kSoptPart>(v, tot);
}

__device__ __forceinline__ constexpr double flat_of(bool f32) { return f32 ? 0x1p-23 : 0x1p-52; }

// The state that pass p starts from, into now (shared; every thread may read
// it): s = 1 for the first, else the step from the sums of pass p - 1, which
// every block takes for itself, from the same numbers; the first block keeps
// state and result row. sums / state slots alternate with p.
template <bool F32>
__device__ __forceinline__ void sopt_step(int p, int shares, int64_t n, int m, double tol, double* state,
                                          const double* part, double* out, double* now) {
    __shared__ double tot[kSoptPart];
    const bool keep = blockIdx.x == 0;
    const double* before = state + ((p + 1) & 1) * kStLen;
    if (p == 0) {
        if (threadIdx.x == 0) {
            now[kStS] = 1.0;
            now[kStLo] = 0.0;
            now[kStHi] = INFINITY;
            now[kStIter] = 0.0;
            now[kStBest] = -INFINITY;
            now[kStOver] = 0.0;
            now[kStRowS] = 0.0;
        }
        if (keep && threadIdx.x < MDGMI_NFIELDS_S) out[threadIdx.x] = NAN;
    } else if (before[kStOver] != 0.0) {
        if (threadIdx.x < kStLen) now[threadIdx.x] = before[threadIdx.x];
    } else {
        sopt_total(part + (size_t)((p + 1) & 1) * shares * kSoptPart, shares, tot, [](const double* q) { return *q; });
        if (threadIdx.x == 0) {
            double b[kStLen], nx[kStLen];
            for (int k = 0; k < kStLen; k++) b[k] = before[k];
            sopt_update(tot, b, n, m, tol, flat_of(F32), nx, out, keep);
            for (int k = 0; k < kStLen; k++) now[k] = nx[k];
        }
    }
    __syncthreads();
    if (keep && threadIdx.x < kStLen) state[(p & 1) * kStLen + threadIdx.x] = now[threadIdx.x];
}

template <typename T, int BITS>
__global__ __launch_bounds__(kSearchThreads) void k_sopt_pass(const T* __restrict__ llr,
                                                              const uint32_t* __restrict__ tx,
                                                              const uint32_t* __restrict__ labels, int M, int64_t n,
                                                              int shares, double tol, int p, double* state,
                                                              double* part, double* out) {
    __shared__ double now[kStLen];
    sopt_step<sizeof(T) == 4>(p, shares, n, BITS, tol, state, part, out, now);
    if (now[kStOver] != 0.0) return;
    sopt_share<T, BITS>(llr, tx, labels, M, n, (int)blockIdx.x, shares, (T)now[kStS],
                        part + ((size_t)(p & 1) * shares + blockIdx.x) * kSoptPart);
}

// The step after the last pass launched ahead, and k_sopt_rest's words; one block.
template <bool F32>
__global__ __launch_bounds__(kSearchThreads) void k_sopt_settle(int64_t n, int m, int shares, double tol,
                                                                double* state, const double* part, double* out) {
    __shared__ double now[kStLen];
    sopt_step<F32>(kSoptAhead, shares, n, m, tol, state, part, out, now);
    uint32_t* sync = (uint32_t*)(state + kStSync);
    if (threadIdx.x == 0) sync[kSyncTicket] = sync[kSyncDone] = sync[kSyncPass] = 0u;
}

// The passes after the first kSoptAhead, in one launch. Work is dealt in
// tickets: ticket t is share t mod shares of pass t / shares (a share is always
// the same samples, so the sums do not depend on who takes it), and a block
// that draws a share of a later pass first waits until the pass before is
// published. Every wait ends, also where not all blocks are resident: the
// shares of the pass waited for were drawn earlier, by blocks that are running
// and that wait, in turn, only for passes before it; after the last pass the
// end is published instead, and the block that sees it leaves. The block that
// completes a pass sums the shares in order, updates the state and publishes.
// 10-45 us a pass beside its work, by the blocks that wait, against 5 us for a
// launch: hence the launches ahead.
template <typename T, int BITS>
__global__ __launch_bounds__(kSearchThreads) void k_sopt_rest(const T* __restrict__ llr,
                                                              const uint32_t* __restrict__ tx,
                                                              const uint32_t* __restrict__ labels, int M, int64_t n,
                                                              int shares, double tol, double* state, double* part,
                                                              double* out) {
    __shared__ double tot[kSoptPart], now[kStLen];
    __shared__ uint32_t s_ticket, s_last;
    uint32_t* sync = (uint32_t*)(state + kStSync);
    state += (kSoptAhead & 1) * kStLen;
    // one thread looks for the block: where the block starts late, the last pass
    // may be publishing its state at this moment, and of waves that go by their own
    // reads some could leave and the rest wait for a ticket nobody draws (once the
    // word is set, every share of every pass has been drawn and summed)
    if (threadIdx.x == 0) s_last = get(state + kStOver) != 0.0 ? 1u : 0u;
    __syncthreads();
    if (s_last != 0u) return;
    for (;;) {
        if (threadIdx.x == 0) {
            const uint32_t t = __hip_atomic_fetch_add(sync + kSyncTicket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t pass = t / (uint32_t)shares;
            uint32_t seen = 0u;
            if (pass > 0u) {
                while ((seen = __hip_atomic_load(sync + kSyncPass, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < pass)
                    __builtin_amdgcn_s_sleep(16);
            }
            s_ticket = seen == kSoptOver ? kSoptOver : t;
        }
        __syncthreads();
        const uint32_t ticket = __builtin_amdgcn_readfirstlane(s_ticket);
        if (ticket == kSoptOver) return;
        const int share = (int)(ticket % (uint32_t)shares);
        const uint32_t pass = ticket / (uint32_t)shares;
        sopt_share<T, BITS>(llr, tx, labels, M, n, share, shares, (T)get(state + kStS), tot);
        if (threadIdx.x == 0) {
#pragma unroll
            for (int k = 0; k < kSoptPart; k++) put(part + (size_t)share * kSoptPart + k, tot[k]);
            drain();
            const uint32_t done = __hip_atomic_fetch_add(sync + kSyncDone, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_last = done + 1u == (pass + 1u) * (uint32_t)shares ? 1u : 0u;
        }
        __syncthreads();
        if (s_last != 0u) {
            if (threadIdx.x < kStLen) now[threadIdx.x] = get(state + threadIdx.x);
            sopt_total(part, shares, tot, [](const double* q) { return get(q); });
            if (threadIdx.x == 0) {
                double b[kStLen], nx[kStLen];
                for (int k = 0; k < kStLen; k++) b[k] = now[k];
                sopt_update(tot, b, n, BITS, tol, flat_of(sizeof(T) == 4), nx, out, true);
                for (int k = 0; k < kStLen; k++) put(state + k, nx[k]);
                drain();
                __hip_atomic_store(sync + kSyncPass, nx[kStOver] != 0.0 ? kSoptOver : pass + 1u, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        __syncthreads();
    }
}

// ---- per-bit GMI of given LLRs (s = 1) ---------------------------------
// GMI_k = 1 - mean_i log2(1 + exp(-v_ik)): per-bit FP64 sums of the cost and
// its square, one pass, then a one-block finish in a fixed order.
constexpr int kBitsPart = 2 * MDGMI_MAX_BITS + 1;

template <typename T>
__global__ __launch_bounds__(kSoptThreads) void k_bits_pass(const T* __restrict__ llr,
                                                             const uint32_t* __restrict__ tx,
                                                             const uint32_t* __restrict__ labels, int M, int64_t n,
                                                             int m, double* __restrict__ part) {
    double v[kBitsPart] = {};
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint32_t row = tx[i];
        const bool row_ok = row < (uint32_t)M;
        const uint32_t slot = labels[row_ok ? row : 0u];
        bool fin = row_ok;
#pragma unroll
        for (int k = 0; k < MDGMI_MAX_BITS; k++) {
            if (k < m) {
                const T lam = llr[i * m + k];
                const T u = ((slot >> k) & 1u) ? -lam : lam;   // cost = log(1 + e^u)
                double c = (double)((u > T(0) ? u : T(0)) + log1p(exp(-fabs(u)))) * kLog2e;
                if (!row_ok) c = NAN;
                fin = fin && __builtin_isfinite(c);
                v[2 * k] += c;
                v[2 * k + 1] += c * c;
            }
        }
        v[2 * MDGMI_MAX_BITS] += fin ? 0.0 : 1.0;
    }
    block_reduce_vals<kBitsPart>(v, part + (size_t)blockIdx.x * kBitsPart);
}

__global__ __launch_bounds__(256) void k_bits_finish(const double* __restrict__ part, int nblocks, int64_t n, int m,
                                                     double* __restrict__ out) {
    double v[kBitsPart] = {};
    for (int b = threadIdx.x; b < nblocks; b += blockDim.x) {
#pragma unroll
        for (int k = 0; k < kBitsPart; k++) v[k] += part[(size_t)b * kBitsPart + k];
    }
    __shared__ double tot[kBitsPart];
    block_reduce_vals<kBitsPart>(v, tot);
    __syncthreads();
    if (threadIdx.x != 0) return;
    const double N = (double)n;
    for (int k = 0; k < m; k++) {
        const double s1 = tot[2 * k], s2 = tot[2 * k + 1];
        const double var = n > 1 ? (s2 - s1 * s1 / N) / (N - 1.0) : 0.0;
        out[2 * k] = 1.0 - s1 / N;
        out[2 * k + 1] = sqrt(fmax(var, 0.0) / N);
    }
    out[2 * m] = N;
    out[2 * m + 1] = tot[2 * MDGMI_MAX_BITS];
}

int sopt_blocks(int64_t n) {
    const int64_t want = (n + kSoptThreads - 1) / kSoptThreads;
    const int64_t cap = (int64_t)device_cu_count() * 8;
    return (int)std::max<int64_t>(1, std::min(want, cap));
}

}  // namespace

size_t bits_workspace_bytes(int64_t n) { return (size_t)sopt_blocks(n) * kBitsPart * sizeof(double); }

hipError_t launch_bits(const mdgmi_format* f, const void* llr, bool f64, const uint32_t* tx, int64_t n, double* out,
                       void* ws, hipStream_t st) {
    double* part = (double*)ws;
    const int nb = sopt_blocks(n);
    if (f64)
        hipLaunchKernelGGL(k_bits_pass<double>, dim3(nb), dim3(kSoptThreads), 0, st, (const double*)llr, tx,
                           f->d_labels, f->M, n, f->m, part);
    else
        hipLaunchKernelGGL(k_bits_pass<float>, dim3(nb), dim3(kSoptThreads), 0, st, (const float*)llr, tx,
                           f->d_labels, f->M, n, f->m, part);
    hipLaunchKernelGGL(k_bits_finish, dim3(1), dim3(256), 0, st, part, nb, n, f->m, out);
    return hipGetLastError();
}

namespace {

// shares of a pass: at most two 512-thread blocks per CU, a few samples per
// thread, so that the next step has few partial sums to add
int sopt_shares(int64_t n) {
    return (int)std::min<int64_t>((n + kSearchThreads - 1) / kSearchThreads, (int64_t)device_cu_count() * 2);
}

}  // namespace

size_t sopt_workspace_bytes(int64_t n) {
    return (size_t)(kStateLen + 2 * (size_t)sopt_shares(n) * kSoptPart) * sizeof(double);
}

namespace {

template <typename T>
hipError_t launch_sopt_t(const mdgmi_format* f, const T* llr, const uint32_t* tx, int64_t n, int shares, double tol,
                         double* state, double* part, double* out, hipStream_t st) {
#define MDGMI_SOPT(B)                                                                                              \
    case B:                                                                                                        \
        for (int p = 0; p < kSoptAhead; p++)                                                                       \
            hipLaunchKernelGGL((k_sopt_pass<T, B>), dim3(shares), dim3(kSearchThreads), 0, st, llr, tx, f->d_labels, \
                               f->M, n, shares, tol, p, state, part, out);                                         \
        hipLaunchKernelGGL((k_sopt_settle<sizeof(T) == 4>), dim3(1), dim3(kSearchThreads), 0, st, n, B, shares, tol, \
                           state, part, out);                                                                      \
        hipLaunchKernelGGL((k_sopt_rest<T, B>), dim3(shares), dim3(kSearchThreads), 0, st, llr, tx, f->d_labels,    \
                           f->M, n, shares, tol, state, part, out);                                                \
        break;
    switch (f->m) {
        MDGMI_SOPT(1)
        MDGMI_SOPT(2)
        MDGMI_SOPT(3)
        MDGMI_SOPT(4)
        MDGMI_SOPT(5)
        MDGMI_SOPT(6)
        MDGMI_SOPT(7)
        MDGMI_SOPT(8)
        MDGMI_SOPT(9)
        MDGMI_SOPT(10)
        MDGMI_SOPT(11)
        MDGMI_SOPT(12)
        default:
            return hipErrorInvalidValue;
    }
#undef MDGMI_SOPT
    return hipGetLastError();
}

}  // namespace

hipError_t launch_sopt(const mdgmi_format* f, const void* llr, bool f64, const uint32_t* tx, int64_t n, double* out,
                       void* ws, hipStream_t st) {
    double* state = (double*)ws;
    double* part = state + kStateLen;
    const int shares = sopt_shares(n);
    return f64 ? launch_sopt_t(f, (const double*)llr, tx, n, shares, 1e-12, state, part, out, st)
               : launch_sopt_t(f, (const float*)llr, tx, n, shares, 1e-7, state, part, out, st);
}

}  // namespace mdgmi

// The ticket loop of the s-search (k_sopt_rest, its text passed in as KERNEL)
// on the CPU: one block, a thread per wave, a barrier that counts the waves
// still running (as the hardware's does), and device memory whose word "search
// ended" can be made to change between two waves' first reads of it.
//
//   driver S   the block starts while the word is being written, and the first
//              wave reads it set, the others not (S = 1), or the other way
//              round (S = 2); or it starts in time and serves all passes (S = 0)
//
// Exit status 0: every wave ended, after the expected work. 2: a wave that went
// round the loop without a ticket of its own.
#include <atomic>
#include <cmath>
#include <condition_variable>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <mutex>
#include <thread>
#include <vector>

#define __global__
#define __launch_bounds__(x)
#define __shared__ static
constexpr int kWaves = 8, kSearchThreads = 64 * kWaves;
constexpr int kSoptPart = 6, kSoptAhead = 6;
constexpr int kStS = 0, kStOver = 5, kStLen = 7, kStSync = 2 * kStLen;  // (any length: offsets are the driver's own)
constexpr int kSyncTicket = 0, kSyncDone = 1, kSyncPass = 2;
constexpr uint32_t kSoptOver = 0xffffffffu;
constexpr int kShares = 3, kPasses = 4;
struct Idx {
    unsigned x;
};
thread_local Idx threadIdx;
double g_state[2 * kStLen + 2];
double g_part[kShares * kSoptPart];
int g_scenario = 0;
std::atomic<int> g_shares{0}, g_rounds{0};

std::mutex g_mu;
std::condition_variable g_cv;
int g_live = kWaves, g_at = 0;
long g_phase = 0;
void __syncthreads() {
    std::unique_lock<std::mutex> l(g_mu);
    const long p = g_phase;
    if (++g_at == g_live) {
        g_at = 0;
        g_phase++;
        g_cv.notify_all();
    } else {
        g_cv.wait(l, [&] { return g_phase != p; });
    }
}
void wave_ended() {
    std::lock_guard<std::mutex> l(g_mu);
    if (--g_live > 0 && g_at == g_live) {
        g_at = 0;
        g_phase++;
        g_cv.notify_all();
    }
}
// a lane's first read of the word, by wave: what the two sides of the store give
double get(const double* p) {
    if (p == g_state + kStOver && g_scenario != 0) {
        static std::atomic<int> reads[kWaves];
        const int w = (int)threadIdx.x / 64;
        if (reads[w]++ == 0) return (w == 0) == (g_scenario == 1) ? 1.0 : 0.0;
        return 1.0;
    }
    return *p;
}
void put(double* p, double v) { *p = v; }
void drain() {}
void sleep_(int) { std::this_thread::yield(); }
#define __builtin_amdgcn_s_sleep sleep_
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __hip_atomic_fetch_add(p, v, o, s) __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST)
#define __hip_atomic_load(p, o, s) __atomic_load_n(p, __ATOMIC_SEQ_CST)
#define __hip_atomic_store(p, v, o, s) __atomic_store_n(p, v, __ATOMIC_SEQ_CST)
#define __HIP_MEMORY_SCOPE_AGENT 0

template <typename T, int BITS>
void sopt_share(const T*, const uint32_t*, const uint32_t*, int, int64_t, int share, int shares, T, double* tot) {
    if (g_rounds++ > 100 * kWaves) {
        std::puts("a wave goes round without a ticket");
        std::fflush(stdout);
        std::_Exit(2);
    }
    if (share < 0 || share >= shares) std::_Exit(3);
    if (threadIdx.x == 0) {
        g_shares++;
        for (int k = 0; k < kSoptPart; k++) tot[k] = share + 1;
    }
    __syncthreads();
}
template <class Get>
void sopt_total(const double* part, int shares, double* tot, Get g) {
    if (threadIdx.x == 0)
        for (int k = 0; k < kSoptPart; k++) {
            tot[k] = 0.0;
            for (int b = 0; b < shares; b++) tot[k] += g(part + b * kSoptPart + k);
        }
    __syncthreads();
}
double flat_of(bool) { return 0.0; }
int g_updates = 0;
void sopt_update(const double* tot, const double* now, int64_t, int, double, double, double* next, double*, bool) {
    if (tot[0] != kShares * (kShares + 1) / 2) std::_Exit(4);
    for (int k = 0; k < kStLen; k++) next[k] = now[k];
    next[kStOver] = ++g_updates == kPasses ? 1.0 : 0.0;
}

#include KERNEL

int main(int argc, char** argv) {
    g_scenario = argc > 1 ? std::atoi(argv[1]) : 0;
    float llr = 0.0f;
    uint32_t tx = 0, labels = 0;
    double out[16] = {};
    // a late block: the search has ended, its tickets and its end are published
    if (g_scenario != 0) {
        uint32_t* sync = (uint32_t*)(g_state + kStSync);
        sync[kSyncTicket] = sync[kSyncDone] = kPasses * kShares;
        sync[kSyncPass] = kSoptOver;
    }
    std::vector<std::thread> waves;
    for (int w = 0; w < kWaves; w++)
        waves.emplace_back([&, w] {
            threadIdx.x = 64 * w;
            k_sopt_rest<float, 4>(&llr, &tx, &labels, 16, 1, kShares, 1e-7, g_state, g_part, out);
            wave_ended();
        });
    for (auto& t : waves) t.join();
    const int want = g_scenario == 0 ? kPasses * kShares : 0;
    std::printf("shares %d of %d, updates %d\n", (int)g_shares, want, g_updates);
    return g_shares == want && g_updates == (g_scenario == 0 ? kPasses : 0) ? 0 : 5;
}

// Launch-shape autotuner of the block-sigma kernel: times the candidate
// shapes (team width, software-pipeline depth, workgroups per CU) on the
// problem at hand with HIP events and keeps the fastest.  Results are cached
// per process, keyed by device architecture, plan version, precision, block
// size and problem-size class, and optionally in a text file named by
// HINQS_TUNE_CACHE.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <fstream>
#include <map>
#include <mutex>
#include <string>

#include "common.hpp"

namespace hinqs {

namespace {

int env_flag(const char *name) {
    const char *v = std::getenv(name);
    return (v && *v) ? std::atoi(v) : 0;
}

int kindex(int k) { return k <= 1 ? 0 : k <= 2 ? 1 : k <= 4 ? 2 : k <= 8 ? 3 : 4; }

// Process-wide cache of tuned shapes keyed by (device arch, precision, k, problem-size bucket).
std::mutex g_tune_mutex;
std::map<std::string, SigmaCfg> g_tune_cache;

// The kernels that a plan's numbers mean: raised when a field changes its meaning or
// its kernel is replaced, so that plans saved for other kernels are tuned again.
constexpr int PLAN_VERSION = 2;

std::string tune_key(const Ctx &c, int k, int precision) {
    hipDeviceProp_t prop;
    std::string arch = "gpu";
    if (hipGetDeviceProperties(&prop, c.device) == hipSuccess) arch = prop.gcnArchName;
    const int dbucket = c.ndet > 0 ? (int)std::lround(2.0 * std::log2((double)c.ndet)) : 0;
    const int nbucket = c.ndet > 0 ? (int)std::lround((double)c.nnz / (double)c.ndet / 16.0) : 0;
    // sets on either side of SIGMA_SMALL_ROWS take different kernels and share a bucket
    return arch + "|v" + std::to_string(PLAN_VERSION) + "|p" + std::to_string(precision) + "|k" + std::to_string(k) +
           (c.ndet <= SIGMA_SMALL_ROWS ? "|s" : "|d") + std::to_string(dbucket) + "|n" + std::to_string(nbucket);
}

void load_tune_file() {
    static bool loaded = false;
    if (loaded) return;
    loaded = true;
    const char *path = std::getenv("HINQS_TUNE_CACHE");
    if (!path || !*path) return;
    std::ifstream f(path);
    std::string key;
    SigmaCfg g;
    while (f >> key >> g.team >> g.unr >> g.occ >> g.pipe >> g.ms) g_tune_cache[key] = g;
}

void store_tune_file() {
    const char *path = std::getenv("HINQS_TUNE_CACHE");
    if (!path || !*path) return;
    std::ofstream f(path, std::ios::trunc);
    for (const auto &kv : g_tune_cache)
        f << kv.first << " " << kv.second.team << " " << kv.second.unr << " " << kv.second.occ << " "
          << kv.second.pipe << " " << kv.second.ms << "\n";
}

}  // namespace

SigmaCfg autotune_sigma(Ctx &c, int k, int precision) {
    if (!c.have_elements) throw Error(HINQS_E_NOT_READY, "matrix elements are not built");
    if (precision != HINQS_FP64 && precision != HINQS_FP32)
        throw Error(HINQS_E_INVALID_ARG, "precision must be HINQS_FP64 or HINQS_FP32");
    const int K = k <= 1 ? 1 : k <= 2 ? 2 : k <= 4 ? 4 : k <= 8 ? 8 : 16;
    SigmaCfg &slot = c.sigma_cfg[precision == HINQS_FP64 ? 0 : 1][kindex(K)];
    const std::string key = tune_key(c, K, precision);
    {
        std::lock_guard<std::mutex> lk(g_tune_mutex);
        load_tune_file();
        auto it = g_tune_cache.find(key);
        if (it != g_tune_cache.end()) {
            slot = it->second;
            return slot;
        }
    }
    hipStream_t s = c.stream;
    const size_t esz = precision == HINQS_FP64 ? 8 : 4;
    DBuf<char> X, S;
    X.ensure((size_t)c.ndet * K * esz);
    S.ensure((size_t)c.ndet * K * esz);
    HQ_CHECK(hipMemsetAsync(X.p, 0, (size_t)c.ndet * K * esz, s));
    struct Events {
        hipEvent_t a = nullptr, b = nullptr;
        ~Events() {
            if (a) (void)hipEventDestroy(a);
            if (b) (void)hipEventDestroy(b);
        }
    } ev;
    HQ_CHECK(hipEventCreate(&ev.a));
    HQ_CHECK(hipEventCreate(&ev.b));
    const int vw = precision == HINQS_FP64 ? 2 : 4;
    const int lpn = K >= vw ? K / vw : 1;
    const bool verbose = env_flag("HINQS_VERBOSE") != 0;
    auto time_cfg = [&](SigmaCfg &g) {
        auto run = [&]() { sigma_launch(c, K, precision, g, X.p, K, S.p, K, s); };
        run();
        HQ_CHECK(hipEventRecord(ev.a, s));
        for (int r = 0; r < 3; ++r) run();
        HQ_CHECK(hipEventRecord(ev.b, s));
        HQ_CHECK(hipEventSynchronize(ev.b));
        float ms = 0.f;
        HQ_CHECK(hipEventElapsedTime(&ms, ev.a, ev.b));
        g.ms = ms / 3.0;
        if (verbose)
            std::fprintf(stderr, "[hinqs] tune k=%d p=%d pipe %d team %d unr %d occ %d: %.4f ms\n", K, precision,
                         g.pipe, g.team, g.unr, g.occ, g.ms);
    };
    // the default shape is kept unless a candidate is clearly (> 3 %) faster,
    // so the choice does not flip between near-equal shapes from run to run
    SigmaCfg best = default_cfg(c, K, precision);
    time_cfg(best);
    const int teams[] = {16, 32, 64};
    const int unrs[] = {2, 4};
    const int occs[] = {2, 4, 8};
    for (int team : teams) {
        if (team < 4 * lpn) continue;
        for (int unr : unrs) {
            if (unr == 2 && lpn >= 8) continue;  // the same kernel as 4
            for (int occ : occs) {
                SigmaCfg g;
                g.team = team;
                g.unr = unr;
                g.occ = occ;
                time_cfg(g);
                if (g.ms < 0.97 * best.ms) best = g;
            }
        }
    }
    slot = best;
    {
        std::lock_guard<std::mutex> lk(g_tune_mutex);
        g_tune_cache[key] = best;
        store_tune_file();
    }
    return best;
}

}  // namespace hinqs

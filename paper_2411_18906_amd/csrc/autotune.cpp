// Launch-shape tuning for the MC kernels (see autotune.h).
#include "autotune.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <sys/stat.h>

#include "mc_kernels.h"

namespace pyhea {

namespace {
std::mutex g_mu;
int g_forced = -1;
int g_forced_eval = -1;
int g_stream_G = 0, g_stream_threads = 0;
int g_forced_lookahead = 0;
bool g_measure = true;
bool g_graphs = true;

// measured shapes by key string; loaded from the cache file on first use
std::mutex g_tune_mu;
bool g_tune_loaded = false;
std::map<std::string, LaunchShape> g_tuned;

std::string device_tag() {
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return "unknown";
    std::string arch = prop.gcnArchName;
    const size_t colon = arch.find(':');
    if (colon != std::string::npos) arch = arch.substr(0, colon);
    return arch + "x" + std::to_string(prop.multiProcessorCount);
}

std::string key_string(const TuneKey &k) {
    char buf[160];
    // "mc2": shapes measured on kernels of another layout are not taken
    std::snprintf(buf, sizeof(buf), "mc2/%s/%d/%d/%d/%d/%d/%d", device_tag().c_str(), k.lattice, k.M, k.S, k.B,
                  k.nbucket, k.budget);
    return buf;
}

std::string cache_path() {
    if (const char *p = std::getenv("PYHEA_TUNE_CACHE")) return p;
    const char *home = std::getenv("HOME");
    if (!home || !*home) return "";
    return std::string(home) + "/.cache/pyhea/mc_launch_shapes.txt";
}

// lines: key store W K CH us_per_step (later lines override earlier ones)
void load_cache_locked() {
    if (g_tune_loaded) return;
    g_tune_loaded = true;
    const std::string path = cache_path();
    if (path.empty()) return;
    FILE *f = std::fopen(path.c_str(), "r");
    if (!f) return;
    char key[160];
    LaunchShape s{};
    double us = 0.0;
    while (std::fscanf(f, "%159s", key) == 1) {
        // the rest of the line: lines of another format are passed over
        char rest[128];
        if (!std::fgets(rest, sizeof(rest), f)) break;
        if (std::sscanf(rest, "%d %d %d %d %lf", &s.store, &s.W, &s.K, &s.CH, &us) != 5 ||
            std::strncmp(key, "mc2/", 4) != 0)
            continue;
        if (s.store < 0 || s.store > 2 || s.K < 1 || s.K > kMaxLookahead || s.W < 1 || s.W > kMaxWaves || s.CH < 1 ||
            s.CH > kChunk)
            continue;
        s.lds = 0;
        g_tuned[key] = s;
    }
    std::fclose(f);
}
}  // namespace

namespace {
int chunk_for(const Geometry &g) { return g.S * g.M * g.M <= 128 ? kChunk : kChunk / 2; }
}  // namespace

std::vector<LaunchShape> candidate_launches(const Geometry &g, int B, int lds_budget, int n_chains) {
    std::vector<LaunchShape> out;
    const int W = wave_budget(n_chains);
    for (int store : {(int)kStoreLds8, (int)kStoreLds4, (int)kStoreGlobal})
        for (int K : {kMaxLookahead, 1})
            for (int CH = chunk_for(g); CH >= 1; CH /= 2) {   // the largest chunk that fits
                const int64_t lds = mc_lds_bytes(g.S, g.M, B, CH) + species_store_bytes(store, g.Npad);
                if (lds > lds_budget) continue;
                out.push_back(LaunchShape{store, W, K, CH, (int)lds});
                break;
            }
    return out;
}

int64_t launch_lds_bytes(const Geometry &g, int B, const LaunchShape &s) {
    return mc_lds_bytes(g.S, g.M, B, s.CH) + species_store_bytes(s.store, g.Npad);
}

TuneKey tune_key(const Geometry &g, int B, int n_chains) {
    TuneKey k;
    k.lattice = g.lattice;
    k.M = g.M;
    k.S = g.S;
    k.B = B;
    k.nbucket = g.Npad > 0 ? (int)std::floor(std::log2((double)g.Npad)) : 0;
    k.budget = wave_budget(n_chains);
    return k;
}

bool tuned_launch(const TuneKey &k, LaunchShape *s) {
    const std::string key = key_string(k);
    std::lock_guard<std::mutex> lk(g_tune_mu);
    load_cache_locked();
    auto it = g_tuned.find(key);
    if (it == g_tuned.end()) return false;
    *s = it->second;
    return true;
}

void record_tuned_launch(const TuneKey &k, const LaunchShape &s, double us_per_step) {
    const std::string key = key_string(k);
    std::lock_guard<std::mutex> lk(g_tune_mu);
    load_cache_locked();
    g_tuned[key] = s;
    const std::string path = cache_path();
    if (path.empty()) return;
    // create the directory chain if needed (best effort; the cache is optional)
    for (size_t i = 1; i < path.size(); ++i)
        if (path[i] == '/') mkdir(path.substr(0, i).c_str(), 0755);
    if (FILE *f = std::fopen(path.c_str(), "a")) {
        std::fprintf(f, "%s %d %d %d %d %.4f\n", key.c_str(), s.store, s.W, s.K, s.CH, us_per_step);
        std::fclose(f);
    }
}

bool measure_enabled() {
    std::lock_guard<std::mutex> lk(g_mu);
    return g_measure;
}

void set_measure_enabled(bool on) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_measure = on;
}

bool graphs_enabled() {
    std::lock_guard<std::mutex> lk(g_mu);
    return g_graphs;
}

void set_graphs_enabled(bool on) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_graphs = on;
}

int wave_budget(int n_chains) {
    // every chain of a launch should be resident at once: 256 CUs x 16 wavefronts
    const int n = n_chains < 1 ? 1 : n_chains;
    return std::max(1, std::min(kMaxWaves, 4096 / n));
}

LaunchShape choose_launch(const Geometry &g, int B, int lds_budget, int variant, int n_chains) {
    int stores[3], ns = 0;
    if (variant == 2) {
        stores[ns++] = kStoreGlobal;
    } else if (variant == 1) {
        stores[ns++] = kStoreLds4;
        stores[ns++] = kStoreGlobal;
    } else {
        stores[ns++] = kStoreLds8;
        stores[ns++] = kStoreLds4;
        stores[ns++] = kStoreGlobal;
    }
    const int fk = forced_lookahead();
    const int W = std::max(wave_budget(n_chains), 4);
    const int K = fk > 0 ? fk : kMaxLookahead;
    const int ch0 = variant == 5 ? 1 : variant == 6 ? 4 : chunk_for(g);
    // the first store whose LDS holds the chain with chunks of at least half the
    // usual size, with as many members as fit
    LaunchShape best{kStoreGlobal, W, K, 1, mc_lds_bytes(g.S, g.M, B, 1)};
    for (int si = 0; si < ns; ++si)
        for (int CH = ch0; CH >= std::max(1, ch0 / 2); CH /= 2) {
            const int64_t lds = mc_lds_bytes(g.S, g.M, B, CH) + species_store_bytes(stores[si], g.Npad);
            if (lds <= lds_budget) return LaunchShape{stores[si], W, K, CH, (int)lds};
        }
    return best;
}

int forced_variant() {
    std::lock_guard<std::mutex> lk(g_mu);
    return g_forced;
}

void set_forced_variant(int v) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_forced = v;
}

int forced_eval_kernel() {
    std::lock_guard<std::mutex> lk(g_mu);
    return g_forced_eval;
}

void set_forced_eval_kernel(int v) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_forced_eval = v;
}

void forced_stream_shape(int *layers_per_group, int *threads) {
    std::lock_guard<std::mutex> lk(g_mu);
    *layers_per_group = g_stream_G;
    *threads = g_stream_threads;
}

void set_forced_stream_shape(int layers_per_group, int threads) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_stream_G = layers_per_group;
    g_stream_threads = threads;
}

int forced_lookahead() {
    std::lock_guard<std::mutex> lk(g_mu);
    return g_forced_lookahead;
}

void set_forced_lookahead(int k) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_forced_lookahead = k;
}


}  // namespace pyhea

// Launch-shape tuner of the labeling kernels: wavefronts per workgroup,
// timed on the device the first time a tune_key is seen, then cached for the
// process (and in the file named by SAL_TUNE_CACHE, if set).
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <tuple>
#include <utility>

#include "runtime.h"
#include "tune_cache.h"

namespace sal {
namespace {

std::mutex g_mu;
TuneMap g_cache;
bool g_loaded = false;

std::string arch_name(int device) {
    hipDeviceProp_t p;
    if (hipGetDeviceProperties(&p, device) != hipSuccess) return "unknown";
    return std::string(p.gcnArchName);
}

void load_file() {
    g_loaded = true;
    const char *path = std::getenv("SAL_TUNE_CACHE");
    if (path) tune_cache_read(path, &g_cache);
}

void save_file() {
    const char *path = std::getenv("SAL_TUNE_CACHE");
    if (path) tune_cache_write(path, g_cache);
}

}  // namespace

// Fills opt->points_per_lane (1) and opt->block_waves when it is 0 (auto).
sal_status tune_launch(sal_context *ctx, const sal_surface_set *set, int64_t n, const float *x,
                       const float *y, const float *z, int32_t *labels, sal_label_options *opt) {
    opt->points_per_lane = 1;   // the kernels hold one point per lane
    if (opt->block_waves != 0) return SAL_OK;
    const char *off = std::getenv("SAL_TUNE");
    if ((off && std::strcmp(off, "0") == 0) || n <= 0) {
        opt->block_waves = 4;
        return SAL_OK;
    }
    const TuneKey key = tune_key(ctx->device, opt->precision, set->n_tri, n, set->n_surf, arch_name(ctx->device));
    {
        std::lock_guard<std::mutex> lk(g_mu);
        if (!g_loaded) load_file();
        auto it = g_cache.find(key);
        if (it != g_cache.end()) {
            opt->block_waves = it->second.second;
            return SAL_OK;
        }
    }
    // Trial passes over a prefix of the points, writing labels that the real
    // launch overwrites: one untimed, so that the first shape does not also pay
    // for the device warming up, then one of each shape.  The result does not
    // depend on the shape.
    const int64_t trial_n = n < kTrialPoints ? n : kTrialPoints;
    LabelScratch sc = context_scratch(ctx);
    sc.counters = ctx->tune_counters;   // the call's own counters stay untouched
    sal_label_options trial = *opt;
    trial.winding_type = SAL_WINDING_NONE;
    trial.cull_bounds = 0;
    const int shapes[4] = {4, 1, 2, 8};
    float best = 1e30f;
    int best_b = 4;
    for (int k = -1; k < 4; ++k) {
        trial.block_waves = shapes[k < 0 ? 0 : k];
        SAL_HIP(hipEventRecord(ctx->ev[5], ctx->stream));
        const sal_status ts = enqueue_label_with(ctx, set, trial_n, nullptr, x, y, z, trial, labels, nullptr,
                                                 nullptr, ctx->stream, nullptr, sc);
        if (ts != SAL_OK) return ts;
        SAL_HIP(hipEventRecord(ctx->ev[6], ctx->stream));
        SAL_HIP(hipEventSynchronize(ctx->ev[6]));
        float ms = 0.0f;
        SAL_HIP(hipEventElapsedTime(&ms, ctx->ev[5], ctx->ev[6]));
        if (k >= 0 && ms < best) {
            best = ms;
            best_b = trial.block_waves;
        }
    }
    opt->block_waves = best_b;
    std::lock_guard<std::mutex> lk(g_mu);
    g_cache[key] = {opt->points_per_lane, opt->block_waves};
    save_file();
    return SAL_OK;
}

}  // namespace sal

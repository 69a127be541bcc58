// The launch-shape tuner's file cache: plain text, one entry per line.
#include "tune_cache.h"

#include <cstdio>

#include "runtime.h"

namespace sal {

namespace {

int bucket(int64_t v) {
    int b = 0;
    while (v > 1 && b < 62) {
        v >>= 1;
        ++b;
    }
    return b;
}

}  // namespace

TuneKey tune_key(int device, int precision, int64_t n_tri, int64_t n, int n_surf, const std::string &arch) {
    return TuneKey(device, precision, bucket(n_tri), bucket(n < kTrialPoints ? n : kTrialPoints), arch,
                   n <= kPointFormMax ? kTunePoints : kTuneGroups, bucket(n_surf));
}

bool tune_cache_read(const char *path, TuneMap *out) {
    if (!path || !out) return false;
    FILE *f = std::fopen(path, "r");
    if (!f) return false;
    char arch[128];
    int dev, prec, tri, points, form, surfaces, ppl, bw;
    while (std::fscanf(f, "%127s %d %d %d %d %d %d %d %d", arch, &dev, &prec, &tri, &points, &form,
                       &surfaces, &ppl, &bw) == 9)
        (*out)[TuneKey(dev, prec, tri, points, arch, form, surfaces)] = {ppl, bw};
    std::fclose(f);
    return true;
}

bool tune_cache_write(const char *path, const TuneMap &m) {
    if (!path) return false;
    FILE *f = std::fopen(path, "w");
    if (!f) return false;
    for (const auto &kv : m)
        std::fprintf(f, "%s %d %d %d %d %d %d %d %d\n", std::get<4>(kv.first).c_str(),
                     std::get<0>(kv.first), std::get<1>(kv.first), std::get<2>(kv.first),
                     std::get<3>(kv.first), std::get<5>(kv.first), std::get<6>(kv.first),
                     kv.second.first, kv.second.second);
    return std::fclose(f) == 0;
}

}  // namespace sal

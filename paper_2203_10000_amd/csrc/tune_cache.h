// The launch-shape tuner's file cache (host only, no device calls).
#pragma once

#include <cstdint>
#include <map>
#include <string>
#include <tuple>
#include <utility>

namespace sal {

// (device, precision, log2 triangles, log2 trial points, arch name, form, log2
// surfaces).  The form is the labeling kernels that the call runs: workgroup sizes
// measured on one say nothing of another, nor do those of one surface of many (in
// the point form the size also decides whether a point's surfaces are shared out).
// Files written before the forms were told apart have 0, 1, 2 or 4 in its place.
enum TuneForm { kTunePoints = 16, kTuneGroups = 17 };
using TuneKey = std::tuple<int, int, int, int, std::string, int, int>;
// -> (points per lane, wavefronts per workgroup)
using TuneMap = std::map<TuneKey, std::pair<int, int>>;

// Points of a trial at most: enough workgroups to fill the device, so that every
// larger count runs the same trials and shares their entry.
constexpr int64_t kTrialPoints = (int64_t)1 << 19;

// Key of a call on n points against n_surf surfaces of n_tri triangles in all.
TuneKey tune_key(int device, int precision, int64_t n_tri, int64_t n, int n_surf, const std::string &arch);

// One entry per line: "arch dev prec tri points form surfaces ppl bw".  Reading stops at
// the first line that does not parse (or has an arch name over 127 bytes)
// and keeps the entries before it; a missing file reads as empty.
bool tune_cache_read(const char *path, TuneMap *out);
bool tune_cache_write(const char *path, const TuneMap &m);

}  // namespace sal

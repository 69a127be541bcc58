// Host-side objects behind the opaque handles of sal.h.
#pragma once

#include <algorithm>
#include <vector>

#include "sal_internal.h"

// Device scratch owned by a context; grows, never shrinks.
struct sal_context {
    int device = 0;
    hipStream_t stream = nullptr;
    uint64_t stream_token = sal::new_stream_token();   // another with each set_stream
    hipEvent_t ev[8] = {};
    // flag list and spatial order of the wavefront-per-64-points form
    sal::FlagEntry *flag_list = nullptr;
    uint32_t *ord_idx1 = nullptr;
    uint16_t *ord_key1 = nullptr;
    uint32_t *ord_perm = nullptr;
    int64_t point_cap = 0;
    uint32_t *ord_hist = nullptr;
    int64_t tile_cap = 0;
    uint32_t *ord_tot = nullptr;
    int64_t inst_cap = 0;
    int32_t *span_w = nullptr;
    uint32_t *open_spans = nullptr;
    int64_t span_cap = 0;
    sal::PairBits *pairs = nullptr;
    int64_t pair_cap = 0;
    unsigned long long *work = nullptr;   // sal::kNumWork
    unsigned long long *counters = nullptr;  // sal::kNumCounters
    unsigned long long *tune_counters = nullptr;
    int64_t *host_words = nullptr;   // pinned: what a mesh call reads back
    int n_cu = 0;
    // batched form: the instance table on the device and its host copy
    sal::LabelInst *batch_insts = nullptr;
    int64_t batch_insts_cap = 0;
    std::vector<sal::LabelInst> batch_table;   // what batch_insts holds (empty: nothing)
    unsigned long long *batch_counters = nullptr;
    int64_t batch_counters_n = 0;
    hipStream_t capture_stream = nullptr;
    hipGraphExec_t batch_graph = nullptr;
    std::vector<uint64_t> batch_graph_fields;   // everything the graph reads or is shaped by
                                                // (empty: no valid graph)
};

struct sal_surface_set {
    uint64_t uid = 0;      // unique per creation (graph cache keys)
    int device = 0;
    int n_surf = 0;
    int64_t n_tri = 0, n_strips = 0, bytes = 0;   // (n_strips: leaf patches)
    sal::TriRec *rec = nullptr;
    sal::SurfaceDev *surf = nullptr;        // n_surf entries
    sal::PatchEntry *ent = nullptr;         // patch trees of all surfaces
    sal::LeafBox *leaf = nullptr;           // leaf boxes of all surfaces
    float lo[3] = {}, hi[3] = {};           // box of all surfaces
    std::vector<sal::SurfaceDev> host_table;
    bool balls_ready = false;              // ball_w of every surface known
};

namespace sal {

sal_status build_surface_set(sal_context *ctx, const sal_surface_desc *desc, int32_t n,
                             uint32_t flags, sal_surface_set **out);
void destroy_surface_set(sal_surface_set *set);

// Finds the winding number of each surface's ball centre (plain FP64 form,
// one launch per surface, synchronising the stream) the first time culling
// is asked for; until then no ball is used.
sal_status ensure_surface_balls(sal_context *ctx, const sal_surface_set *set);

// Points of one launch sequence: larger calls run in pieces (their scratch is
// some 34 bytes a point).
constexpr int64_t kChunkPoints = (int64_t)1 << 27;

// Up to this many points are labeled one per wavefront, in the order given.  The
// 64-point form pays six sorting launches first, and with few wavefronts on the
// chip the chain of one is the time.  Measured (us, point form / 64-point form;
// 16,384, 32,768 and 60,000 points): lattice points, one surface, 30 / 75, 50 / 77,
// 85 / 80; box points, four surfaces, 86 / 94, 155 / 108, 267 / 109; points near
// two surfaces of 162,000 triangles, 75 / 276, 141 / 286, 249 / 296.
constexpr int64_t kPointFormMax = 32768;

// The same for an instance of a batch, whose other instances fill the chip.  Where
// those between kBatchCrowdMin and this are many, their points together are past the
// point form's range and the sort of each pays; below kBatchCrowdMin the sort's 2048
// bins an instance cost more (us, point form / 64-point form; one surface of 320
// triangles, four of 5,120): 8 instances of 8,000 points 116 / 108, 231 / 194; 32 of
// 4,000 257 / 214, 474 / 402; 256 of 8,000 3356 / 1384, 6332 / 3013; but 8 of 4,000
// 78 / 104, 135 / 171; 128 of 1,000 511 / 531, 728 / 1272.
constexpr int64_t kBatchPointMax = 8192, kBatchCrowdMin = 2048, kBatchCrowd = 65536;

// Instances of up to so many points take the point form; sizes: of all instances.
inline int64_t batch_point_max(const std::vector<int64_t> &sizes) {
    int64_t crowd = 0;
    for (const int64_t n : sizes)
        if (n > kBatchCrowdMin && n <= kBatchPointMax) crowd += n;
    return crowd >= kBatchCrowd ? kBatchCrowdMin : kBatchPointMax;
}

// Tile size and count of the spatial order for n points: up to kSmallOrder small
// tiles, so that there is a workgroup for each CU (us, tiles of 2048 / 1024: 196,608
// lattice points 88 / 83, 200,003 box points 142 / 135, 60,001 points near two
// surfaces 280 / 267); above, the bins of more tiles cost more than that gives (two
// rounds under 20 surfaces 2616 / 2647).
constexpr int64_t kSmallOrder = (int64_t)1 << 18;
inline int32_t order_tile(int64_t n) {
    int64_t tile = n <= kSmallOrder ? kMinTile : 2 * kMinTile;
    while ((n + tile - 1) / tile > kMaxTiles) tile *= 2;
    return (int32_t)tile;
}
inline int64_t order_tiles(int64_t n) { return (n + order_tile(n) - 1) / order_tile(n); }

// The most tiles that any m <= n points have: where the tiles double their number
// halves, so n itself may have fewer (262,144 points 256, 262,145 points 129).
inline int64_t order_tiles_upto(int64_t n) {
    int64_t most = order_tiles(n);
    if (n > kSmallOrder) most = std::max(most, order_tiles(kSmallOrder));
    if (n > 2 * kMinTile * kMaxTiles) most = kMaxTiles;
    return most;
}

// From this many (point, surface) pairs on, a pass over spans of 512 points
// settles most of them first.  Below, its one more serial launch costs what it
// saves.
constexpr int64_t kSpanPairs = (int64_t)1 << 20;
inline int64_t span_count(int64_t n) { return (n + kSpanPoints - 1) / kSpanPoints; }

// Wavefronts per CU that share the open pairs: four times what its registers hold
// at once, so that the last ones even out (6M lattice points, 20 surfaces in two
// rounds, 24 instances; us): 24 872, 2998, 1208; 64 822, 2893, 1142.
constexpr int kPairWaves = 64;
inline int64_t group_count(int64_t n) { return (n + 63) / 64; }

// What one launch sequence of the 64-point form needs.
struct ScratchSize {
    int64_t points = 0, tiles = 0, insts = 0, spans = 0, pairs = 0;   // (spans, pairs: x surfaces)
};
// Grows the context's labeling scratch to hold it.
sal_status ensure_label_scratch(sal_context *ctx, const ScratchSize &need);

// What a call on up to n points against n_surf surfaces needs (nothing for the
// point form).  It never falls as n grows: a round sizes the scratch for its
// largest level, the tuner's trials run on a part of the points.
inline ScratchSize label_scratch_size(int64_t n, int n_surf) {
    ScratchSize z;
    if (n <= kPointFormMax) return z;
    const int64_t c = std::min(n, kChunkPoints);
    z.points = c;
    z.tiles = order_tiles_upto(c);
    z.insts = 1;
    z.spans = span_count(c) * n_surf;
    z.pairs = group_count(c) * n_surf;
    return z;
}
// Grows the scratch for such a call.
sal_status ensure_label_scratch(sal_context *ctx, const sal_surface_set *set, int64_t n);

// Validated options with defaults applied.
sal_status resolve_options(const sal_label_options *in, sal_label_options *out);

// Enqueues one labeling pass (winding numbers, and the recheck) of n points;
// counters must be cleared by the caller.  The launch shape is resolved first
// (tune_launch); then ev_start (before the first kernel) and ev_after_pairloop
// are recorded when non-null, so that timings bracketed by them leave out any
// tuning.
sal_status enqueue_label(sal_context *ctx, const sal_surface_set *set, int64_t n, const float *x,
                         const float *y, const float *z, const sal_label_options &opt,
                         int32_t *labels, void *winding, hipEvent_t ev_start,
                         hipEvent_t ev_after_pairloop, int *shape = nullptr,
                         unsigned long long *masks = nullptr);

// The device scratch one labeling pass works in.
struct LabelScratch {
    unsigned long long *counters;
    FlagEntry *flag_list;
    unsigned long long *work;
    int32_t *span_w;
    uint32_t *open_spans;
    PairBits *pairs;
    OrderScratch ord;
};

// The context's own scratch (sized by ensure_label_scratch).
LabelScratch context_scratch(const sal_context *ctx);

// The kernels' view of n points against a set; order, group and tile bases 0.
LabelInst make_inst(const sal_surface_set *set, int64_t n, const float *x, const float *y, const float *z,
                    int32_t *labels, void *winding, int64_t wstride, unsigned long long *masks,
                    unsigned long long *counters);

// The launches of one labeling pass with a resolved launch shape and the
// given scratch, on `stream`; the counters must be cleared by the caller.
sal_status enqueue_label_with(sal_context *ctx, const sal_surface_set *set, int64_t n,
                              const int64_t *n_dev, const float *x, const float *y,
                              const float *z, const sal_label_options &opt, int32_t *labels,
                              void *winding, hipEvent_t ev_mid, hipStream_t stream,
                              unsigned long long *masks, const LabelScratch &sc);

// Address of the allocation-free entry point's scratch array on `device`
// (looked up once per device, with the device current); nullptr on error.
void *noalloc_scratch(int device);

// The launches of one labeling pass with a resolved launch shape, on
// `stream`.  With n_dev set the point count is read on the device and n is the
// capacity the grids are sized for (the form a captured graph uses).
sal_status enqueue_label_on(sal_context *ctx, const sal_surface_set *set, int64_t n,
                            const int64_t *n_dev, const float *x, const float *y, const float *z,
                            const sal_label_options &opt, int32_t *labels, void *winding,
                            hipEvent_t ev_mid, hipStream_t stream,
                            unsigned long long *masks = nullptr);

// Resolves points_per_lane (1) and block_waves left at 0: the workgroup sizes
// are timed on a prefix of the points; the first use of a size bucket
// synchronises the stream.  Cached per process.
sal_status tune_launch(sal_context *ctx, const sal_surface_set *set, int64_t n, const float *x,
                       const float *y, const float *z, int32_t *labels, sal_label_options *opt);

}  // namespace sal
